// S9: the smoothing-length network (not in the paper): an 8 -> 64 -> 64 -> 1
// MLP with exact-erf GELU, FP32, whose output ln(H_conv / H_prev) seeds the
// iteration of eqs. (hi), (thacker). Features, inference, training (forward,
// backward, Adam) are all kernels here.
//
// Parameter vector (4801 floats): W1 [64][8], b1 [64], W2 [64][64], b2 [64],
// w3 [64], b3. Every kernel stages it in LDS (19 KB). The dense products of
// the forward and backward passes run on the matrix cores (FP32 MFMA), 16
// samples per wavefront. The batch gradient is reduced deterministically:
// one partial row per 16-sample tile, then a fixed-order sum over the rows
// (no float atomics).
#include <math.h>

#include <mutex>

#include "crk_internal.h"
#include "crk_rows.h"

namespace crk {
namespace {

constexpr int kIn = 8, kHid = 64;
constexpr int oW1 = 0, ob1 = oW1 + kHid * kIn, oW2 = ob1 + kHid, ob2 = oW2 + kHid * kHid,
              ow3 = ob2 + kHid, ob3 = ow3 + kHid, kNP = ob3 + 1;   // kNP = 4801
constexpr int kAdamLanes = 32;                                      // lanes summing one parameter's partials

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * __expf(-0.5f * x * x);
}

// (all loads before the first store: one wait for memory, not one a step)
__device__ __forceinline__ void load_theta(const float *__restrict__ th, float *s) {
    constexpr int N = (kNP + kBlock - 1) / kBlock;
    float t[N];
#pragma unroll
    for (int k = 0; k < N; k++) {
        const int e = threadIdx.x + k * kBlock;
        t[k] = th[e < kNP ? e : kNP - 1];
    }
#pragma unroll
    for (int k = 0; k < N; k++) {
        const int e = threadIdx.x + k * kBlock;
        if (e < kNP) s[e] = t[k];
    }
    __syncthreads();
}

// ---------------------------------------------------------------- matrix cores
// v_mfma_f32_16x16x4_f32: D[16x16] = A[16x4] B[4x16] + C with, for lane l,
// c = l % 16 and g = l / 16: A[c][g], B[g][c] and D[4g + r][c] (r = 0..3).
typedef float f4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4v mfma4(float a, float b, f4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Forward on the matrix cores, 16 samples (the columns) per wavefront step.
// Layer 1: Z1 = W1 F as four 16-row tiles over two k-steps. Layer 2: Z2 = W2
// A1, where the k-step (mt, r) takes the hidden units 16 mt + 4 g + r, i.e.
// the values each lane already holds in register r of tile mt (the sum over
// k runs in a permuted order, so no data moves between lanes); the matching
// W2 entries are per-lane constants. Output: each lane's share of w3.a2,
// then a sum over the four lane groups of a column.
__global__ __launch_bounds__(kBlock) void k_hnet_fwd(const float *__restrict__ theta,
                                                     const float *__restrict__ feat, int64_t nb,
                                                     float *y) {
    __shared__ float s[kNP];
    load_theta(theta, s);
    const int lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    float w1a[4][2], w2a[4][4][4], b1r[4][4], b2r[4][4], w3r[4][4];
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++) w1a[mt][ks] = s[oW1 + (16 * mt + c) * kIn + 4 * ks + g];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int h = 16 * mt + 4 * g + r;   // the hidden unit of register r of tile mt
            b1r[mt][r] = s[ob1 + h];
            b2r[mt][r] = s[ob2 + h];
            w3r[mt][r] = s[ow3 + h];
#pragma unroll
            for (int m2 = 0; m2 < 4; m2++) w2a[m2][mt][r] = s[oW2 + (16 * m2 + c) * kHid + h];
        }
    }
    const float b3 = s[ob3];
    const int64_t wstep = (int64_t)gridDim.x * (kBlock / 64) * 16;
    for (int64_t t0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * 16; t0 < nb; t0 += wstep) {
        const int64_t smp = t0 + c;
        const bool act = smp < nb;
        f4v z1[4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++) z1[mt] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            const float bf = act ? feat[(int64_t)(4 * ks + g) * nb + smp] : 0.0f;
#pragma unroll
            for (int mt = 0; mt < 4; mt++) z1[mt] = mfma4(w1a[mt][ks], bf, z1[mt]);
        }
        float a1[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++) a1[mt][r] = gelu(z1[mt][r] + b1r[mt][r]);
        f4v z2[4];
#pragma unroll
        for (int m2 = 0; m2 < 4; m2++) z2[m2] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int m2 = 0; m2 < 4; m2++) z2[m2] = mfma4(w2a[m2][mt][r], a1[mt][r], z2[m2]);
        float part = 0.0f;
#pragma unroll
        for (int m2 = 0; m2 < 4; m2++)
#pragma unroll
            for (int r = 0; r < 4; r++) part += w3r[m2][r] * gelu(z2[m2][r] + b2r[m2][r]);
        part += __shfl_xor(part, 16);
        part += __shfl_xor(part, 32);
        if (g == 0 && act) y[smp] = part + b3;
    }
}

// Sum over the 16 lanes of a DPP row (every lane gets the total)
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum16(float x) {
    x += dpp_f32<0xB1>(x);    // quad_perm(1,0,3,2)
    x += dpp_f32<0x4E>(x);    // quad_perm(2,3,0,1)
    x += dpp_f32<0x141>(x);   // row_half_mirror
    x += dpp_f32<0x140>(x);   // row_mirror
    return x;
}

// Gradient on the matrix cores: a block takes a tile of 16 samples (the
// columns; lane c = l % 16 is a sample, g = l / 16 picks four hidden units
// per register tile), its wavefront w the hidden units 16 w .. 16 w + 15 of
// each layer, and writes one partial gradient row. Forward as in k_hnet_fwd.
// Backward: dZ2 = dy w3 gelu'(z2) in the same layout; dA1 = W2^T dZ2 on the
// matrix cores with the permuted k order of the forward; dZ1 = dA1 gelu'(z1).
// What the other wavefronts' units are needed for passes through LDS (row
// stride 17). Weight gradients are sums over the tile's samples, so the sample
// index becomes the k of the product: dW2 = dZ2 A1^T, db2 (a column of ones),
// dW1 = dZ1 F^T and db1 (F padded with a row of ones) run on the matrix cores
// from the transposed tiles; dw3 and db3 are row sums over the 16 sample
// lanes. Bound by the latency of this chain (8192 samples are two tiles a CU):
// a wavefront per tile, four tiles a block, took 31 us of them, this 16.
constexpr int kTS = 17;   // LDS row stride of the 64 x 16 tiles
__global__ __launch_bounds__(kBlock) void k_hnet_grad(const float *__restrict__ theta,
                                                      const float *__restrict__ feat,
                                                      const float *__restrict__ target, int64_t nb,
                                                      float inv_b, float *partial, float *ploss) {
    static_assert(kBlock == 256, "a wavefront per 16 of 64 hidden units");
    __shared__ float s[kNP];
    __shared__ float Ta1[kHid * kTS], Tg2[kHid * kTS], Tdz2[kHid * kTS], Tdz1[kHid * kTS];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int64_t tile = blockIdx.x;
    const int64_t smp = tile * 16 + c;
    const bool act = smp < nb;
    const float tgt = act ? target[smp] : 0.0f;
    float bf[2], fb[4];   // F, and B of dW1: F[c][s] for c < 8, ones for c == 8 (db1), else 0
#pragma unroll
    for (int ks = 0; ks < 2; ks++) bf[ks] = act ? feat[(int64_t)(4 * ks + g) * nb + smp] : 0.0f;
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
        const int64_t sk = tile * 16 + 4 * ks + g;
        fb[ks] = c < kIn ? (sk < nb ? feat[(int64_t)c * nb + sk] : 0.0f) : (c == kIn ? 1.0f : 0.0f);
    }
    load_theta(theta, s);
    const int h0 = 16 * w + 4 * g;   // this lane's units h0 .. h0 + 3
    // forward
    f4v z1 = f4v{0.0f, 0.0f, 0.0f, 0.0f}, z2 = z1, da1 = z1;
#pragma unroll
    for (int ks = 0; ks < 2; ks++) z1 = mfma4(s[oW1 + (16 * w + c) * kIn + 4 * ks + g], bf[ks], z1);
#pragma unroll
    for (int r = 0; r < 4; r++) {
        z1[r] += s[ob1 + h0 + r];
        Ta1[(h0 + r) * kTS + c] = gelu(z1[r]);
    }
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < 4; mt++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int h = 16 * mt + 4 * g + r;
            z2 = mfma4(s[oW2 + (16 * w + c) * kHid + h], Ta1[h * kTS + c], z2);
        }
    float g2[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
        z2[r] += s[ob2 + h0 + r];
        g2[r] = gelu(z2[r]);
        Tg2[(h0 + r) * kTS + c] = g2[r];
    }
    __syncthreads();
    float part = 0.0f;
#pragma unroll
    for (int m2 = 0; m2 < 4; m2++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int h = 16 * m2 + 4 * g + r;
            part += s[ow3 + h] * Tg2[h * kTS + c];
        }
    part += __shfl_xor(part, 16);
    part += __shfl_xor(part, 32);
    const float res = act ? part + s[ob3] - tgt : 0.0f;
    const float dy = 2.0f * res * inv_b;
    float *out = partial + tile * kNP;
    // loss and db3: sums over the tile's samples
    const float lsum = row_sum16(res * res), dysum = row_sum16(dy);
    if (threadIdx.x == 0) {
        ploss[tile] = lsum;
        out[ob3] = dysum;
    }
    // dZ2 (and dw3 from the same registers)
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int h = h0 + r;
        Tdz2[h * kTS + c] = dy * s[ow3 + h] * gelu_d(z2[r]);
        const float dw3 = row_sum16(dy * g2[r]);
        if (c == 0) out[ow3 + h] = dw3;
    }
    __syncthreads();
    // dA1 = W2^T dZ2, then dZ1
#pragma unroll
    for (int m2 = 0; m2 < 4; m2++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int h = 16 * m2 + 4 * g + r;
            da1 = mfma4(s[oW2 + h * kHid + 16 * w + c], Tdz2[h * kTS + c], da1);
        }
#pragma unroll
    for (int r = 0; r < 4; r++) Tdz1[(h0 + r) * kTS + c] = da1[r] * gelu_d(z1[r]);
    // (the tiles below are this wavefront's own rows, but A1, which is there)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // dW2 and db2: k = the tile's samples
    float av[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) av[ks] = Tdz2[(16 * w + c) * kTS + 4 * ks + g];
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
        f4v acc = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 4; ks++) acc = mfma4(av[ks], Ta1[(16 * mt + c) * kTS + 4 * ks + g], acc);
#pragma unroll
        for (int r = 0; r < 4; r++) out[oW2 + (h0 + r) * kHid + 16 * mt + c] = acc[r];
    }
    f4v acc = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 4; ks++) acc = mfma4(av[ks], c == 0 ? 1.0f : 0.0f, acc);
    if (c == 0)
#pragma unroll
        for (int r = 0; r < 4; r++) out[ob2 + h0 + r] = acc[r];
    // dW1 (columns 0..7) and db1 (column 8)
    acc = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 4; ks++) acc = mfma4(Tdz1[(16 * w + c) * kTS + 4 * ks + g], fb[ks], acc);
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int h = h0 + r;
        if (c < kIn) out[oW1 + h * kIn + c] = acc[r];
        else if (c == kIn) out[ob1 + h] = acc[r];
    }
}

// Fixed-order sum of the partial rows, then one Adam step per parameter
// (bias-corrected, beta1 0.9, beta2 0.999, eps 1e-8). kAdamLanes running sums a
// parameter, sum c over the rows c, c + kAdamLanes, ..., added up as a binary
// tree. A block takes kAdamPar parameters, so that a row is read 64 bytes at a
// time (a lane per sum and row read a line of which it used four). One more
// block sums the loss in the order of the tiles, beside the others.
constexpr int kAdamPar = 16, kAdamBlocks = (kNP + kAdamPar - 1) / kAdamPar;
__global__ __launch_bounds__(kBlock) void k_hnet_adam(const float *__restrict__ partial,
                                                      const float *__restrict__ ploss, int64_t nblk,
                                                      float *theta, float *m, float *v, float lr,
                                                      float bc1, float bc2, float *grad_out, float inv_b,
                                                      float *loss) {
    constexpr int kGroups = kBlock / kAdamPar, kSums = kAdamLanes / kGroups;
    __shared__ __align__(16) float s[1024];
    static_assert(kAdamLanes * kAdamPar <= 1024, "the running sums fit");
    if (blockIdx.x == kAdamBlocks) {
        float L = 0.0f;
        for (int64_t b0 = 0; b0 < nblk; b0 += 1024) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 1024; k += kBlock)
                s[k + threadIdx.x] = b0 + k + threadIdx.x < nblk ? ploss[b0 + k + threadIdx.x] : 0.0f;
            __syncthreads();
            // (zeros follow the last tile)
            const int q = nblk - b0 < 1024 ? (int)(nblk - b0) : 1024;
            if (threadIdx.x == 0)
                for (int k = 0; k < q; k += 64)
#pragma unroll
                    for (int u = 0; u < 64; u++) L += s[k + u];
        }
        if (threadIdx.x == 0) loss[0] = L * inv_b;
        return;
    }
    const int p = threadIdx.x % kAdamPar, c0 = threadIdx.x / kAdamPar;
    const int e = blockIdx.x * kAdamPar + p;
    float g[kSums];
#pragma unroll
    for (int q = 0; q < kSums; q++) g[q] = 0.0f;
    // eight rows of a running sum in flight at a time
    const float *pe = partial + (e < kNP ? e : 0);
    for (int64_t b = c0; b < nblk; b += 8 * kAdamLanes) {
        float x[8][kSums];
#pragma unroll
        for (int u = 0; u < 8; u++)
#pragma unroll
            for (int q = 0; q < kSums; q++) {
                const int64_t r = b + u * kAdamLanes + q * kGroups;
                x[u][q] = pe[(r < nblk ? r : nblk - 1) * kNP];
            }
#pragma unroll
        for (int u = 0; u < 8; u++)
#pragma unroll
            for (int q = 0; q < kSums; q++)
                if (b + u * kAdamLanes + q * kGroups < nblk) g[q] += x[u][q];
    }
#pragma unroll
    for (int q = 0; q < kSums; q++) s[(c0 + q * kGroups) * kAdamPar + p] = g[q];
    __syncthreads();
    if (threadIdx.x >= kAdamPar || e >= kNP) return;
    float t[kAdamLanes];
#pragma unroll
    for (int q = 0; q < kAdamLanes; q++) t[q] = s[q * kAdamPar + p];
#pragma unroll
    for (int o = 1; o < kAdamLanes; o <<= 1)
#pragma unroll
        for (int q = 0; q < kAdamLanes; q += 2 * o) t[q] += t[q + o];
    const float gs = t[0];
    if (grad_out) grad_out[e] = gs;
    if (!theta) return;
    float mm = 0.9f * m[e] + 0.1f * gs;
    float vv = 0.999f * v[e] + 0.001f * gs * gs;
    m[e] = mm;
    v[e] = vv;
    theta[e] -= lr * (mm / bc1) / (sqrtf(vv / bc2) + 1e-8f);
}

// Features at radius H: kernel-weighted counts N_w(h) = (4 pi/3) h^3 sum
// W(r, h) at h = H, H/2, H/4 and raw counts within H and H/2 (self
// included), see crk.h for the eight definitions. G lanes per particle
// share the candidates and combine their five sums at the end, and each forms
// one of the features (one logarithm a lane, where the first lane's six kept
// the others waiting). When the
// last build's gather rows are given and a particle's H is the support they
// were built with, its row is the candidate set (it holds every j with r < H,
// self aside); otherwise a flattened walk of its support. With the rows
// tiled through LDS and two partners loading ahead, 64^3 takes 106 us, 212
// with the entries read one by one.
template <int G>
__global__ __launch_bounds__(kBlock) void k_hnet_features(const double4 *__restrict__ posH,
                                                          const int32_t *__restrict__ cbeg,
                                                          const int32_t *__restrict__ cend, Levels v,
                                                          int64_t n, const double *__restrict__ H,
                                                          const int64_t *__restrict__ goff,
                                                          const int32_t *__restrict__ gidx,
                                                          double Nres, float *feat) {
    const int64_t gid = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int l = (int)(gid % G);
    const int64_t i = gid / G;
    if (i >= n) return;   // whole groups leave together
    const double4 pi = posH[i];
    const double h = H[i];
    double s1 = 0.0, s2 = 0.0, s4 = 0.0, c1 = 0.0, c2 = 0.0;
    const double h2 = h * h, ih = 1.0 / h;
    const auto weight = [](double q) {
        const double w = 1.0 - q, w2 = w * w;
        return w2 * w2 * w2 * (1.0 + q * (6.0 + q * (35.0 / 3.0)));
    };
    // a partner within h at distance h q
    const auto add = [&](double r2, double q) {
        s1 += weight(q);
        if (r2 < 0.25 * h2) {
            s2 += weight(2.0 * q);
            c2 += 1.0;
            if (r2 < 0.0625 * h2) s4 += weight(4.0 * q);
        }
    };
    static_assert(G == 8, "a lane per feature");
    // a wavefront's rows and the tables of its walks, one after the other, so
    // that five blocks fit a CU
    constexpr int NR = flat_ranges<G>(), NG = 64 / G;
    struct Walks {
        int32_t b[NG][NR], c[NG][NR + 1];
        double x[NG][3 * NR];
        AxisTab ax[NG];
    };
    __shared__ union {
        Walks walks;
        RowTile<G, 4> rows;
    } s_w[kBlock / 64];
    auto &sw = s_w[threadIdx.x >> 6];
    if (goff && h == pi.w) {
        if (l == 0) add(0.0, 0.0);   // self
        const int64_t b = goff[i];
        const int cnt = (int)(goff[i + 1] - b);
        const Box box{v.L, 1.0 / v.L};
        if (l == 0) c1 = (double)(cnt + 1);
        row_sum<G, 2>(sw.rows, gidx, b, cnt, (int32_t)i, threadIdx.x & 63, [&](int32_t j) { return posH[j]; },
                      [&](const double4 &pj) {
            const double r2 = r2_exact(pair_image(pi.x - pj.x, box), pair_image(pi.y - pj.y, box),
                                       pair_image(pi.z - pj.z, box));
            add(r2, sqrt_dist(r2) * ih);
        });
    } else {
        const int grp = (threadIdx.x & 63) / G;
        flat_candidates<G, NR>(posH, cbeg, cend, v, i, pi, h, l, sw.walks.b[grp], sw.walks.c[grp], sw.walks.x[grp],
                               sw.walks.ax[grp],
                               [&](bool valid, double r2) {
                                   if (valid && r2 < h2) {
                                       add(r2, sqrt(r2) * ih);
                                       c1 += 1.0;
                                   }
                                   return false;
                               });
    }
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) {
        s1 += __shfl_xor(s1, m, G);
        s2 += __shfl_xor(s2, m, G);
        s4 += __shfl_xor(s4, m, G);
        c1 += __shfl_xor(c1, m, G);
        c2 += __shfl_xor(c2, m, G);
    }
    // (4 pi/3) h^3 * kW h^-3 sum = (4 pi/3) kW sum, the same at every radius
    const double c = 4.0 / 3.0 * kPi * kW;
    const double N1 = c * s1, N2 = c * s2, N4 = c * s4;
    // lane l forms feature l
    const double cb = cbrt(l == 6 ? (double)n : Nres / N1);
    double num = N1;
    if (l == 2) num = 8.0 * N2;
    if (l == 3) num = 64.0 * N4;
    if (l == 4) num = c1;
    if (l == 5) num = 8.0 * c2;
    if (l == 6) num = h * cb;
    float f = l == 1 ? (float)(cb - 1.0) : (float)log(num / (l == 6 ? v.L : Nres));
    if (l == 7) f = 1.0f;
    feat[l * n + i] = f;
}

// seed = H_prev exp(y), clamped to [H_prev / 8, 8 H_prev] and below L/2;
// a non-finite network output keeps H_prev
__global__ __launch_bounds__(kBlock) void k_hnet_seed(const double *__restrict__ Hprev,
                                                      const float *__restrict__ y, int64_t n,
                                                      double hmax, double *Hseed) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double h = Hprev[i];
    double o = (double)y[i];
    double s = isfinite(o) ? h * exp(o) : h;
    s = fmin(fmax(s, 0.125 * h), 8.0 * h);
    Hseed[i] = fmin(s, hmax);
}

__global__ __launch_bounds__(kBlock) void k_hnet_targets(const double *__restrict__ Hprev,
                                                         const double *__restrict__ Hconv, int64_t n,
                                                         float *t) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) t[i] = (float)log(Hconv[i] / Hprev[i]);
}

}  // namespace

// ---------------------------------------------------------------- allocation-free training step
// crk_hnet_train_step_noalloc keeps the partial gradient rows and losses of
// up to kStaticTiles 16-sample tiles in this file-scope device array instead
// of the context workspace. Each device holds its own copy (9.8 MB) until the
// process ends, and every call on that device shares it. Host code never
// passes the array's name to a kernel: it is a host-side stand-in there. The
// device address comes from hipGetSymbolAddress, taken once per device by
// hnet_scratch_init (called from crk_create with the device current).
constexpr int64_t kStaticTiles = 512;   // batches of up to 8192 samples
constexpr int64_t kStaticWords = kStaticTiles * (kNP + 1) + 64;
static __device__ __align__(256) float scratch[kStaticWords];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_dev[kMaxDevices] = {};
}  // namespace

crk_status hnet_scratch_init(crk_ctx *c) {
    if (c->device < 0 || c->device >= kMaxDevices)
        return set_err(c, CRK_ERR_INVALID_ARG, "device %d beyond the static scratch table", c->device);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_dev[c->device]) return CRK_OK;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
        (void)hipGetLastError();
        return set_err(c, CRK_ERR_HIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    }
    g_scratch_dev[c->device] = (float *)p;
    return CRK_OK;
}

static float *hnet_scratch(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_dev[device];
}

}  // namespace crk

using namespace crk;

extern "C" {

crk_status crk_hnet_features(crk_ctx *c, double Nres, const double *H_sorted, float *feat) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!H_sorted || !feat || !(Nres > 0.0)) return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_features: bad argument");
    if (c->nc == 0) return set_err(c, CRK_ERR_STATE, "crk_build_cells has not run");
    CRK_HIP(c, hipSetDevice(c->device));
    int64_t n = c->n;
    {
        KTimer kt_(c, "k_hnet_features");
        constexpr int GF = 8;
        // the gather rows serve the particles whose H is the one they were
        // built with (graph-mode lists are capacity-bound, so never those)
        const bool rows = c->built && !c->graph_mode;
        k_hnet_features<GF><<<(unsigned)((n * GF + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(
            (const double4 *)c->posH.p, (const int32_t *)c->cbeg.p, (const int32_t *)c->cend.p,
            levels(c), n, H_sorted, rows ? (const int64_t *)c->goff.p : nullptr,
            rows ? (const int32_t *)c->gidx.p : nullptr, Nres, feat);
    }
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

crk_status crk_hnet_forward(crk_ctx *c, const float *theta, const float *feat, int64_t nb, float *y) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!theta || !feat || !y || nb < 1) return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_forward: bad argument");
    CRK_HIP(c, hipSetDevice(c->device));
    {
        KTimer kt_(c, "k_hnet_fwd");
        // 16 samples per wavefront step; enough blocks to fill the device, each
        // wavefront striding over the batch
        const int64_t tiles = (nb + 15) / 16;
        int64_t nbk = (tiles + kBlock / 64 - 1) / (kBlock / 64);
        if (nbk > 4096) nbk = 4096;
        k_hnet_fwd<<<(unsigned)nbk, kBlock, 0, c->stream>>>(theta, feat, nb, y);
    }
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

crk_status crk_hnet_train_step(crk_ctx *c, float *theta, float *adam_m, float *adam_v, int64_t step,
                               float lr, const float *feat, const float *target, int64_t nb,
                               float *grad, float *loss) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!feat || !target || nb < 1 || (theta && (!adam_m || !adam_v || step < 1)) || (!theta && !grad))
        return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_train_step: bad argument");
    CRK_HIP(c, hipSetDevice(c->device));
    int64_t nblk = (nb + 15) / 16;   // one partial row per 16-sample tile
    CRK_TRY(ensure(c, c->hnet_part, (size_t)nblk * (kNP + 1) * sizeof(float) + 64));
    float *part = (float *)c->hnet_part.p;
    float *ploss = part + nblk * kNP;
    const float *th_in = theta;
    if (!theta) return set_err(c, CRK_ERR_INVALID_ARG, "theta is NULL");
    {
        KTimer kt_(c, "k_hnet_grad");
        k_hnet_grad<<<(unsigned)nblk, kBlock, 0, c->stream>>>(th_in, feat, target, nb, 1.0f / (float)nb, part, ploss);
    }
    // (the loss goes straight to host memory)
    float *pin = (float *)c->pinned.p + 256;
    float bc1 = 1.0f - powf(0.9f, (float)step), bc2 = 1.0f - powf(0.999f, (float)step);
    {
        KTimer kt_(c, "k_hnet_adam");
        k_hnet_adam<<<kAdamBlocks + (loss ? 1 : 0), kBlock, 0, c->stream>>>(
            part, ploss, nblk, lr > 0.0f ? theta : nullptr, adam_m, adam_v, lr, bc1, bc2, grad, 1.0f / (float)nb, pin);
    }
    CRK_HIP(c, hipGetLastError());
    if (loss) {
        CRK_HIP(c, hipStreamSynchronize(c->stream));
        *loss = pin[0];
    }
    return CRK_OK;
}

crk_status crk_hnet_train_step_noalloc(crk_ctx *c, float *theta, float *adam_m, float *adam_v,
                                       int64_t step, float lr, const float *feat,
                                       const float *target, int64_t nb, float *grad, float *loss) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!theta || !feat || !target || nb < 1 || (lr > 0.0f && (!adam_m || !adam_v || step < 1)))
        return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_train_step_noalloc: bad argument");
    if (nb > kStaticTiles * 16)
        return set_err(c, CRK_ERR_INVALID_ARG,
                       "crk_hnet_train_step_noalloc: %lld samples exceed the static scratch (at most %lld)",
                       (long long)nb, (long long)(kStaticTiles * 16));
    float *part = hnet_scratch(c->device);
    if (!part) return set_err(c, CRK_ERR_STATE, "static scratch address not set up for device %d", c->device);
    CRK_HIP(c, hipSetDevice(c->device));
    // the same kernels and partial layout as crk_hnet_train_step: every
    // partial row and loss of tiles 0 .. nblk-1 is written before it is read
    const int64_t nblk = (nb + 15) / 16;
    float *ploss = part + nblk * kNP;
    {
        KTimer kt_(c, "k_hnet_grad");
        k_hnet_grad<<<(unsigned)nblk, kBlock, 0, c->stream>>>(theta, feat, target, nb, 1.0f / (float)nb, part, ploss);
    }
    const float bc1 = 1.0f - powf(0.9f, (float)step), bc2 = 1.0f - powf(0.999f, (float)step);
    {
        KTimer kt_(c, "k_hnet_adam");
        k_hnet_adam<<<kAdamBlocks + (loss ? 1 : 0), kBlock, 0, c->stream>>>(
            part, ploss, nblk, lr > 0.0f ? theta : nullptr, adam_m, adam_v, lr, bc1, bc2, grad, 1.0f / (float)nb, loss);
    }
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

crk_status crk_hnet_targets(crk_ctx *c, int64_t n, const double *H_prev, const double *H_conv,
                            float *target) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (n < 1 || !H_prev || !H_conv || !target)
        return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_targets: bad argument");
    CRK_HIP(c, hipSetDevice(c->device));
    k_hnet_targets<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(H_prev, H_conv, n, target);
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

crk_status crk_hnet_seed(crk_ctx *c, const float *theta, double Nres, const double *H_prev, double *H_seed) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!theta || !H_prev || !H_seed) return set_err(c, CRK_ERR_INVALID_ARG, "crk_hnet_seed: bad argument");
    if (c->nc == 0) return set_err(c, CRK_ERR_STATE, "crk_build_cells has not run");
    CRK_HIP(c, hipSetDevice(c->device));
    int64_t n = c->n;
    CRK_TRY(ensure(c, c->hnet_feat, (size_t)n * (kIn + 1) * sizeof(float)));
    float *feat = (float *)c->hnet_feat.p, *y = feat + (size_t)n * kIn;
    CRK_TRY(crk_hnet_features(c, Nres, H_prev, feat));
    CRK_TRY(crk_hnet_forward(c, theta, feat, n, y));
    k_hnet_seed<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(H_prev, y, n,
                                                                                  0.49 * c->L, H_seed);
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

}  // extern "C"
