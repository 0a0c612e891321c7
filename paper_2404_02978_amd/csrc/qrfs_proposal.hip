// qrfs_proposal.hip -- learned proposal density for the frequency sampler:
// the 5 -> 128 -> 128 -> 2 network (forward, fused forward + backward,
// fixed-order gradient reduction, Adam), the sampling table (mixture over
// baselines plus a defensive share of the plain density, inverse CDF) and
// the learned R2 sampler with 1/q cell areas.
//
// Density over (ell = ln|f|, theta) for aperture D, outer scale L0 and a
// baseline of length |B| and direction theta_B:
//   q = p(ell) (1 + alpha(ell) cos 2(theta - theta_B)) / (2 pi),
//   p proportional to exp(o0), alpha = 0.9 tanh(o1),
// o = network(2 (ell - lmin)/Lw - 1, 2 theta_B/pi - 1, ln D / 4,
//             ln L0 / 4 - 1, ln|B| / 4 - 1/2).
#include <hip/hip_runtime.h>

#include "qrfs_device.hpp"
#include "qrfs_proposal.hpp"

namespace qrfs {
namespace prop {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int ROWS = 48;     // rows of a training tile: three 16-row matrix tiles
constexpr int ROWS_F = 64;   // rows of a tile of the forward-only kernels, which keep one matrix less
constexpr int THREADS = 512; // 8 waves, one per 16 hidden units
constexpr int ST = 132;      // floats per row of the LDS matrices: 16-byte rows, and the 16 lanes
                             // of a 16-byte operand read on 16 different groups of 4 banks

struct RowSpec {
    // rows [0, n_sample) are training samples of context ctxlist[q / m];
    // rows [n_sample, n_sample + n_grid) are normaliser grid points of
    // context ctxlist[(q - n_sample) / G]
    uint32_t n_sample, n_grid, m, G, n_ctx;
    const int32_t* ctxlist;
    const double* ctx4;     // [n_ctx][4] = D, L0, |B|, theta_B
    const double* ell;      // training rows
    const double* theta;
    const double* h;
    // per context slot, written by k_grid: sum of h, log Z, the four features
    // of its geometry; per grid row: exp(o0) / sum of exp(o0)
    double* Hc;
    double* logZ;
    float* feat;
    double* soft;
    double lmin, Lw;
};

// The network inputs that depend on the context only (x[1..4]).
__device__ __forceinline__ void context_features(const double* c, float x[4]) {
    x[0] = (float)(2.0 * c[3] / 3.141592653589793 - 1.0);
    x[1] = (float)(log(c[0]) / 4.0);
    x[2] = (float)(log(c[1]) / 4.0 - 1.0);
    x[3] = (float)(log(c[2]) / 4.0 - 0.5);
}
__device__ __forceinline__ float ell_feature(double ell, double lmin, double Lw) {
    return (float)(2.0 * (ell - lmin) / Lw - 1.0);
}

// Inputs of a row: the 5 features, 1 (for the bias of layer 1), 0, 0.
constexpr int XW = 8;

template <int NR>
struct NetSmem {
    __attribute__((aligned(16))) float W2[HID * ST];  // row i: weights of hidden unit i
    __attribute__((aligned(16))) float h1[NR * ST];   // activations, row-major
    __attribute__((aligned(16))) float h2[NR * ST];
    float W3[2 * HID];
    float b2[HID];
    float b3[2];
    float x[NR][XW];
};

// What a lane keeps of layer 1: the column of [W1 b1 0 0] that it feeds to the
// matrix instructions, of hidden unit 16 (t / 64) + t % 16.
struct Layer1 {
    float w[2];
};

template <int NR>
__device__ __forceinline__ Layer1 load_params(const float* __restrict__ prm, NetSmem<NR>& s) {
    const int t = threadIdx.x;
    for (int i = t; i < HID * HID / 2; i += THREADS) {  // pairs (OFF_W2 is even)
        const float2 v = ((const float2*)(prm + OFF_W2))[i];
        *(float2*)&s.W2[(2 * i / HID) * ST + 2 * i % HID] = v;
    }
    if (t < 2 * HID) s.W3[t] = prm[OFF_W3 + t];
    if (t < HID) s.b2[t] = prm[OFF_B2 + t];
    if (t < 2) s.b3[t] = prm[OFF_B3 + t];
    const int u = 16 * (t >> 6) + (t & 15), lh = (t & 63) >> 4;
    Layer1 l;
    l.w[0] = prm[OFF_W1 + u * 5 + lh];
    l.w[1] = lh == 0 ? prm[OFF_W1 + u * 5 + 4] : lh == 1 ? prm[OFF_B1 + u] : 0.0f;
    return l;
}

__device__ __forceinline__ void put_inputs(float (&x)[XW], float x0, const float f[4]) {
    x[0] = x0;
#pragma unroll
    for (int j = 0; j < 4; ++j) x[1 + j] = f[j];
    x[5] = 1.0f;
    x[6] = x[7] = 0.0f;
}

__device__ __forceinline__ f32x4 mfma_16(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Forward of the tile's rows (inputs in x, a barrier after them).  Leaves h1
// and h2 and returns, in the 8 threads of row r = t / 8, its outputs.  Wave w
// computes units [16 w, 16 w + 16) of all rows of both hidden layers with
// v_mfma_f32_16x16x4 (lane l: operand row l % 16; layer 1: contraction value
// 4 q + l / 16 in step q; layer 2: 4 (l / 16) + q of each 16; result rows
// 4 (l / 16) + i, column l % 16): FP32 products and sums at twice the rate of
// the vector ALU, whose one thread per (row, 32 units) this replaces.
template <int NR>
__device__ __forceinline__ void forward_tile(NetSmem<NR>& s, const float (*x)[XW],
                                             const Layer1& l1, float o[2]) {
    constexpr int MT = NR / 16;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, li = lane & 15, lh = lane >> 4;
    const int u = 16 * wave + li;
    {
        f32x4 acc[MT] = {};
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int m = 0; m < MT; ++m)
                acc[m] = mfma_16(x[16 * m + li][4 * q + lh], l1.w[q], acc[m]);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                s.h1[(16 * m + 4 * lh + i) * ST + u] = tanhf(acc[m][i]);
    }
    __syncthreads();
    f32x4 acc[MT] = {};
#pragma unroll
    for (int g = 0; g < HID / 16; ++g) {
        const f32x4 B = *(const f32x4*)&s.W2[u * ST + 16 * g + 4 * lh];
        f32x4 A[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
            A[m] = *(const f32x4*)&s.h1[(16 * m + li) * ST + 16 * g + 4 * lh];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = mfma_16(A[m][q], B[q], acc[m]);
    }
    const float b2 = s.b2[u];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s.h2[(16 * m + 4 * lh + i) * ST + u] = tanhf(acc[m][i] + b2);
    __syncthreads();
    // outputs: 8 threads per row, 16 units each, added in a fixed tree
    const int r = t >> 3, part = t & 7;
    float p0 = 0.0f, p1 = 0.0f;
    if (r < NR) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * part + 4 * j;
            const f32x4 hv = *(const f32x4*)&s.h2[r * ST + k];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p0 = fmaf(s.W3[k + e], hv[e], p0);
                p1 = fmaf(s.W3[HID + k + e], hv[e], p1);
            }
        }
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) {
        p0 += __shfl_xor(p0, off);
        p1 += __shfl_xor(p1, off);
    }
    o[0] = s.b3[0] + p0;
    o[1] = s.b3[1] + p1;
}

// Forward only: out[q][2] for rows q < n_rows (ell[q], ctx4[q]).  Blocks walk
// tiles, so the parameters are loaded once per block.
__global__ __launch_bounds__(THREADS) void k_forward(const float* __restrict__ prm, int64_t n_rows,
                                                     const double* __restrict__ ell,
                                                     const double* __restrict__ ctx4, double lmin,
                                                     double Lw, float* __restrict__ out) {
    __shared__ NetSmem<ROWS_F> s;
    const Layer1 l1 = load_params(prm, s);
    const int64_t n_tiles = (n_rows + ROWS_F - 1) / ROWS_F;
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int64_t base = tile * ROWS_F;
        if (threadIdx.x < ROWS_F) {
            const int64_t q = base + threadIdx.x;
            float x0 = 0.0f, f[4] = {0, 0, 0, 0};
            if (q < n_rows) {
                x0 = ell_feature(ell[q], lmin, Lw);
                context_features(ctx4 + 4 * q, f);
            }
            put_inputs(s.x[threadIdx.x], x0, f);
        }
        __syncthreads();
        float o[2];
        forward_tile(s, s.x, l1, o);
        const int64_t q = base + (threadIdx.x >> 3);
        if ((threadIdx.x & 7) == 0 && q < n_rows) {
            out[2 * q] = o[0];
            out[2 * q + 1] = o[1];
        }
        // (the barrier after the next inputs separates this tile's reads of h1, h2)
        __syncthreads();
    }
}

// The block's maximum or sum of v in a fixed order (red: one entry per wave).
template <bool MAX>
__device__ __forceinline__ double block_reduce(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double u = __shfl_xor(v, off);
        v = MAX ? fmax(v, u) : v + u;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) v = MAX ? fmax(v, red[w]) : v + red[w];
    return v;
}

// Per context slot c of a step.  Block c: the grid points' o0, log Z =
// log(sum_j exp(o0_j) Lw / G), the softmax over the grid and the context's
// features; block n_ctx + c: H_c, the sum of h over its sample rows.  All in a
// fixed order.
__global__ __launch_bounds__(THREADS) void k_grid(const float* __restrict__ prm, RowSpec rs,
                                                  float* __restrict__ og) {
    __shared__ NetSmem<ROWS_F> s;
    __shared__ double red[THREADS / 64];
    const int t = threadIdx.x;
    if (blockIdx.x >= rs.n_ctx) {
        const uint32_t c = blockIdx.x - rs.n_ctx;
        const double* h = rs.h + (int64_t)rs.ctxlist[c] * rs.m;
        double a = 0.0;
        uint32_t i = t;
        for (; i + 3 * THREADS < rs.m; i += 4 * THREADS) {
            double v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = h[i + e * THREADS];
#pragma unroll
            for (int e = 0; e < 4; ++e) a += v[e];
        }
        for (; i < rs.m; i += THREADS) a += h[i];
        a = block_reduce<false>(a, red);
        if (t == 0) rs.Hc[c] = a;
        return;
    }
    const uint32_t c = blockIdx.x;
    const Layer1 l1 = load_params(prm, s);
    float f[4];
    context_features(rs.ctx4 + 4 * (int64_t)rs.ctxlist[c], f);
    if (t == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) rs.feat[4 * c + j] = f[j];
    float* o = og + (size_t)c * rs.G;
    for (uint32_t g0 = 0; g0 < rs.G; g0 += ROWS_F) {
        if (t < ROWS_F) {
            const uint32_t j = g0 + t;
            put_inputs(s.x[t],
                       j < rs.G ? ell_feature(rs.lmin + (j + 0.5) * rs.Lw / rs.G, rs.lmin, rs.Lw)
                                : 0.0f,
                       f);
        }
        __syncthreads();
        float ov[2];
        forward_tile(s, s.x, l1, ov);
        const uint32_t j = g0 + (t >> 3);
        if ((t & 7) == 0 && j < rs.G) o[j] = ov[0];
        __syncthreads();
    }
    // this block's o0 back from memory (written by itself, before a barrier)
    __threadfence_block();
    double mx = -1e300;
    for (uint32_t j = t; j < rs.G; j += THREADS) mx = fmax(mx, (double)o[j]);
    mx = block_reduce<true>(mx, red);
    double se = 0.0;
    for (uint32_t j = t; j < rs.G; j += THREADS) se += exp((double)o[j] - mx);
    se = block_reduce<false>(se, red);
    for (uint32_t j = t; j < rs.G; j += THREADS)
        rs.soft[(size_t)c * rs.G + j] = exp((double)o[j] - mx) / se;
    if (t == 0) rs.logZ[c] = mx + log(se * rs.Lw / rs.G);
}

// 1 / sum of H_c (0 if the sum is not positive), in a fixed order; all lanes of
// a wave call it (one thread that adds H_c by H_c waits on each load: 4 us for
// 16 contexts).
__device__ __forceinline__ double inverse_H(const RowSpec& rs) {
    double H = 0.0;
    for (uint32_t c = threadIdx.x & 63; c < rs.n_ctx; c += 64) H += rs.Hc[c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) H += __shfl_xor(H, off);
    return H > 0.0 ? 1.0 / H : 0.0;
}

// Inputs of a training tile, row by row: a sample's weight w = -h / H and
// C = cos 2 (theta - theta_B); a normaliser's w = dL/do0 and C = 2, its mark.
struct TileRows {
    float x[ROWS][XW];
    double w[ROWS], C[ROWS];
};
__device__ __forceinline__ void load_row(const RowSpec& rs, double invH, uint32_t q, uint32_t r1,
                                         int r, TileRows& d) {
    float x0 = 0.0f, f[4] = {0, 0, 0, 0};
    double w = 0.0, C = 0.0;
    if (q < r1) {
        const bool sample = q < rs.n_sample;
        const uint32_t n = sample ? q : q - rs.n_sample, per = sample ? rs.m : rs.G;
        const uint32_t cs = n / per, j = n % per;
        double ell;
        if (sample) {
            const int64_t i = (int64_t)rs.ctxlist[cs] * rs.m + j;
            ell = rs.ell[i];
            w = -rs.h[i] * invH;
            C = cos(2.0 * (rs.theta[i] - rs.ctx4[4 * (int64_t)rs.ctxlist[cs] + 3]));
        } else {
            ell = rs.lmin + (j + 0.5) * rs.Lw / rs.G;
            w = rs.Hc[cs] * invH * rs.soft[n];
            C = 2.0;
        }
        x0 = ell_feature(ell, rs.lmin, rs.Lw);
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = rs.feat[4 * cs + e];
    }
    put_inputs(d.x[r], x0, f);
    d.w[r] = w;
    d.C[r] = C;
}

// A sum over the tiles of a block in two binary32 numbers; add() keeps what its
// rounding leaves over (Knuth's two-sum), so that however many rows a block has,
// binary32 rounds within a tile of 48 only.  RMS error of the gradient of 16
// contexts x 20000 rows, 1255 rows a block: 6.3e-7 with one number, 5.4e-8 so
// (with blocks of 64 rows 1.3e-7).
template <typename T>
struct TileSum {
    T hi = {}, lo = {};
    __device__ __forceinline__ void add(const T& x) {
        const T s = hi + x, v = s - hi;
        lo += (hi - (s - v)) + (x - v);
        hi = s;
    }
};

// Fused forward + backward over rows [block * chunk, (block + 1) * chunk) of
// the step in tiles of 48; the block's gradient stays in registers over its
// tiles and goes to gpart[block][NPARAM] once, with its loss.  One block per
// compute unit (its parameters and activations take 150 KB of LDS).  Matrix
// work per row: 3 x 2 x 128^2 flops (hidden layer forward, its weight gradient
// and the gradient of layer 1's activations), all on v_mfma_f32_16x16x4: 23 us
// for 33792 rows at its rate.  The two waves of a SIMD hide little else, so the
// rest is kept off that path: the small layers' gradients are sums in registers
// of values that pass by anyway, or 12 more matrix instructions (layer 1), and
// two waves compute the loss and fetch the next tile's rows beside the other
// waves' matrix work.  33792 rows: 56 us (68 with loops over the rows in LDS for
// the small layers); with the exact sums over the tiles, which go out in binary64,
// a training step of them takes 88 us, 85 before.
__global__ __launch_bounds__(THREADS) void k_train(const float* __restrict__ prm, RowSpec rs,
                                                   uint32_t chunk, double* __restrict__ gpart,
                                                   double* __restrict__ lpart) {
    __shared__ NetSmem<ROWS> s;
    __shared__ __attribute__((aligned(16))) float d2[ROWS * ST];  // dL/d(pre-activation 2)
    __shared__ float dout[ROWS][2];
    __shared__ double s_o0[ROWS], s_aC[ROWS];
    __shared__ TileRows rows[2];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, li = lane & 15, lh = lane >> 4;
    const Layer1 l1 = load_params(prm, s);
    const double invH = inverse_H(rs);
    const uint32_t n_rows = rs.n_sample + rs.n_grid;
    const uint32_t r0 = blockIdx.x * chunk;
    const uint32_t r1 = r0 + chunk < n_rows ? r0 + chunk : n_rows;
    const int u0 = (wave & 3) * 32, k0 = (wave >> 2) * 64;  // tile of the W2 gradient
    const int i2 = t % HID, part2 = t / HID;                // unit and rows part2 + 4 j of d2
    TileSum<f32x4> gW2[2][4];
    TileSum<f32x4> gX;             // [k = 16 wave + 4 lh + i][li]: W1, b1 in column 5
    TileSum<float> gA0, gA1, gB;   // W3 and b2 of unit i2 over its rows
    TileSum<float> gO0, gO1;       // b3 over row t / 8 of the tiles
    double loss = 0.0;             // wave 6: over row `lane` of the tiles
    if (t < ROWS) load_row(rs, invH, r0 + t, r1, t, rows[0]);
    __syncthreads();

    int b = 0;
    for (uint32_t base = r0; base < r1; base += ROWS, b ^= 1) {
        const TileRows& in = rows[b];
        float o[2];
        forward_tile(s, in.x, l1, o);
        if ((t & 7) == 0 && t < 8 * ROWS) {
            const int r = t >> 3;
            const bool sample = !(in.C[r] > 1.5);
            const float wg = (float)in.w[r], C = sample ? (float)in.C[r] : 0.0f;
            const float ta = tanhf(o[1]);
            const float alpha = 0.9f * ta;
            const float g1 = sample ? wg * C / (1.0f + alpha * C) * 0.9f * (1.0f - ta * ta) : 0.0f;
            dout[r][0] = wg;
            dout[r][1] = g1;
            gO0.add(wg);
            gO1.add(g1);
            s_o0[r] = (double)o[0];
            s_aC[r] = (double)alpha * (double)C;
        }
        __syncthreads();
        {
            const float w0 = s.W3[i2], w1 = s.W3[HID + i2];
            float a0 = 0.0f, a1 = 0.0f, ab = 0.0f;
#pragma unroll 4
            for (int j = 0; j < ROWS / 4; ++j) {
                const int r = part2 + 4 * j;
                const float hv = s.h2[r * ST + i2], e0 = dout[r][0], e1 = dout[r][1];
                const float d = (e0 * w0 + e1 * w1) * (1.0f - hv * hv);
                d2[r * ST + i2] = d;
                a0 = fmaf(e0, hv, a0);
                a1 = fmaf(e1, hv, a1);
                ab += d;
            }
            gA0.add(a0);
            gA1.add(a1);
            gB.add(ab);
        }
        __syncthreads();
        if (wave == 6 && lane < ROWS) {
            if (!(in.C[lane] > 1.5))
                loss += (double)dout[lane][0] * (s_o0[lane] + log(1.0 + s_aC[lane]));
        } else if (wave == 7 && lane < ROWS && base + ROWS < r1) {
            load_row(rs, invH, base + ROWS + lane, r1, lane, rows[b ^ 1]);
        }
        // hidden layer's weights: gradient [u][k] = sum_r d2[r][u] h1[r][k], the
        // wave's 32 x 64 of it
        f32x4 tW2[2][4] = {};
#pragma unroll 4
        for (int g = 0; g < ROWS / 4; ++g) {
            const int r = 4 * g + lh;
            float A[2], B[4];
#pragma unroll
            for (int e = 0; e < 2; ++e) A[e] = d2[r * ST + u0 + 16 * e + li];
#pragma unroll
            for (int e = 0; e < 4; ++e) B[e] = s.h1[r * ST + k0 + 16 * e + li];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int f = 0; f < 4; ++f) tW2[e][f] = mfma_16(A[e], B[f], tW2[e][f]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int f = 0; f < 4; ++f) gW2[e][f].add(tW2[e][f]);
        // dL/d(pre-activation 1): sum_u d2[r][u] W2[u][k], the wave's 16 k; its
        // results are the next product's operand as they lie (row k = l % 16,
        // contraction over the rows 16 m + 4 (l / 16) + i)
        {
            f32x4 acc[3] = {}, tX = {};
            const int k = 16 * wave + li;
#pragma unroll
            for (int g = 0; g < HID / 16; ++g) {
                f32x4 A[3];
#pragma unroll
                for (int m = 0; m < 3; ++m)
                    A[m] = *(const f32x4*)&d2[(16 * m + li) * ST + 16 * g + 4 * lh];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float B = s.W2[(16 * g + 4 * lh + q) * ST + k];
#pragma unroll
                    for (int m = 0; m < 3; ++m) acc[m] = mfma_16(A[m][q], B, acc[m]);
                }
            }
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 16 * m + 4 * lh + i;
                    const float hv = s.h1[r * ST + k];
                    tX = mfma_16(acc[m][i] * (1.0f - hv * hv), in.x[r][li & 7], tX);
                }
            gX.add(tX);
        }
        __syncthreads();
    }
    double* gp = gpart + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                gp[OFF_W2 + (u0 + 16 * e + 4 * lh + i) * HID + k0 + 16 * f + li] =
                    (double)gW2[e][f].hi[i] + gW2[e][f].lo[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 16 * wave + 4 * lh + i;
        const double v = (double)gX.hi[i] + gX.lo[i];
        if (li < 5) gp[OFF_W1 + k * 5 + li] = v;
        if (li == 5) gp[OFF_B1 + k] = v;
    }
    // the four parts of the units' sums, the rows' sums of b3
    double* red = (double*)d2;
    red[t] = (double)gA0.hi + gA0.lo;
    red[THREADS + t] = (double)gA1.hi + gA1.lo;
    red[2 * THREADS + t] = (double)gB.hi + gB.lo;
    if ((t & 7) == 0 && t < 8 * ROWS) {
        s_o0[t >> 3] = (double)gO0.hi + gO0.lo;
        s_aC[t >> 3] = (double)gO1.hi + gO1.lo;
    }
    __syncthreads();
    if (t < 3 * HID) {
        const double* v = red + (t / HID) * THREADS + i2;
        const double a = (v[0] + v[HID]) + (v[2 * HID] + v[3 * HID]);
        gp[t < 2 * HID ? OFF_W3 + t : OFF_B2 + i2] = a;
    } else if (wave == 6) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
        if (lane == 0) lpart[blockIdx.x] = loss;
    } else if (lane < 2) {
        const double* v = lane ? s_aC : s_o0;
        double a = 0.0;
        for (int r = 0; r < ROWS; ++r) a += v[r];
        gp[OFF_B3 + lane] = a;
    }
}

// grad[p] = sum over blocks (fixed order, binary64); loss = sum of lpart plus
// sum_c (H_c / H) log Z_c; with ADAM (Kingma & Ba, 2015, bias correction, step
// t >= 1) the update of parameter p follows at once.  256 threads share 32
// parameters: 8 groups of blocks each, 8 loads in flight per thread (one thread
// per parameter over all blocks waited on every load: 149 us for 528 blocks).
struct AdamArgs {
    float* m1;
    float* m2;
    float lr, b1, b2, eps, c1, c2;
};
constexpr int GR_P = 32;

template <bool ADAM>
__global__ __launch_bounds__(256) void k_grad_reduce(const double* __restrict__ gpart, int n_blocks,
                                                     const double* __restrict__ lpart, RowSpec rs,
                                                     float* __restrict__ grad,
                                                     double* __restrict__ loss,
                                                     float* __restrict__ prm, AdamArgs ad) {
    __shared__ double red[8][GR_P];
    const int t = threadIdx.x, pl = t % GR_P, g = t / GR_P;
    const int p = blockIdx.x * GR_P + pl;
    double a = 0.0;
    if (p < NPARAM) {
        int b = g;
        for (; b + 7 * 8 < n_blocks; b += 64) {
            double v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = gpart[(int64_t)(b + 8 * e) * NPARAM + p];
#pragma unroll
            for (int e = 0; e < 8; ++e) a += v[e];
        }
        for (; b < n_blocks; b += 8) a += gpart[(int64_t)b * NPARAM + p];
    }
    red[g][pl] = a;
    __syncthreads();
    if (g == 0 && p < NPARAM) {
        for (int e = 1; e < 8; ++e) a += red[e][pl];
        const float gr = (float)a;
        grad[p] = gr;
        if constexpr (ADAM) {
            const float m = ad.b1 * ad.m1[p] + (1.0f - ad.b1) * gr;
            const float v = ad.b2 * ad.m2[p] + (1.0f - ad.b2) * gr * gr;
            ad.m1[p] = m;
            ad.m2[p] = v;
            prm[p] -= ad.lr * (m / ad.c1) / (sqrtf(v / ad.c2) + ad.eps);
        }
    }
    if (loss && blockIdx.x == 0) {
        // one wave: the blocks' shares and the contexts' constants, strided by
        // lane, then a fixed tree
        if (t < 64) {
            const double invH = inverse_H(rs);
            double L = 0.0;
            for (int b = t; b < n_blocks; b += 64) L += lpart[b];
            for (uint32_t c = t; c < rs.n_ctx; c += 64) L += rs.Hc[c] * invH * rs.logZ[c];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) L += __shfl_xor(L, off);
            if (t == 0) *loss = L;
        }
    }
}

// Training rows: context c, row r uses R2 point index + 1 + c m + r;
// h = f^2 W F^2 2 (1 - cos(2 pi f |B| cos(theta - theta_B))).
__global__ void k_rows(uint64_t s0x, uint64_t s0y, uint64_t index, int64_t n_ctx, int64_t m,
                       const double* __restrict__ ctx4, double c_psd, double r0_m53,
                       double fmin, double Lw, double* __restrict__ ell,
                       double* __restrict__ theta, double* __restrict__ h) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_ctx * m) return;
    const double* c = ctx4 + 4 * (i / m);
    double ux, uy;
    r2_point(s0x, s0y, index + 1u + (uint64_t)i, ux, uy);
    const double l = log(fmin) + Lw * ux;
    const double th = 2.0 * 3.141592653589793 * uy;
    const double f = exp(l);
    const double W = psd_phase(1, c_psd, r0_m53, 1.0 / (c[1] * c[1]), f);
    const double F = aperture_filter(c[0], 0.0, f);
    const double proj = f * c[2] * cos(th - c[3]);
    ell[i] = l;
    theta[i] = th;
    h[i] = f * f * W * F * F * 2.0 * (1.0 - cospi(2.0 * proj));
}

// Sampling table from the network outputs o[b][j][2] on the cell midpoints
// (one block): per baseline p_b = exp(o0)/Z_b, alpha_b = 0.9 tanh(o1);
// mixture over baselines, defensive share beta of the plain density, CDF.
__global__ __launch_bounds__(256) void k_table(const float* __restrict__ o, int64_t nB,
                                               int n_cells, const double* __restrict__ bth,
                                               double Lw, double beta, double* __restrict__ p,
                                               double* __restrict__ alpha,
                                               double* __restrict__ phi,
                                               double* __restrict__ cdf,
                                               double* __restrict__ scratch) {
    // scratch: [nB] max, [nB] Z
    double* mx = scratch;
    double* Z = scratch + nB;
    const double dl = Lw / n_cells;
    for (int64_t b = threadIdx.x; b < nB; b += blockDim.x) {
        double m = -1e300;
        for (int j = 0; j < n_cells; ++j) m = fmax(m, (double)o[(b * n_cells + j) * 2]);
        double z = 0.0;
        for (int j = 0; j < n_cells; ++j) z += exp((double)o[(b * n_cells + j) * 2] - m) * dl;
        mx[b] = m;
        Z[b] = z;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n_cells; j += blockDim.x) {
        double pb = 0.0, A = 0.0, B = 0.0;
        for (int64_t b = 0; b < nB; ++b) {
            const double pj = exp((double)o[(b * n_cells + j) * 2] - mx[b]) / Z[b];
            const double al = 0.9 * tanh((double)o[(b * n_cells + j) * 2 + 1]);
            pb += pj / (double)nB;
            A += pj * al * cos(2.0 * bth[b]) / (double)nB;
            B += pj * al * sin(2.0 * bth[b]) / (double)nB;
        }
        const double pp = (1.0 - beta) * pb + beta / Lw;
        p[j] = pp;
        alpha[j] = (1.0 - beta) * sqrt(A * A + B * B) / pp;
        phi[j] = 0.5 * atan2(B, A);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int j = 0; j < n_cells; ++j) tot += p[j] * dl;
        double run = 0.0;
        for (int j = 0; j < n_cells; ++j) {
            p[j] /= tot;
            cdf[j] = run;
            run += p[j] * dl;
        }
    }
}

// Learned sampler: point n = index + 1 + i; cell j = max{c : cdf[c] <= u1};
// ell = lmin + j dl + (u1 - cdf[j]) / p[j]; t + (alpha/2) sin 2t = 2 pi u2 by
// 12 Newton steps from 2 pi u2; theta = t + phi[j]; area = f^2 / (K q).
__global__ __launch_bounds__(256) void k_sample_learned(
    uint64_t s0x, uint64_t s0y, uint64_t index, int64_t n, int64_t K, double lmin, double Lw,
    int n_cells, const double* __restrict__ tp, const double* __restrict__ ta,
    const double* __restrict__ tphi, const double* __restrict__ tcdf, double* __restrict__ fx,
    double* __restrict__ fy, double* __restrict__ area) {
    __shared__ double sp[MAX_CELLS], sa[MAX_CELLS], sphi[MAX_CELLS], scdf[MAX_CELLS];
    for (int j = threadIdx.x; j < n_cells; j += blockDim.x) {
        sp[j] = tp[j];
        sa[j] = ta[j];
        sphi[j] = tphi[j];
        scdf[j] = tcdf[j];
    }
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double ux, uy;
    r2_point(s0x, s0y, index + 1u + (uint64_t)i, ux, uy);
    int lo = 0, hi = n_cells - 1;  // largest j with cdf[j] <= ux (cdf[0] = 0)
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (scdf[mid] <= ux) lo = mid;
        else hi = mid - 1;
    }
    const int j = lo;
    const double dl = Lw / n_cells;
    const double ell = lmin + j * dl + (ux - scdf[j]) / sp[j];
    const double target = 2.0 * 3.141592653589793 * uy;
    double t = target;
    const double al = sa[j];
    for (int it = 0; it < 12; ++it) t -= (t + 0.5 * al * sin(2.0 * t) - target) / (1.0 + al * cos(2.0 * t));
    const double th = t + sphi[j];
    const double f = exp(ell);
    const double q = sp[j] * (1.0 + al * cos(2.0 * t)) / (2.0 * 3.141592653589793);
    double s, c;
    sincos(th, &s, &c);
    fx[i] = f * c;
    fy[i] = f * s;
    area[i] = f * f / ((double)K * q);
}

}  // namespace prop

// ----------------------------------------------------------- launchers ----
static inline int64_t cdivp(int64_t a, int64_t b) { return (a + b - 1) / b; }

// compute units of the current device (blocks of the persistent kernels)
static int prop_units() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
        n = 256;
    return n;
}

hipError_t prop_launch_forward(const float* prm, int64_t n, const double* ell, const double* ctx4,
                               double lmin, double Lw, float* out, hipStream_t st) {
    const int64_t tiles = cdivp(n, prop::ROWS_F);
    const int units = prop_units();
    hipLaunchKernelGGL(prop::k_forward, dim3((unsigned)(tiles < units ? tiles : units)),
                       dim3(prop::THREADS), 0, st, prm, n, ell, ctx4, lmin, Lw, out);
    return hipGetLastError();
}

hipError_t prop_launch_rows(uint64_t s0x, uint64_t s0y, uint64_t index, int64_t n_ctx, int64_t m,
                            const double* ctx4, double c_psd, double r0, double fmin, double fmax,
                            double* ell, double* theta, double* h, hipStream_t st) {
    const int64_t n = n_ctx * m;
    hipLaunchKernelGGL(prop::k_rows, dim3((unsigned)cdivp(n, 256)), dim3(256), 0, st, s0x, s0y,
                       index, n_ctx, m, ctx4, c_psd, pow(r0, -5.0 / 3.0), fmin, log(fmax / fmin),
                       ell, theta, h);
    return hipGetLastError();
}

// Rows per block of a step's n rows: one block per compute unit, whole
// 16-row matrix tiles.
static int64_t step_chunk(int64_t n, int units) {
    const int64_t chunk = cdivp(n, units);
    return chunk <= prop::ROWS ? prop::ROWS : cdivp(chunk, 16) * 16;
}

StepSizes prop_step_sizes(int64_t n_ctx, int64_t m, int64_t G) {
    StepSizes z;
    const int64_t n = n_ctx * (m + G);
    z.chunk = step_chunk(n, prop_units());
    z.blocks = cdivp(n, z.chunk);
    z.doubles = (size_t)(2 * n_ctx + n_ctx * G + z.blocks);
    z.floats = (size_t)(4 * n_ctx + n_ctx * G);
    return z;
}

hipError_t prop_launch_step(float* prm, const StepSizes& z, int64_t n_ctx, int64_t m,
                            const int32_t* ctxlist, const double* ctx4, const double* ell,
                            const double* theta, const double* h, int G, double lmin, double Lw,
                            double* dscratch, float* fscratch, double* gpart, float* grad,
                            double* loss, float* m1, float* m2, float lr, int64_t t,
                            hipStream_t st) {
    prop::RowSpec rs;
    rs.n_sample = (uint32_t)(n_ctx * m);
    rs.n_grid = (uint32_t)(n_ctx * G);
    rs.m = (uint32_t)m;
    rs.G = (uint32_t)G;
    rs.n_ctx = (uint32_t)n_ctx;
    rs.ctxlist = ctxlist;
    rs.ctx4 = ctx4;
    rs.ell = ell;
    rs.theta = theta;
    rs.h = h;
    rs.Hc = dscratch;
    rs.logZ = dscratch + n_ctx;
    rs.soft = dscratch + 2 * n_ctx;
    double* lpart = rs.soft + n_ctx * G;
    rs.feat = fscratch;
    float* og = fscratch + 4 * n_ctx;
    rs.lmin = lmin;
    rs.Lw = Lw;
    hipLaunchKernelGGL(prop::k_grid, dim3((unsigned)(2 * n_ctx)), dim3(prop::THREADS), 0, st, prm,
                       rs, og);
    hipLaunchKernelGGL(prop::k_train, dim3((unsigned)z.blocks), dim3(prop::THREADS), 0, st, prm, rs,
                       (uint32_t)z.chunk, gpart, lpart);
    prop::AdamArgs ad{};
    const dim3 g((unsigned)cdivp(NPARAM, prop::GR_P));
    if (m1) {
        ad.m1 = m1;
        ad.m2 = m2;
        ad.lr = lr;
        ad.b1 = 0.9f;
        ad.b2 = 0.999f;
        ad.eps = 1e-8f;
        ad.c1 = 1.0f - powf(ad.b1, (float)t);
        ad.c2 = 1.0f - powf(ad.b2, (float)t);
        hipLaunchKernelGGL(prop::k_grad_reduce<true>, g, dim3(256), 0, st, gpart, (int)z.blocks,
                           lpart, rs, grad, loss, prm, ad);
    } else {
        hipLaunchKernelGGL(prop::k_grad_reduce<false>, g, dim3(256), 0, st, gpart, (int)z.blocks,
                           lpart, rs, grad, loss, prm, ad);
    }
    return hipGetLastError();
}

hipError_t prop_launch_table(const float* o, int64_t nB, int n_cells, const double* bth,
                             double Lw, double beta, double* p, double* alpha, double* phi,
                             double* cdf, double* scratch, hipStream_t st) {
    hipLaunchKernelGGL(prop::k_table, dim3(1), dim3(256), 0, st, o, nB, n_cells, bth, Lw, beta, p,
                       alpha, phi, cdf, scratch);
    return hipGetLastError();
}

hipError_t prop_launch_sample(uint64_t s0x, uint64_t s0y, uint64_t index, int64_t n, int64_t K,
                              double lmin, double Lw, int n_cells, const double* p,
                              const double* alpha, const double* phi, const double* cdf,
                              double* fx, double* fy, double* area, hipStream_t st) {
    hipLaunchKernelGGL(prop::k_sample_learned, dim3((unsigned)cdivp(n, 256)), dim3(256), 0, st,
                       s0x, s0y, index, n, K, lmin, Lw, n_cells, p, alpha, phi, cdf, fx, fy, area);
    return hipGetLastError();
}

}  // namespace qrfs
