// qrfs_separable.hip -- Eq. 3 on point sets with product structure, in
// binary64 on the FP64 matrix instructions of gfx950.
//
// Points x_uv = p_u + q_v (a time series under frozen flow; a regular grid)
// factor the phase of a frequency: f.x_uv = phi_u + psi_v, so
//   a cos 2 pi(phi + psi) + b sin 2 pi(phi + psi)
//     = cos 2 pi psi (a cos 2 pi phi + b sin 2 pi phi)
//     + sin 2 pi psi (b cos 2 pi phi - a sin 2 pi phi),
// and the sum over frequencies is, per realisation, a matrix product
// [U x 2K] [2K x V] with U + V instead of U V sines and cosines per
// frequency.  The general kernels evaluate one sine and cosine (37 vector
// instructions in binary64) per term; here a term is 4 flops of the product.
#include "qrfs_mfma.hpp"

namespace qrfs {

// Block: one realisation, an output tile of 16 MU rows x 16 NV columns, WV
// waves that split the frequencies (each wave a range of whole groups of 8)
// and are summed in a fixed tree through LDS.
//
// A wave takes 128 frequencies at a time: lane l draws the Philox block of
// frequencies 2l and 2l + 1 and stages (f, a w, b w) in LDS; then, 4
// frequencies per step, lane (i = l % 16, h = l / 16) takes frequency h of
// the step, evaluates e^(i phi) for its MU rows and e^(i psi) for its NV
// columns, forms the two row factors and feeds 2 MU NV matrix instructions:
// both operands are born in the lane that the instruction reads them from,
// nothing goes through LDS but the staged frequencies.
//
// Bound: the FP64 datapath, which the matrix instructions share with the
// vector ALU (measured: the times add).  Per step a 2 x 2 wave spends 8
// matrix instructions (64 cycles each) and 4 sine / cosine pairs (~35
// instructions of 4 cycles).  2000 realisations x 1936 frequencies x 1024
// differential samples: 0.60 ms (the matrix instructions alone 0.43 ms at
// 73.7 TFLOP/s), against 9.4 ms for both telescopes in the general kernel.
//
// DIFF: the sums at x minus the sums at x + delta (the differential piston
// of two telescopes): the coefficients are first turned by delta,
//   a' = a (1 - cos 2 pi f.delta) - b sin 2 pi f.delta,
//   b' = b (1 - cos 2 pi f.delta) + a sin 2 pi f.delta,
// with 1 - cos = 2 sin^2, so the contraction runs once instead of twice and
// nothing cancels afterwards.
constexpr int SEP_KC = 128;  // frequencies a wave stages at a time

template <int MU, int NV, int WV>
struct SepSmem {
    static constexpr int TILE = 256 * MU * NV;
    static constexpr int STAGE = WV * SEP_KC * 4;
    static constexpr int TREE = (WV / 2) * TILE;
    // the staged frequencies, then (after the loop) the partial tiles
    __attribute__((aligned(16))) double d[STAGE > TREE ? STAGE : TREE];
};

template <bool DIFF, int MU, int NV, int WV>
__global__ __launch_bounds__(64 * WV) void k_separable(SepArgs a, int ut, int vt) {
    __shared__ SepSmem<MU, NV, WV> sm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lh = lane >> 4;
    const int64_t tiles = (int64_t)ut * vt;
    const int64_t r = a.r0 + (int64_t)blockIdx.x / tiles;
    const int tile = (int)((int64_t)blockIdx.x % tiles);
    const int u0 = (tile / vt) * 16 * MU, v0 = (tile % vt) * 16 * NV;
    const int64_t s = r / a.R_block;
    const double* fx = a.fx + s * a.K;
    const double* fy = a.fy + s * a.K;
    const double* w = a.w + s * a.K;

    // the lane's rows and columns
    double rx[MU], ry[MU], cx[NV], cy[NV];
#pragma unroll
    for (int m = 0; m < MU; ++m) {
        const double t = (double)((u0 + 16 * m + li) * a.V);
        rx[m] = a.ox + t * a.sx;
        ry[m] = a.oy + t * a.sy;
    }
#pragma unroll
    for (int n = 0; n < NV; ++n) {
        const double t = (double)(v0 + 16 * n + li);
        cx[n] = t * a.sx;
        cy[n] = t * a.sy;
    }
    f64x4 acc[MU][NV];
#pragma unroll
    for (int m = 0; m < MU; ++m)
#pragma unroll
        for (int n = 0; n < NV; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};

    const int64_t kw = ((a.K + 8 * WV - 1) / (8 * WV)) * 8;
    const int64_t kb = wave * kw;
    const int64_t ke = kb + kw < a.K ? kb + kw : a.K;
    double* st = sm.d + wave * SEP_KC * 4;
    for (int64_t k0 = kb; k0 < ke; k0 += SEP_KC) {
        {
            const int64_t k = k0 + 2 * lane;
            double g[4] = {0.0, 0.0, 0.0, 0.0};
            if (k < ke) coef4_f64(a.seed, a.counter + (uint64_t)r, (uint32_t)(k >> 1), a.mode, g);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool ok = k + h < ke;
                const double f0 = ok ? fx[k + h] : 0.0, f1 = ok ? fy[k + h] : 0.0;
                const double wk = ok ? w[k + h] : 0.0;
                double ca = wk * g[2 * h], cb = wk * g[2 * h + 1];
                if constexpr (DIFF) {
                    double sh, ch;
                    sincos2pi_reduced(0.5 * frac_centered(f0 * a.dx + f1 * a.dy), sh, ch);
                    const double oc = 2.0 * sh * sh, sd = 2.0 * sh * ch;
                    const double ta = fma(ca, oc, -(cb * sd));
                    cb = fma(cb, oc, ca * sd);
                    ca = ta;
                }
                double2* dst = (double2*)(st + (2 * lane + h) * 4);
                dst[0] = make_double2(f0, f1);
                dst[1] = make_double2(ca, cb);
            }
        }
        // the wave's own stage: written and read by the same wave
        __builtin_amdgcn_wave_barrier();
        __threadfence_block();
        const int64_t left = ke - k0;
        const int steps = left >= SEP_KC ? SEP_KC / 4 : (int)((left + 3) / 4);
        for (int g = 0; g < steps; ++g) {
            const double2* src = (const double2*)(st + (4 * g + lh) * 4);
            const double2 f = src[0], c = src[1];
            double A[MU], B[MU];
#pragma unroll
            for (int m = 0; m < MU; ++m) {
                double sn, cs;
                sincos2pi_reduced(frac_centered(fma(f.x, rx[m], f.y * ry[m])), sn, cs);
                A[m] = fma(c.x, cs, c.y * sn);
                B[m] = fma(c.y, cs, -(c.x * sn));
            }
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                double sn, cs;
                sincos2pi_reduced(frac_centered(fma(f.x, cx[n], f.y * cy[n])), sn, cs);
#pragma unroll
                for (int m = 0; m < MU; ++m) acc[m][n] = mfma_f64(A[m], cs, acc[m][n]);
#pragma unroll
                for (int m = 0; m < MU; ++m) acc[m][n] = mfma_f64(B[m], sn, acc[m][n]);
            }
        }
        __threadfence_block();
        __builtin_amdgcn_wave_barrier();
    }

    // fixed tree over the waves: the upper half stores, the lower half adds
#pragma unroll
    for (int half = WV / 2; half > 0; half >>= 1) {
        __syncthreads();
        if (wave >= half && wave < 2 * half) {
            double* dst = sm.d + (wave - half) * (256 * MU * NV) + lane;
#pragma unroll
            for (int m = 0; m < MU; ++m)
#pragma unroll
                for (int n = 0; n < NV; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[((m * NV + n) * 4 + i) * 64] = acc[m][n][i];
        }
        __syncthreads();
        if (wave < half) {
            const double* src = sm.d + wave * (256 * MU * NV) + lane;
#pragma unroll
            for (int m = 0; m < MU; ++m)
#pragma unroll
                for (int n = 0; n < NV; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][n][i] += src[((m * NV + n) * 4 + i) * 64];
        }
    }
    if (wave == 0) {
        double* out = a.out + r * a.P;
#pragma unroll
        for (int m = 0; m < MU; ++m)
#pragma unroll
            for (int n = 0; n < NV; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int v = v0 + 16 * n + li;
                    const int64_t p = (int64_t)(u0 + 16 * m + lh + 4 * i) * a.V + v;
                    if (v < a.V && p < a.P) out[p] = acc[m][n][i];
                }
    }
}

// Differential pistons of a time series: tiles of 32 x 32 samples (a row is
// 32 consecutive samples).  4 waves per block when the realisations alone
// give every SIMD two waves, else 16 waves that split the frequencies.
hipError_t launch_series_diff(const SepArgs& args, hipStream_t st) {
    SepArgs a = args;
    const int ut = (int)((a.P + 32 * a.V - 1) / (32 * a.V)), vt = a.V / 32;
    const int64_t tiles = (int64_t)ut * vt;
    const int64_t step = kMaxLaunchBlocks / tiles;  // realisations per launch
    for (a.r0 = 0; a.r0 < a.R; a.r0 += step) {
        const int64_t n = (a.R - a.r0 < step ? a.R - a.r0 : step) * tiles;
        if (n >= 512)
            hipLaunchKernelGGL((k_separable<true, 2, 2, 4>), dim3((unsigned)n), dim3(256), 0, st,
                               a, ut, vt);
        else
            hipLaunchKernelGGL((k_separable<true, 2, 2, 16>), dim3((unsigned)n), dim3(1024), 0, st,
                               a, ut, vt);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qrfs
