// qrfs_temporal.hip -- frozen-flow temporal structure function of the
// differential piston (the statistical test of Sec. 4.4): aperture centres
// moved by the wind, and the time-lag estimator over piston time series.
#include "qrfs_device.hpp"
#include "qrfs_internal.hpp"

namespace qrfs {

// Points 0 .. M-1: c1 - v t_m, points M .. 2M-1: c2 - v t_m, t_m = m dt
// (Taylor: at time t the telescope at c sees the screen at c - v t).
__global__ void k_taylor_points(double c1x, double c1y, double c2x, double c2y, double vx,
                                double vy, double dt, int64_t M, double* __restrict__ px,
                                double* __restrict__ py) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * M) return;
    const bool second = i >= M;
    const double t = (double)(second ? i - M : i) * dt;
    px[i] = (second ? c2x : c1x) - vx * t;
    py[i] = (second ? c2y : c1y) - vy * t;
}

constexpr int TS_THREADS = 256;
constexpr int TS_MAX_SHARES = 4096;
constexpr int TS_B = 8;     // lags, and positions, of a register tile
constexpr int TS_STR = 10;  // doubles per 8 positions in LDS: 16-byte reads, and 64 lanes at
                            // consecutive blocks fall on different banks

// Block b: realisations [b RB, (b+1) RB).  For each, the differential piston
// dp[m] (DIFF: given; else p1[m] - p2[m]) goes to LDS and
// sum_m (dp[m + j] - dp[m])^2 is formed for every lag j, two vector
// instructions per pair (m, j) in binary64: the bound.  A thread works on
// tiles of 8 positions x 8 lags in registers, walking the positions of a
// group of 8 lags with the upper window carried from tile to tile, so a tile
// (64 pairs, 128 instructions) costs 8 16-byte LDS reads; with one lag per
// thread and two 8-byte reads per pair the loop was bound by LDS.  Groups g
// and G-1-g are walked one after the other, so that every lane has G - 1
// tiles although long lags have few positions, and `tpp` threads share a
// pair of groups to fill the block.  The last two tiles of a group, where
// m + j passes the end of the series, are masked and done apart.
// Thread j % 256 then owns lag j: it adds the tpp shares in order, and the
// realisation's mean over pairs and its square to registers.  Writes
// part[b][j][0..1]; the fixed-order reduction over blocks gives the mean
// over realisations and its standard error.
// 2000 realisations x 1024 samples: 115 us (55 us at the full issue rate;
// 963 us with one lag per thread).
template <typename T, bool DIFF, int MAXM>
__global__ __launch_bounds__(TS_THREADS) void k_temporal_rows(const T* __restrict__ pist,
                                                              int64_t R, int M, int RB, int tpp,
                                                              double* __restrict__ part) {
    constexpr int MAXJ = MAXM / TS_THREADS;
    // MAXM / 8 blocks of positions and one of zeros; shares of the tpp threads
    __shared__ __attribute__((aligned(16))) double dp[(MAXM / TS_B + 1) * TS_STR];
    __shared__ double share[TS_MAX_SHARES];
    const int tid = threadIdx.x;
    const int G = (M + TS_B - 1) / TS_B;  // groups of lags = blocks of positions
    const int NP = (G + 1) / 2;           // pairs of groups
    const int q = tid / NP, ga = tid % NP, gb = G - 1 - ga;
    const bool active = q < tpp;
    // unmasked tiles of group g: position blocks [0, G - 2 - g)
    const int na = G - 2 - ga > 0 ? G - 2 - ga : 0;
    const int nb = gb > ga && G - 2 - gb > 0 ? G - 2 - gb : 0;
    const int t0 = active ? q * (na + nb) / tpp : 0;
    const int t1 = active ? (q + 1) * (na + nb) / tpp : 0;

    double s1[MAXJ], s2[MAXJ];
#pragma unroll
    for (int i = 0; i < MAXJ; ++i) s1[i] = s2[i] = 0.0;
    const int64_t r0 = (int64_t)blockIdx.x * RB;
    const int64_t r1 = r0 + RB < R ? r0 + RB : R;

    auto load = [&](int blk, double (&v)[TS_B]) {
        const double2* src = (const double2*)&dp[blk * TS_STR];
#pragma unroll
        for (int i = 0; i < TS_B / 2; ++i) {
            const double2 t = src[i];
            v[2 * i] = t.x;
            v[2 * i + 1] = t.y;
        }
    };

    for (int64_t r = r0; r < r1; ++r) {
        const T* p1 = pist + r * (DIFF ? 1 : 2) * M;
        for (int m = tid; m < (G + 1) * TS_B; m += TS_THREADS) {
            double v = 0.0;
            if (m < M) v = DIFF ? (double)p1[m] : (double)p1[m] - (double)p1[M + m];
            dp[(m / TS_B) * TS_STR + m % TS_B] = v;
        }
        __syncthreads();
        double acc[TS_B], keep[TS_B], lo[TS_B], hi[TS_B], x[TS_B];
#pragma unroll
        for (int l = 0; l < TS_B; ++l) acc[l] = keep[l] = 0.0;
        if (active) {
            // tiles [t0, t1) of the na tiles of group ga and the nb of gb
            int g = t0 < na ? ga : gb;
            int b = t0 < na ? t0 : t0 - na;
            load(b + g, lo);
            for (int t = t0; t < t1; ++t) {
                if (t == na && t > t0) {  // on to the second group
#pragma unroll
                    for (int l = 0; l < TS_B; ++l) {
                        keep[l] = acc[l];
                        acc[l] = 0.0;
                    }
                    g = gb;
                    b = 0;
                    load(g, lo);
                }
                load(b, x);
                load(b + g + 1, hi);
#pragma unroll
                for (int i = 0; i < TS_B; ++i)
#pragma unroll
                    for (int l = 0; l < TS_B; ++l) {
                        const int e = i + l;
                        const double d = (e < TS_B ? lo[e % TS_B] : hi[e % TS_B]) - x[i];
                        acc[l] = fma(d, d, acc[l]);
                    }
#pragma unroll
                for (int l = 0; l < TS_B; ++l) lo[l] = hi[l];
                ++b;
            }
            // `acc` belongs to ga if the walk ended there, `keep` to ga if it went on
            if (t1 <= na) {
#pragma unroll
                for (int l = 0; l < TS_B; ++l) {
                    keep[l] = acc[l];
                    acc[l] = 0.0;
                }
            }
            // masked tiles (position blocks G - 2 - g and G - 1 - g) of both groups
            for (int k = q; k < 4; k += tpp) {
                const int gg = k < 2 ? ga : gb;
                const int bb = G - 2 - gg + (k & 1);
                if (bb < 0 || (k >= 2 && gb <= ga)) continue;
                load(bb, x);
                load(bb + gg, lo);
                load(bb + gg + 1 <= G ? bb + gg + 1 : G, hi);
                const int lim = M - TS_B * (bb + gg);  // window positions inside the series
                double ta[TS_B];
#pragma unroll
                for (int l = 0; l < TS_B; ++l) ta[l] = 0.0;
#pragma unroll
                for (int i = 0; i < TS_B; ++i)
#pragma unroll
                    for (int l = 0; l < TS_B; ++l) {
                        const int e = i + l;
                        double d = (e < TS_B ? lo[e % TS_B] : hi[e % TS_B]) - x[i];
                        d = e < lim ? d : 0.0;
                        ta[l] = fma(d, d, ta[l]);
                    }
#pragma unroll
                for (int l = 0; l < TS_B; ++l) {
                    if (k < 2) keep[l] += ta[l];
                    else acc[l] += ta[l];
                }
            }
#pragma unroll
            for (int l = 0; l < TS_B; ++l) share[q * (G * TS_B) + ga * TS_B + l] = keep[l];
            if (gb > ga)
#pragma unroll
                for (int l = 0; l < TS_B; ++l) share[q * (G * TS_B) + gb * TS_B + l] = acc[l];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MAXJ; ++i) {
            const int j = tid + TS_THREADS * i;
            if (j >= 1 && j < M) {
                double a = 0.0;
                for (int k = 0; k < tpp; ++k) a += share[k * (G * TS_B) + j];
                const double v = a / (double)(M - j);
                s1[i] += v;
                s2[i] += v * v;
            }
        }
        // the next realisation's dp is written before the next barrier and
        // read after it; its shares are written after that barrier
    }
#pragma unroll
    for (int i = 0; i < MAXJ; ++i) {
        const int j = tid + TS_THREADS * i;
        if (j < M) {
            part[((int64_t)blockIdx.x * M + j) * 2] = s1[i];
            part[((int64_t)blockIdx.x * M + j) * 2 + 1] = s2[i];
        }
    }
}

static inline int64_t tcdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

hipError_t launch_taylor_points(const double c1[2], const double c2[2], const double v[2],
                                double dt, int64_t M, double* px, double* py, hipStream_t st) {
    hipLaunchKernelGGL(k_taylor_points, dim3((unsigned)tcdiv(2 * M, 256)), dim3(256), 0, st,
                       c1[0], c1[1], c2[0], c2[1], v[0], v[1], dt, M, px, py);
    return hipGetLastError();
}

template <typename T, bool DIFF>
static hipError_t launch_rows_t(const T* pist, int64_t R, int M, int rows, double* part,
                                hipStream_t st) {
    const dim3 g((unsigned)tcdiv(R, rows));
    const int groups = (M + TS_B - 1) / TS_B, np = (groups + 1) / 2;
    // threads per pair of lag groups: the block's 256 threads over the np
    // pairs (np <= 256), at most 16, and as many rows of sums as LDS holds
    int tpp = TS_THREADS / np < 16 ? TS_THREADS / np : 16;
    while (tpp > 1 && tpp * groups * TS_B > TS_MAX_SHARES) --tpp;
    if (M <= 1024)
        hipLaunchKernelGGL((k_temporal_rows<T, DIFF, 1024>), g, dim3(TS_THREADS), 0, st, pist, R, M,
                           rows, tpp, part);
    else
        hipLaunchKernelGGL((k_temporal_rows<T, DIFF, TEMPORAL_MAX_M>), g, dim3(TS_THREADS), 0, st,
                           pist, R, M, rows, tpp, part);
    return hipGetLastError();
}

hipError_t launch_temporal_rows(bool fp64, bool diff, const void* pist, int64_t R, int64_t M,
                                int rows, double* part, hipStream_t st) {
    if (fp64 && diff)
        return launch_rows_t<double, true>((const double*)pist, R, (int)M, rows, part, st);
    if (fp64) return launch_rows_t<double, false>((const double*)pist, R, (int)M, rows, part, st);
    return launch_rows_t<float, false>((const float*)pist, R, (int)M, rows, part, st);
}

}  // namespace qrfs
