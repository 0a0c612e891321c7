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
// instructions of 4 cycles), in a series 2 pairs and 2 rotations by turns that
// are staged with the frequency.  2000 realisations x 1936 frequencies x 1024
// differential samples: 0.46 ms (the matrix instructions alone 0.22 ms at
// 73.7 TFLOP/s; 0.50 with 3 waves per SIMD, 0.60 with 4 pairs), against 9.4 ms for both telescopes in the
// general kernel.
//
// DIFF: the sums at x minus the sums at x + delta (the differential piston
// of two telescopes): the coefficients are first turned by delta,
//   a' = a (1 - cos 2 pi f.delta) - b sin 2 pi f.delta,
//   b' = b (1 - cos 2 pi f.delta) + a sin 2 pi f.delta,
// with 1 - cos = 2 sin^2, so the contraction runs once instead of twice and
// nothing cancels afterwards.
constexpr int SEP_KC = 128;  // frequencies a wave stages at a time

constexpr int sep_stage(bool diff) { return diff ? 8 : 4; }  // doubles per staged frequency

template <bool DIFF, int MU, int NV, int WV>
struct SepSmem {
    static constexpr int TILE = 256 * MU * NV;
    static constexpr int STAGE = WV * SEP_KC * sep_stage(DIFF);
    static constexpr int TREE = (WV / 2) * TILE;
    // the staged frequencies, then (after the loop) the partial tiles
    __attribute__((aligned(16))) double d[STAGE > TREE ? STAGE : TREE];
};

// (sn, cs) turned by the angle of (sin, cos) = (t.x, t.y).
__device__ __forceinline__ void turn(const double2& t, double& sn, double& cs) {
    const double s = fma(sn, t.y, cs * t.x);
    cs = fma(cs, t.y, -(sn * t.x));
    sn = s;
}

// One output tile of realisation r (all threads of the block call it): the
// lane's rows (rx, ry) and columns (cx, cy), frequencies fx, fy, w of the set.
// emit(m, n, i, sum) receives element (16 m + lane / 16 + 4 i, 16 n + lane % 16).
// Returns whether the lane met a weighted coefficient that is not finite: the
// product of the two factors is then NaN where the sum of Eq. 3 is infinite.
template <bool DIFF, int MU, int NV, int WV, typename Emit>
__device__ __forceinline__ bool sep_tile(double* sm, const SepArgs& a, int64_t r,
                                         const double (&rx)[MU], const double (&ry)[MU],
                                         const double (&cx)[NV], const double (&cy)[NV],
                                         const Emit& emit) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lh = lane >> 4;
    const int64_t s = r / a.R_block;
    const double* fx = a.fx + s * a.K;
    const double* fy = a.fy + s * a.K;
    const double* w = a.w + s * a.K;
    f64x4 acc[MU][NV];
#pragma unroll
    for (int m = 0; m < MU; ++m)
#pragma unroll
        for (int n = 0; n < NV; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};

    bool finite = true;
    const int64_t kw = ((a.K + 8 * WV - 1) / (8 * WV)) * 8;
    const int64_t kb = wave * kw;
    const int64_t ke = kb + kw < a.K ? kb + kw : a.K;
    constexpr int FS = sep_stage(DIFF);
    double* st = sm + wave * SEP_KC * FS;
    for (int64_t k0 = kb; k0 < ke; k0 += SEP_KC) {
        {
            const int64_t k = k0 + 2 * lane;
            double g[4] = {0.0, 0.0, 0.0, 0.0};
            if (k < ke) {
                if (a.coef) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (k + q / 2 < ke) g[q] = a.coef[r * 2 * a.K + 2 * k + q];
                } else {
                    coef4_f64(a.seed, a.counter + (uint64_t)r, (uint32_t)(k >> 1), a.mode, g);
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool ok = k + h < ke;
                const double f0 = ok ? fx[k + h] : 0.0, f1 = ok ? fy[k + h] : 0.0;
                const double wk = ok ? w[k + h] : 0.0;
                double ca = wk * g[2 * h], cb = wk * g[2 * h + 1];
                if constexpr (!DIFF) finite &= isfinite(ca) && isfinite(cb);
                if constexpr (DIFF) {
                    double sh, ch;
                    sincos2pi_reduced(0.5 * frac_centered(f0 * a.dx + f1 * a.dy), sh, ch);
                    const double oc = 2.0 * sh * sh, sd = 2.0 * sh * ch;
                    const double ta = fma(ca, oc, -(cb * sd));
                    cb = fma(cb, oc, ca * sd);
                    ca = ta;
                }
                double2* dst = (double2*)(st + (2 * lane + h) * FS);
                dst[0] = make_double2(f0, f1);
                dst[1] = make_double2(ca, cb);
                if constexpr (DIFF) {
                    // the turns from the first 16 rows and columns to the next
                    double s1, c1;
                    const double step = fma(f0, a.sx, f1 * a.sy);
                    sincos2pi_reduced(frac_centered(step * (16.0 * a.V)), s1, c1);
                    dst[2] = make_double2(s1, c1);
                    sincos2pi_reduced(frac_centered(step * 16.0), s1, c1);
                    dst[3] = make_double2(s1, c1);
                }
            }
        }
        // the wave's own stage: written and read by the same wave
        __builtin_amdgcn_wave_barrier();
        __threadfence_block();
        const int64_t left = ke - k0;
        const int steps = left >= SEP_KC ? SEP_KC / 4 : (int)((left + 3) / 4);
        for (int g = 0; g < steps; ++g) {
            const double2* src = (const double2*)(st + (4 * g + lh) * FS);
            const double2 f = src[0], c = src[1];
            double A[MU], B[MU];
            double sn = 0.0, cs = 0.0;
#pragma unroll
            for (int m = 0; m < MU; ++m) {
                if (DIFF && m > 0) {
                    // (B, A) = (Im, Re) of c e^(-i phase), turned back
                    A[m] = A[m - 1];
                    B[m] = -B[m - 1];
                    turn(src[2], B[m], A[m]);
                    B[m] = -B[m];
                    continue;
                }
                sincos2pi_reduced(frac_centered(fma(f.x, rx[m], f.y * ry[m])), sn, cs);
                A[m] = fma(c.x, cs, c.y * sn);
                B[m] = fma(c.y, cs, -(c.x * sn));
            }
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                if (DIFF && n > 0) {
                    turn(src[3], sn, cs);
                } else {
                    sincos2pi_reduced(frac_centered(fma(f.x, cx[n], f.y * cy[n])), sn, cs);
                }
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
            double* dst = sm + (wave - half) * (256 * MU * NV) + lane;
#pragma unroll
            for (int m = 0; m < MU; ++m)
#pragma unroll
                for (int n = 0; n < NV; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[((m * NV + n) * 4 + i) * 64] = acc[m][n][i];
        }
        __syncthreads();
        if (wave < half) {
            const double* src = sm + wave * (256 * MU * NV) + lane;
#pragma unroll
            for (int m = 0; m < MU; ++m)
#pragma unroll
                for (int n = 0; n < NV; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][n][i] += src[((m * NV + n) * 4 + i) * 64];
        }
    }
    if (wave == 0) {
#pragma unroll
        for (int m = 0; m < MU; ++m)
#pragma unroll
            for (int n = 0; n < NV; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) emit(m, n, i, acc[m][n][i]);
    }
    return !finite;
}

template <int WV>
__global__ __launch_bounds__(64 * WV) __attribute__((
    amdgpu_waves_per_eu(4, 8))) void k_series_diff(SepArgs a, int ut, int vt) {
    __shared__ SepSmem<true, 2, 2, WV> sm;
    const int lane = threadIdx.x & 63, li = lane & 15, lh = lane >> 4;
    const int64_t tiles = (int64_t)ut * vt;
    const int64_t r = a.r0 + (int64_t)blockIdx.x / tiles;
    const int tile = (int)((int64_t)blockIdx.x % tiles);
    const int u0 = (tile / vt) * 32, v0 = (tile % vt) * 32;
    double rx[2], ry[2], cx[2], cy[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const double tu = (double)((u0 + 16 * m + li) * a.V), tv = (double)(v0 + 16 * m + li);
        rx[m] = a.ox + tu * a.sx;
        ry[m] = a.oy + tu * a.sy;
        cx[m] = tv * a.sx;
        cy[m] = tv * a.sy;
    }
    double* out = (double*)a.out + r * a.P;
    sep_tile<true, 2, 2, WV>(sm.d, a, r, rx, ry, cx, cy, [&](int m, int n, int i, double v) {
        const int64_t p = (int64_t)(u0 + 16 * m + lh + 4 * i) * a.V + v0 + 16 * n + li;
        if (p < a.P) out[p] = v;
    });
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
            hipLaunchKernelGGL(k_series_diff<4>, dim3((unsigned)n), dim3(256), 0, st, a, ut, vt);
        else
            hipLaunchKernelGGL(k_series_diff<16>, dim3((unsigned)n), dim3(1024), 0, st, a, ut, vt);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------------------------------- regular grids ----
// Whether the points form a grid is decided on the device from their values in
// every call (the host only has pointers).  V = length of the first run of
// equal y (x varies fastest) or equal x, which every block finds from the first
// points; then every point p must equal (x[p mod V], y[p - p mod V]) (or the
// other way round), bit for bit up to the sign of zero: each tile of the first
// realisation checks its own points.  Where one fails, the general kernel,
// which follows, does the work (a kernel of its own that checked all points
// first took 6 us more).  So that few point sets get that far, every block first
// looks at one point per thread, spread over all of them: a disk whose first row
// divides their number fails there (400 realisations of 740 points x 512
// frequencies in FP32: 164 us without this look, 73 with it, 67 without the
// question; 128 x 1024 on a grid of 32 x 32 in FP64 36 and 37 us).
// max_pad: largest ratio of padded tile area to points that is taken.
// Rows and columns are padded to whole units: 16, or 32 in the tiles of 64 x 64
// that grids of at least 4096 points use.
__host__ __device__ constexpr int grid_unit(int64_t P) { return P >= 4096 ? 32 : 16; }

// Whether point p, in column v of its row, is off the grid.
__device__ __forceinline__ bool grid_off(const double* __restrict__ px,
                                         const double* __restrict__ py, int p, int v, int V,
                                         int xfast) {
    return !(px[p] == px[xfast ? v : p - v]) || !(py[p] == py[xfast ? p - v : v]);
}

// The whole block calls it (P > 1).
__device__ __forceinline__ bool grid_shape(const double* __restrict__ px,
                                           const double* __restrict__ py, int64_t P,
                                           double max_pad, int& V, int& xfast, int* s_run) {
    const int tid = threadIdx.x, n = (int)P;
    if (tid == 0) *s_run = GRID_MAX_V + 1;
    __syncthreads();
    xfast = py[1] == py[0] ? 1 : 0;
    const double* q = xfast ? py : px;
    const double q0 = q[0];
    for (int base = 1; base < n && base <= GRID_MAX_V; base += (int)blockDim.x) {
        const int p = base + tid;
        const unsigned long long m = __ballot(p < n && q[p < n ? p : 0] != q0);
        if (m && (tid & 63) == 0) atomicMin(s_run, base + tid + __ffsll(m) - 1);
        __syncthreads();
        const bool found = *s_run <= GRID_MAX_V;
        __syncthreads();
        if (found) break;
    }
    V = *s_run;
    if (V < 2 || V > GRID_MAX_V || n % V) return false;
    const int unit = grid_unit(P);
    const double u = (double)((n / V + unit - 1) / unit * unit);
    if (u * (double)((V + unit - 1) / unit * unit) > max_pad * (double)P) return false;
    const int p = (int)((int64_t)tid * n / (int)blockDim.x);
    return !__syncthreads_or(grid_off(px, py, p, p % V, V, xfast));
}

template <typename T, int MU, int NV, int WV>
__device__ __forceinline__ void grid_tile(double* sm, const SepArgs& a, int64_t r, int U, int V,
                                          int xfast, int u0, int v0, const GridWord& g) {
    const int lane = threadIdx.x & 63, li = lane & 15, lh = lane >> 4;
    if (r == 0) {
        bool bad = false;
        for (int e = threadIdx.x; e < 256 * MU * NV; e += 64 * WV) {
            const int u = u0 + e / (16 * NV), v = v0 + e % (16 * NV);
            if (u < U && v < V) bad |= grid_off(a.px, a.py, u * V + v, v, V, xfast);
        }
        if (__any(bad) && lane == 0) atomicMax(g.word, 2 * g.id + 1);
    }
    double rx[MU], ry[MU], cx[NV], cy[NV];
#pragma unroll
    for (int m = 0; m < MU; ++m) {
        const int u = u0 + 16 * m + li;
        const int64_t p = (int64_t)(u < U ? u : 0) * V;
        rx[m] = xfast ? 0.0 : a.px[p];
        ry[m] = xfast ? a.py[p] : 0.0;
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
        const int v = v0 + 16 * m + li;
        const int64_t p = v < V ? v : 0;
        cx[m] = xfast ? a.px[p] : 0.0;
        cy[m] = xfast ? 0.0 : a.py[p];
    }
    T* out = (T*)a.out + r * a.P;
    const bool inf =
        sep_tile<false, MU, NV, WV>(sm, a, r, rx, ry, cx, cy, [&](int m, int q, int i, double s) {
            const int u = u0 + 16 * m + lh + 4 * i, v = v0 + 16 * q + li;
            if (u < U && v < V) out[(int64_t)u * V + v] = (T)s;
        });
    // infinities go through the general kernel, as if the points were no grid
    if (__any(inf) && lane == 0) atomicMax(g.word, 2 * g.id + 1);
}

// Sums on a grid: blocks take (realisation, tile) in turn, tiles at the edges in
// half the size where that holds them.
// Registers for 4 waves per SIMD, 2 in the largest tiles (700 realisations of 64
// x 64 points x 500 frequencies: 225 us with 2 and 1, 171 so).
template <typename T, int MU, int NV, int WV>
__global__ __launch_bounds__(64 * WV) __attribute__((
    amdgpu_waves_per_eu(MU * NV >= 16 ? 2 : 4, 8))) void k_grid_sum(SepArgs a, double max_pad,
                                                                    GridWord g) {
    __shared__ SepSmem<false, MU, NV, WV> sm;
    __shared__ int s_run;
    int V, xfast;
    const bool ok = grid_shape(a.px, a.py, a.P, max_pad, V, xfast, &s_run);
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicMax(g.word, 2 * g.id + (ok ? 0 : 1));
    if (!ok) return;
    constexpr int HU = MU > 1 ? MU / 2 : 1, HV = NV > 1 ? NV / 2 : 1;
    const int U = (int)(a.P / V);
    const int ut = (U + 16 * MU - 1) / (16 * MU), vt = (V + 16 * NV - 1) / (16 * NV);
    const int64_t tiles = (int64_t)ut * vt, n = a.R * tiles;
    for (int64_t it = blockIdx.x; it < n; it += gridDim.x) {
        const int64_t r = it / tiles;
        const int tile = (int)(it % tiles);
        const int u0 = (tile / vt) * 16 * MU, v0 = (tile % vt) * 16 * NV;
        const bool hu = HU < MU && U - u0 <= 16 * HU, hv = HV < NV && V - v0 <= 16 * HV;
        if (hu && hv)
            grid_tile<T, HU, HV, WV>(sm.d, a, r, U, V, xfast, u0, v0, g);
        else if (hu)
            grid_tile<T, HU, NV, WV>(sm.d, a, r, U, V, xfast, u0, v0, g);
        else if (hv)
            grid_tile<T, MU, HV, WV>(sm.d, a, r, U, V, xfast, u0, v0, g);
        else
            grid_tile<T, MU, NV, WV>(sm.d, a, r, U, V, xfast, u0, v0, g);
        __syncthreads();  // the next item reuses the stage
    }
}

double grid_max_pad(bool fp64, int64_t R_block) {
    // cycles of a SIMD per 64 terms: ~24 here; the general kernels ~180 / R_block
    // + 8 in binary64 and ~55 / R_block + 5 in FP32
    if (fp64) return R_block == 1 ? 6.0 : (R_block == 2 ? 3.0 : (R_block <= 4 ? 1.6 : 0.0));
    return R_block == 1 ? 2.0 : 0.0;
}

template <typename T>
static hipError_t launch_grid_sum_t(const SepArgs& a, double max_pad, GridWord g,
                                    hipStream_t st) {
    // tiles of 64 x 64 spare sines and cosines on the larger grids (13 cycles
    // of a SIMD per 64 terms, 17 in tiles of 32 x 32, 21 in 32 x 16); with few
    // realisations the 16 waves of a block split the frequencies, and where
    // tiles of 32 x 32 leave half the compute units idle they are halved.  1024
    // blocks at most, 2 to 4 per compute unit: where the points are no grid every
    // block only starts and ends (8192 of them took 30 us)
    const int64_t items = a.R * ((a.P + 1023) / 1024);
    if (grid_unit(a.P) == 32 && a.R * ((a.P + 4095) / 4096) >= 512)
        hipLaunchKernelGGL((k_grid_sum<T, 4, 4, 4>),
                           dim3((unsigned)(a.R * (a.P / 4096) < 1024 ? a.R * (a.P / 4096) : 1024)),
                           dim3(256), 0, st, a, max_pad, g);
    else if (items >= 512)
        hipLaunchKernelGGL((k_grid_sum<T, 2, 2, 4>), dim3((unsigned)(items < 1024 ? items : 1024)),
                           dim3(256), 0, st, a, max_pad, g);
    else if (items > 128)
        hipLaunchKernelGGL((k_grid_sum<T, 2, 2, 16>), dim3((unsigned)items), dim3(1024), 0, st, a,
                           max_pad, g);
    else
        hipLaunchKernelGGL((k_grid_sum<T, 2, 1, 16>), dim3((unsigned)(2 * items)), dim3(1024), 0,
                           st, a, max_pad, g);
    return hipGetLastError();
}

hipError_t launch_grid_sum(bool fp64, const SepArgs& a, double max_pad, GridWord g,
                           hipStream_t st) {
    return fp64 ? launch_grid_sum_t<double>(a, max_pad, g, st)
                : launch_grid_sum_t<float>(a, max_pad, g, st);
}

}  // namespace qrfs
