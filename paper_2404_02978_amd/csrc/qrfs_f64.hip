// qrfs_f64.hip -- the binary64 contraction of Eq. 3 for sets shared by many
// realisations, on the FP64 matrix instructions of gfx950.
#include "qrfs_mfma.hpp"

namespace qrfs {

// A block is 8 waves: WR waves own different rows (16 MR each) of one output
// tile of 16 NC columns, and WK = 8 / WR groups of them split the
// frequencies.  Per chunk of 8 frequencies a group builds the basis (cos, sin
// times the amplitude, binary64) of the next chunk in one of its two LDS
// buffers, and each lane draws the Philox blocks of its own A operand:
// lane (i = l % 16, h = l / 16) holds row i and the 4 coefficients of block h
// of the chunk, j = 4 h + q, which step q consumes together with the basis
// values (column i, j = 4 h + q) that the lane reads from LDS with two 16-byte
// loads (the contraction order is permuted, the result is not).  The groups'
// sums are added in a fixed tree, then stored (as this frequency range's share
// when the launch cuts K into ranges) or squared.
//
// Bound: the FP64 datapath, shared by the matrix instructions and the vector
// ALU (measured: the times add).  Per (row, frequency): two coefficients, 86
// vector operations; 16 NC columns, 32 NC multiply-adds; the basis, ~40
// operations per column, shared by the group's 16 MR WR rows.  The vector
// kernel this replaces read two basis values and eight coefficients from LDS
// per 8 multiply-adds and was bound there.
constexpr int FM_WAVES = 8;
constexpr int FM_KC = 8;                // frequencies per chunk
constexpr int FM_STR = 2 * FM_KC + 2;   // doubles per basis column: 16-byte rows, 16 lanes on
                                        // 16 different groups of 4 banks

template <int MR, int NC>
struct FmSmem {
    static constexpr int NT = 16 * NC;
    static constexpr int BASIS = 2 * NT * FM_STR;                // one group's two buffers
    static constexpr int TREE = (FM_WAVES / 2) * 256 * MR * NC;  // half the waves' tiles
};

template <int BASIS, int EPI, int MR, int NC, int WR, int CSRC>
__global__ __launch_bounds__(64 * FM_WAVES) void k_sum_fm(SumArgs a, int64_t row_tiles,
                                                          int64_t col_tiles) {
    using S = FmSmem<MR, NC>;
    constexpr int NT = S::NT, WK = FM_WAVES / WR, GT = 64 * WR;
    constexpr int NB = S::BASIS * WK > S::TREE ? S::BASIS * WK : S::TREE;
    __shared__ __attribute__((aligned(16))) double sB[NB];
    __shared__ double sF[WK][3][FM_KC][4];  // fx, fy, amplitude of three chunks
    __shared__ double sred[WR][NT][2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lh = lane >> 4;
    const int kg = wave / WR, wr = wave % WR;  // frequency group, row wave
    const int gt = tid % GT;                   // thread of the group
    int64_t b = blockIdx.x;
    const int64_t ct = b % col_tiles;
    b /= col_tiles;
    const int64_t ks = b % a.ksplit;  // frequency range
    b /= a.ksplit;
    const int64_t rt = b % row_tiles;
    const int64_t sl = b / row_tiles;
    const int64_t set = a.set0 + sl;
    const int64_t row0 = set * a.R_block + rt * (16 * MR * WR) + wr * (16 * MR);
    const int64_t row_end = (set + 1) * a.R_block < a.R ? (set + 1) * a.R_block : a.R;
    const int64_t col0 = ct * NT;
    const double* fx = a.fx + sl * a.K;
    const double* fy = a.fy + sl * a.K;
    const double* w = a.w + sl * a.K;
    const int64_t twoK = 2 * a.K;
    const int64_t kr = ks * a.kspan;
    const int64_t ke = kr + a.kspan < a.K ? kr + a.kspan : a.K;
    const int64_t nch = (ke - kr + FM_KC * WK - 1) / (FM_KC * WK);  // chunks per group
    const int64_t kb = kr + kg * nch * FM_KC;
    double* basis = sB + kg * S::BASIS;

    // basis work: this thread's column, frequencies part, part + PARTS, ...
    constexpr int PARTS = GT / NT > FM_KC ? FM_KC : GT / NT;
    const int bc = gt % NT, part = gt / NT;
    const bool cok = col0 + bc < a.P;
    const double px = cok ? a.px[col0 + bc] : 0.0;
    const double py = cok ? a.py[col0 + bc] : 0.0;
    double pD = 1.0, pd = 0.0;
    if (BASIS == BASIS_PISTON && cok) {
        pD = a.apD[col0 + bc];
        pd = a.apd[col0 + bc];
    }

    auto load_freq = [&](int64_t ch, double (&f)[3]) {
        const int64_t k = kb + ch * FM_KC + gt;
        const bool ok = gt < FM_KC && ch < nch && k < ke;
        f[0] = ok ? fx[k] : 0.0;
        f[1] = ok ? fy[k] : 0.0;
        f[2] = ok ? w[k] : 0.0;
    };
    auto stage = [&](int64_t ch, const double (&f)[3]) {
        if (gt < FM_KC) {
            double* d = sF[kg][ch % 3][gt];
            d[0] = f[0];
            d[1] = f[1];
            d[2] = f[2];
        }
    };
    auto produce = [&](int64_t ch) {
        double* dst = basis + (ch & 1) * (NT * FM_STR) + bc * FM_STR;
        if (part < PARTS)
#pragma unroll
            for (int i = 0; i < FM_KC / PARTS; ++i) {
                const int kk = part + i * PARTS;
                const double* f = sF[kg][ch % 3][kk];
                const double cfx = f[0], cfy = f[1];
                double t = cfx * px + cfy * py;
                if (BASIS == BASIS_PISTON) t += grad_shift(a.grad);
                const double rf = frac_centered(t);
                double sv, cv;
                if (BASIS == BASIS_DIFF) {
                    // cos 2 pi r - 1 = -2 sin^2 pi r, sin 2 pi r = 2 sin cos
                    double sh, chh;
                    sincos2pi_reduced(0.5 * rf, sh, chh);
                    cv = -2.0 * sh * sh;
                    sv = 2.0 * sh * chh;
                } else {
                    sincos2pi_reduced(rf, sv, cv);
                }
                double amp = f[2];
                if (BASIS == BASIS_PISTON)
                    amp *= aperture_filter(pD, pd, sqrt(cfx * cfx + cfy * cfy)) *
                           grad_factor(a.grad, a.gx, a.gy, cfx, cfy);
                *(double2*)&dst[2 * kk] = make_double2(amp * cv, amp * sv);
            }
    };

    f64x4 acc[MR][NC];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int n = 0; n < NC; ++n) acc[m][n] = f64x4{0.0, 0.0, 0.0, 0.0};

    double f[3];
    load_freq(0, f);
    stage(0, f);
    load_freq(1, f);
    stage(1, f);
    __syncthreads();
    produce(0);
    __syncthreads();
    for (int64_t ch = 0; ch < nch; ++ch) {
        load_freq(ch + 2, f);
        if (ch + 1 < nch) produce(ch + 1);
        const int64_t k0 = kb + ch * FM_KC;
        double g[MR][4];
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const int64_t r = row0 + 16 * m + li;
            // rows past the set feed only rows that are never stored or
            // squared, frequencies past K a basis of zeros
            if constexpr (CSRC == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t j = 2 * k0 + 4 * lh + q;
                    g[m][q] = (r < row_end && j < twoK) ? a.coef[r * twoK + j] : 0.0;
                }
            } else {
                coef4_f64(a.seed, a.counter + (uint64_t)r, (uint32_t)(k0 / 2) + (uint32_t)lh, CSRC,
                          g[m]);
            }
        }
        const double* B = basis + (ch & 1) * (NT * FM_STR) + li * FM_STR + 4 * lh;
        double bv[NC][4];
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            const double2 v0 = *(const double2*)&B[n * 16 * FM_STR];
            const double2 v1 = *(const double2*)&B[n * 16 * FM_STR + 2];
            bv[n][0] = v0.x;
            bv[n][1] = v0.y;
            bv[n][2] = v1.x;
            bv[n][3] = v1.y;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int m = 0; m < MR; ++m) acc[m][n] = mfma_f64(g[m][q], bv[n][q], acc[m][n]);
        stage(ch + 2, f);
        __syncthreads();
    }

    // fixed tree over the frequency groups: the upper half stores, the lower adds
#pragma unroll
    for (int half = WK / 2; half > 0; half >>= 1) {
        if (kg >= half && kg < 2 * half) {
            double* dst = sB + ((kg - half) * WR + wr) * (256 * MR * NC) + lane;
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int n = 0; n < NC; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[((m * NC + n) * 4 + i) * 64] = acc[m][n][i];
        }
        __syncthreads();
        if (kg < half) {
            const double* src = sB + (kg * WR + wr) * (256 * MR * NC) + lane;
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int n = 0; n < NC; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][n][i] += src[((m * NC + n) * 4 + i) * 64];
        }
        __syncthreads();
    }
    // element i of acc[m][n]: row 16 m + lh + 4 i, column 16 n + li
    if (EPI == EPI_STORE) {
        if (kg == 0) {
            double* out = a.ksplit > 1 ? (double*)a.phi_part + ks * a.R * a.P : (double*)a.out;
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
                for (int n = 0; n < NC; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int64_t r = row0 + 16 * m + lh + 4 * i, c = col0 + 16 * n + li;
                        if (r < row_end && c < a.P) out[r * a.P + c] = acc[m][n][i];
                    }
        }
    } else {
        if (kg == 0) {
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                double s2 = 0.0, s4 = 0.0;
#pragma unroll
                for (int m = 0; m < MR; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (row0 + 16 * m + lh + 4 * i < row_end) {
                            const double d2 = acc[m][n][i] * acc[m][n][i];
                            s2 += d2;
                            s4 += d2 * d2;
                        }
#pragma unroll
                for (int off = 16; off < 64; off <<= 1) {
                    s2 += __shfl_xor(s2, off);
                    s4 += __shfl_xor(s4, off);
                }
                if (lh == 0) {
                    sred[wr][16 * n + li][0] = s2;
                    sred[wr][16 * n + li][1] = s4;
                }
            }
        }
        __syncthreads();
        if (tid < NT && col0 + tid < a.P) {
            double t2 = 0.0, t4 = 0.0;
#pragma unroll
            for (int v = 0; v < WR; ++v) {
                t2 += sred[v][tid][0];
                t4 += sred[v][tid][1];
            }
            double* dst = a.partial + ((sl * row_tiles + rt) * a.P + col0 + tid) * 2;
            dst[0] = t2;
            dst[1] = t4;
        }
    }
}

// ----------------------------------------------------------- launchers ----
static inline int64_t fcdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Tile of a problem: 16 rows per wave where a set has no more, else 32;
// columns per block and row waves that share a basis by the estimated time
// of the fullest compute unit.  Blocks come in whole rounds of the 256 compute
// units; a block's wave takes 16 MR rows and WR / 8 of its range's frequencies,
// and a (row, frequency) costs 86 operations for its coefficients, 2 per
// column, and the basis of its columns shared by the group's rows: ~40
// operations each, ~300 with the binary64 filter of two edges.  (Fewer row
// waves and columns: more and shorter blocks that fill the chip evenly, but
// more basis work and coefficients drawn more often.)  A wave instruction
// takes 4 cycles of a SIMD; the kernel reaches about 0.6 of that at 2.4 GHz.
FmShape fm_shape(int basis, int64_t K, int64_t R, int64_t R_block, int64_t P, int ksplit) {
    FmShape s{};
    s.MR = R_block <= 16 ? 1 : 2;
    s.us = 1e300;
    const int64_t n_sets = fcdiv(R, R_block);
    const double col_ops = basis == BASIS_PISTON ? 300.0 : 40.0;
    const int nc_max = P <= 16 ? 1 : (P <= 32 ? 2 : 4);
    for (int nc = nc_max; nc >= 1; nc >>= 1)
        for (int wr = 8; wr >= 1; wr >>= 1) {
            const int64_t blocks =
                ksplit * n_sets * fcdiv(R_block, 16 * s.MR * wr) * fcdiv(P, 16 * nc);
            const double per_row = 86.0 + 32.0 * nc + col_ops * nc / (s.MR * wr);
            // 8 waves on 4 SIMDs, 16 MR rows on 64 lanes, 4 cycles
            const double us = (double)fcdiv(blocks, 256) * ((double)K / ksplit) * wr * s.MR *
                              per_row * (0.25 / 0.6 / 2400.0);
            if (us < s.us * 0.97) {
                s.us = us;
                s.NC = nc;
                s.WR = wr;
            }
        }
    return s;
}

template <int BASIS, int EPI, int MR, int NC, int WR>
static hipError_t launch_fm_w(const SumArgs& a, hipStream_t st) {
    const int64_t row_tiles = fcdiv(a.R_block, 16 * MR * WR), col_tiles = fcdiv(a.P, 16 * NC);
    const dim3 g((unsigned)((a.set1 - a.set0) * row_tiles * col_tiles * a.ksplit)), b(64 * FM_WAVES);
    if (a.coef)
        hipLaunchKernelGGL((k_sum_fm<BASIS, EPI, MR, NC, WR, 2>), g, b, 0, st, a, row_tiles,
                           col_tiles);
    else if (a.mode == 1)
        hipLaunchKernelGGL((k_sum_fm<BASIS, EPI, MR, NC, WR, 1>), g, b, 0, st, a, row_tiles,
                           col_tiles);
    else
        hipLaunchKernelGGL((k_sum_fm<BASIS, EPI, MR, NC, WR, 0>), g, b, 0, st, a, row_tiles,
                           col_tiles);
    return hipGetLastError();
}

template <int BASIS, int EPI, int MR, int NC>
static hipError_t launch_fm_n(const SumArgs& a, int WR, hipStream_t st) {
    if (WR == 8) return launch_fm_w<BASIS, EPI, MR, NC, 8>(a, st);
    if (WR == 4) return launch_fm_w<BASIS, EPI, MR, NC, 4>(a, st);
    if (WR == 2) return launch_fm_w<BASIS, EPI, MR, NC, 2>(a, st);
    return launch_fm_w<BASIS, EPI, MR, NC, 1>(a, st);
}

template <int BASIS, int EPI, int MR>
static hipError_t launch_fm_m(const SumArgs& a, const FmShape& s, hipStream_t st) {
    if (s.NC == 4) return launch_fm_n<BASIS, EPI, MR, 4>(a, s.WR, st);
    if (s.NC == 2) return launch_fm_n<BASIS, EPI, MR, 2>(a, s.WR, st);
    return launch_fm_n<BASIS, EPI, MR, 1>(a, s.WR, st);
}

template <int BASIS, int EPI>
static hipError_t launch_fm_t(const SumArgs& a, hipStream_t st) {
    const FmShape s = fm_shape(BASIS, a.K, a.R, a.R_block, a.P, a.ksplit);
    return s.MR == 1 ? launch_fm_m<BASIS, EPI, 1>(a, s, st) : launch_fm_m<BASIS, EPI, 2>(a, s, st);
}

hipError_t launch_sum_fm(int basis, int epi, const SumArgs& a, hipStream_t st) {
    if (epi == EPI_SFSUM) return launch_fm_t<BASIS_DIFF, EPI_SFSUM>(a, st);
    if (basis == BASIS_PHASE) return launch_fm_t<BASIS_PHASE, EPI_STORE>(a, st);
    if (basis == BASIS_PISTON) return launch_fm_t<BASIS_PISTON, EPI_STORE>(a, st);
    return launch_fm_t<BASIS_DIFF, EPI_STORE>(a, st);
}

}  // namespace qrfs
