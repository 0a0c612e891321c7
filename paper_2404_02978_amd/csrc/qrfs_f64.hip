// qrfs_f64.hip -- the binary64 contraction of Eq. 3 for sets shared by many
// realisations, on the FP64 matrix instructions of gfx950.
#include "qrfs_mfma.hpp"

namespace qrfs {

// --------------------------------------------------------- coefficients ----
// The generator of qrfs_device.hpp with tables of 64 entries in LDS, for a kernel
// that draws most of its time (gen_gauss_table.py): entry i holds r, about 1 / c,
// and 2 ln r for the mantissas around c = 1/2 + (i + 1/2) / 128 (r = 1 in the last,
// so that u near 1 cancels nothing), and sin, cos of 2 pi (i + 1/2) / 64 in two
// parts each.  With u = (2m + 1) 2^-24 = f 2^e: -2 ln u = 2 ln r - 2 log1p(f r - 1)
// - 2 e ln 2, |f r - 1| <= 1/128, log1p by its series through the 8th power (first
// omitted term 2e-18), small terms first; 2 ln r - 2 e ln 2 is exact but for the
// latter's low part.  The angle is the entry's, turned by what is left of it, at most
// 1/128 revolution, by the first terms of the series for 1/8.  A million pairs: within
// 3.04e-16 of the radius, 5.70e-17 RMS (sqrt, log and sincospi: 3.04e-16 and
// 5.72e-17), at ~56 vector instructions a pair in the place of ~100.  1e5 realisations
// x 4096 frequencies x 32 baselines: 2.16 ms, 2.70 without the tables, 2.07 with
// tables whose rounding showed (3.87e-16 and 7.0e-17).
static __device__ __attribute__((aligned(16))) const double kGaussTab[64][6] = {
    {1.9844961240301546, 1.370730080234921, 0.049067674327418015, 0.9987954562051724,
     -6.79610372051828e-19, -1.2291693337075465e-17},
    {1.9541984737338076, 1.3399602430187656, 0.14673047445536175, 0.989176509964781,
     3.726947147046568e-18, -4.098730993704711e-17},
    {1.9248120305217513, 1.3096566329796246, 0.2429801799032639, 0.970031253194544,
     -8.751431529719663e-18, 1.8365300348428844e-17},
    {1.8962962962953356, 1.2798053320812528, 0.33688985339222005, 0.9415440651830208,
     -4.200094003347509e-19, -2.789637954769834e-17},
    {1.8686131391203746, 1.250393037767651, 0.4275550934302821, 0.9039892931234433,
     9.411189816295473e-18, -6.609754468748431e-18},
    {1.8417266182762306, 1.2214070222320856, 0.5141027441932218, 0.8577286100002721,
     -4.5712707523615624e-17, -4.818344793633662e-17},
    {1.815602836459876, 1.1928351077406205, 0.5956993044924334, 0.8032075314806449,
     -1.3438641936579467e-17, -3.306060980481491e-17},
    {1.790209790622127, 1.164665628899968, 0.6715589548470184, 0.7409511253549591,
     -4.048903774929669e-17, -1.4708616952297345e-17},
    {1.7655172417868847, 1.1368874045796815, 0.7409511253549591, 0.6715589548470184,
     -1.4708616952297345e-17, -4.048903774929669e-17},
    {1.7414965986366826, 1.1094897153984675, 0.8032075314806449, 0.5956993044924334,
     -3.306060980481491e-17, -1.3438641936579467e-17},
    {1.718120804970509, 1.0824622766041898, 0.8577286100002721, 0.5141027441932218,
     -4.818344793633662e-17, -4.5712707523615624e-17},
    {1.6953642380174592, 1.0557952148654977, 0.9039892931234433, 0.4275550934302821,
     -6.609754468748431e-18, 9.411189816295473e-18},
    {1.673202613990444, 1.0294790457097065, 0.9415440651830208, 0.33688985339222005,
     -2.789637954769834e-17, -4.200094003347509e-19},
    {1.6516129032291549, 1.0035046551246865, 0.970031253194544, 0.2429801799032639,
     1.8365300348428844e-17, -8.751431529719663e-18},
    {1.6305732484066429, 0.9778632782612817, 0.989176509964781, 0.14673047445536175,
     -4.098730993704711e-17, 3.726947147046568e-18},
    {1.610062892710059, 0.9525464840569384, 0.9987954562051724, 0.049067674327418015,
     -1.2291693337075465e-17, -6.79610372051828e-19},
    {1.5900621121693315, 0.9275461594531862, 0.9987954562051724, -0.049067674327418015,
     -1.2291693337075465e-17, 6.79610372051828e-19},
    {1.570552146878473, 0.9028544868861559, 0.989176509964781, -0.14673047445536175,
     -4.098730993704711e-17, -3.726947147046568e-18},
    {1.5515151512604133, 0.8784639408295902, 0.970031253194544, -0.2429801799032639,
     1.8365300348428844e-17, 8.751431529719663e-18},
    {1.5329341317351102, 0.8543672641237663, 0.9415440651830208, -0.33688985339222005,
     -2.789637954769834e-17, 4.200094003347509e-19},
    {1.5147928994074684, 0.8305574591119012, 0.9039892931234433, -0.4275550934302821,
     -6.609754468748431e-18, -9.411189816295473e-18},
    {1.4970760230447533, 0.8070277754901554, 0.8577286100002721, -0.5141027441932218,
     -4.818344793633662e-17, 4.5712707523615624e-17},
    {1.4797687864697993, 0.7837717004266551, 0.8032075314806449, -0.5956993044924334,
     -3.306060980481491e-17, 1.3438641936579467e-17},
    {1.4628571431962445, 0.7607829415757124, 0.7409511253549591, -0.6715589548470184,
     -1.4708616952297345e-17, 4.048903774929669e-17},
    {1.4463276836141494, 0.7380554238091577, 0.6715589548470184, -0.7409511253549591,
     -4.048903774929669e-17, 1.4708616952297345e-17},
    {1.430167597768992, 0.7155832772826898, 0.5956993044924334, -0.8032075314806449,
     -1.3438641936579467e-17, 3.306060980481491e-17},
    {1.4143646408867057, 0.6933608264313307, 0.5141027441932218, -0.8577286100002721,
     -4.5712707523615624e-17, 4.818344793633662e-17},
    {1.3989071038259322, 0.6713825832774205, 0.4275550934302821, -0.9039892931234433,
     9.411189816295473e-18, 6.609754468748431e-18},
    {1.3837837837863356, 0.6496432388061635, 0.33688985339222005, -0.9415440651830208,
     -4.200094003347509e-19, 2.789637954769834e-17},
    {1.3689839569053195, 0.6281376547913169, 0.2429801799032639, -0.970031253194544,
     -8.751431529719663e-18, -1.8365300348428844e-17},
    {1.354497354183659, 0.606860858376649, 0.14673047445536175, -0.989176509964781,
     3.726947147046568e-18, 4.098730993704711e-17},
    {1.3403141361270006, 0.5858080328678739, 0.049067674327418015, -0.9987954562051724,
     -6.79610372051828e-19, 1.2291693337075465e-17},
    {1.3264248704667203, 0.5649745111499556, -0.049067674327418015, -0.9987954562051724,
     6.79610372051828e-19, 1.2291693337075465e-17},
    {1.3128205125175074, 0.5443557713700216, -0.14673047445536175, -0.989176509964781,
     -3.726947147046568e-18, 4.098730993704711e-17},
    {1.2994923854879543, 0.5239474310232026, -0.2429801799032639, -0.970031253194544,
     8.751431529719663e-18, -1.8365300348428844e-17},
    {1.2864321608071907, 0.5037452395150694, -0.33688985339222005, -0.9415440651830208,
     4.200094003347509e-19, 2.789637954769834e-17},
    {1.2736318407941747, 0.4837450728380759, -0.4275550934302821, -0.9039892931234433,
     -9.411189816295473e-18, 6.609754468748431e-18},
    {1.2610837438445397, 0.46394293087899996, -0.5141027441932218, -0.8577286100002721,
     4.5712707523615624e-17, 4.818344793633662e-17},
    {1.2487804878024695, 0.4443349306784512, -0.5956993044924334, -0.8032075314806449,
     1.3438641936579467e-17, 3.306060980481491e-17},
    {1.236714975848238, 0.42491730243295933, -0.6715589548470184, -0.7409511253549591,
     4.048903774929669e-17, 1.4708616952297345e-17},
    {1.224880382493843, 0.405686384570231, -0.7409511253549591, -0.6715589548470184,
     1.4708616952297345e-17, 4.048903774929669e-17},
    {1.2132701424608696, 0.3866386224698317, -0.8032075314806449, -0.5956993044924334,
     3.306060980481491e-17, 1.3438641936579467e-17},
    {1.2018779342719892, 0.36777055753975674, -0.8577286100002721, -0.5141027441932218,
     4.818344793633662e-17, 4.5712707523615624e-17},
    {1.1906976746938116, 0.34907883316606103, -0.9039892931234433, -0.4275550934302821,
     6.609754468748431e-18, -9.411189816295473e-18},
    {1.1797235025772344, 0.33056018234117346, -0.9415440651830208, -0.33688985339222005,
     2.789637954769834e-17, 4.200094003347509e-19},
    {1.168949771955645, 0.31221142978148464, -0.970031253194544, -0.2429801799032639,
     -1.8365300348428844e-17, 8.751431529719663e-18},
    {1.1583710407215355, 0.2940294859193955, -0.989176509964781, -0.14673047445536175,
     4.098730993704711e-17, -3.726947147046568e-18},
    {1.1479820630471371, 0.27601134650382164, -0.9987954562051724, -0.049067674327418015,
     1.2291693337075465e-17, 6.79610372051828e-19},
    {1.1377777775188667, 0.2581540840951675, -0.9987954562051724, 0.049067674327418015,
     1.2291693337075465e-17, -6.79610372051828e-19},
    {1.127753303961548, 0.24045485399062727, -0.989176509964781, 0.14673047445536175,
     4.098730993704711e-17, 3.726947147046568e-18},
    {1.1179039301295621, 0.2229108818480654, -0.970031253194544, 0.2429801799032639,
     -1.8365300348428844e-17, -8.751431529719663e-18},
    {1.1082251082215009, 0.20551946790902775, -0.9415440651830208, 0.33688985339222005,
     2.789637954769834e-17, -4.200094003347509e-19},
    {1.0987124463487308, 0.1882779818218978, -0.9039892931234433, 0.4275550934302821,
     6.609754468748431e-18, 9.411189816295473e-18},
    {1.089361702129727, 0.17118386067460278, -0.8577286100002721, 0.5141027441932218,
     4.818344793633662e-17, -4.5712707523615624e-17},
    {1.0801687763734018, 0.15423460669273936, -0.8032075314806449, 0.5956993044924334,
     3.306060980481491e-17, -1.3438641936579467e-17},
    {1.0711297068679422, 0.1374277846385894, -0.7409511253549591, 0.6715589548470184,
     1.4708616952297345e-17, -4.048903774929669e-17},
    {1.0622406641458795, 0.12076102243997866, -0.6715589548470184, 0.7409511253549591,
     4.048903774929669e-17, -1.4708616952297345e-17},
    {1.0534979423841346, 0.10423200227290863, -0.5956993044924334, 0.8032075314806449,
     1.3438641936579467e-17, -3.306060980481491e-17},
    {1.0448979589410512, 0.08783846740527679, -0.5141027441932218, 0.8577286100002721,
     4.5712707523615624e-17, -4.818344793633662e-17},
    {1.0364372469627228, 0.07157821570154965, -0.4275550934302821, 0.9039892931234433,
     -9.411189816295473e-18, -6.609754468748431e-18},
    {1.02811245003605, 0.055449096490463035, -0.33688985339222005, 0.9415440651830208,
     4.200094003347509e-19, -2.789637954769834e-17},
    {1.0199203189587593, 0.039449011153749325, -0.2429801799032639, 0.970031253194544,
     8.751431529719663e-18, 1.8365300348428844e-17},
    {1.0118577072759711, 0.023575911041746167, -0.14673047445536175, 0.989176509964781,
     -3.726947147046568e-18, -4.098730993704711e-17},
    {1.0, 0.0, -0.049067674327418015, 0.9987954562051724,
     6.79610372051828e-19, -1.2291693337075465e-17},
};
// -2 log1p(d) = -2 d + d^2 (1 - 2 d / 3 + 2 d^2 / 4 - ...)
constexpr double kLog1p[7] = {2.0 / 8, -2.0 / 7, 2.0 / 6, -2.0 / 5, 2.0 / 4, -2.0 / 3, 1.0};

struct GaussTab {
    double2 ln[64], sc[64], lo[64];  // r, 2 ln r; sin, cos; their low parts
};

__device__ __forceinline__ double gauss_radius_tab(const GaussTab& t, uint32_t x) {
    const double M = (double)((x >> 8) | 1u);  // 2m + 1
    const double f = __builtin_amdgcn_frexp_mant(M);
    const double e = (double)(__builtin_amdgcn_frexp_exp(M) - 24);
    const double2 L = t.ln[((uint32_t)__double2hiint(M) >> 14) & 63u];
    const double d = fma(f, L.x, -1.0);
    double p = kLog1p[0];
#pragma unroll
    for (int n = 1; n < 7; ++n) p = fma_s(p, d, kLog1p[n]);
    const double a = fma(e, -kTwoLn2Hi, L.y) + fma(-2.0, d, fma(d * d, p, e * -kTwoLn2Lo));
    double r = __builtin_amdgcn_rsq(a);
    r = fma(r, fma(-0.5 * a, r * r, 0.5), r);
    const double g = a * r;
    return fma(fma(-g, g, a), 0.5 * r, g);
}

__device__ __forceinline__ void sincos_tab(const GaussTab& t, uint32_t x, double& s, double& c) {
    const double2 sc = t.sc[x >> 26], lo = t.lo[x >> 26];
    const double z = fma((double)((x >> 9) & 0x1ffffu), 0x1p-23, 0x1p-24 - 0x1p-7);
    const double w = z * z;
    double ps = kSin2pi[4];
#pragma unroll
    for (int n = 5; n < 8; ++n) ps = fma_s(ps, w, kSin2pi[n]);
    ps *= z;
    double pc = kCos2pi[4];  // cos - 1
#pragma unroll
    for (int n = 5; n < 8; ++n) pc = fma_s(pc, w, kCos2pi[n]);
    pc *= w;
    s = sc.x + fma(sc.y, ps, fma(sc.x, pc, lo.x));
    c = sc.y + fma(-sc.x, ps, fma(sc.y, pc, lo.y));
}

__device__ __forceinline__ void coef4_tab(const GaussTab& t, uint64_t seed, uint64_t real,
                                          uint32_t blk, int mode, double g[4]) {
    double s, c;
    if (mode == 0) {
        const U32x4 x = coef_block(seed, real, blk);
        double rho = gauss_radius_tab(t, x.x);
        sincos_tab(t, x.y, s, c);
        g[0] = rho * c;
        g[1] = rho * s;
        rho = gauss_radius_tab(t, x.z);
        sincos_tab(t, x.w, s, c);
        g[2] = rho * c;
        g[3] = rho * s;
    } else {
        for (int h = 0; h < 2; ++h) {
            const U32x4 x = coef_block(seed, real, 2u * blk + (uint32_t)h);
            sincos_tab(t, x.y, s, c);
            const double rn = 1.4142135623730951 * (gauss_radius_tab(t, x.x) * c);
            sincos_tab(t, x.z, s, c);
            g[2 * h] = rn * c;
            g[2 * h + 1] = -rn * s;
        }
    }
}

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
// ALU (measured: the times add).  Per (row, frequency): two coefficients, ~56
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

// Registers for two blocks per compute unit where their sums leave room (32 rows
// x 64 columns per wave do not: 20 to 30 % slower with the spills).
template <int MR, int NC, int WR>
constexpr int fm_min_waves() {
    return WR >= 2 && MR * NC <= 4 ? 4 : 2;
}

template <int BASIS, int EPI, int MR, int NC, int WR, int CSRC>
__global__ __launch_bounds__(64 * FM_WAVES) __attribute__((
    amdgpu_waves_per_eu(fm_min_waves<MR, NC, WR>(), 8))) void
k_sum_fm(SumArgs a, int64_t row_tiles, int64_t col_tiles) {
    using S = FmSmem<MR, NC>;
    constexpr int NT = S::NT, WK = FM_WAVES / WR, GT = 64 * WR;
    constexpr int NB = S::BASIS * WK > S::TREE ? S::BASIS * WK : S::TREE;
    __shared__ __attribute__((aligned(16))) double sB[NB];
    __shared__ double sF[WK][3][FM_KC][4];  // fx, fy, amplitude of three chunks
    __shared__ double sred[WR][NT][2];
    __shared__ __attribute__((aligned(16))) GaussTab tab;

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

    if (CSRC < 2 && tid < 192) {
        const double2* src = (const double2*)kGaussTab[tid & 63] + (tid >> 6);
        (tid < 64 ? tab.ln : tid < 128 ? tab.sc : tab.lo)[tid & 63] = *src;
    }
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
                coef4_tab(tab, a.seed, a.counter + (uint64_t)r, (uint32_t)(k0 / 2) + (uint32_t)lh,
                          CSRC, g[m]);
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
// and a (row, frequency) costs ~56 operations for its coefficients, 2 per
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
            const double per_row = 56.0 + 32.0 * nc + col_ops * nc / (s.MR * wr);
            // 8 waves on 4 SIMDs, 16 MR rows on 64 lanes, 4 cycles
            const double us = (double)fcdiv(blocks, 256) * ((double)K / ksplit) * wr * s.MR *
                              per_row * (0.25 / 0.6 / 2400.0);
            if (us < s.us) {
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
