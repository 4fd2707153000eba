// HIP kernels for gfx950: the toy model of the paper's illustration, one
// particle diffusing on the two-dimensional asymmetric funnel of eq (U)
// (parameters of Table 1), many trajectories at once.
//
// One thread per trajectory (a group of 8 or 16 lanes under the tube ratchets
// when there are too few trajectories to fill the chip; see funnel_lanes), float64
// throughout.  Overdamped Langevin steps X += D F + sqrt(2 kT D) xi with
// D = dt / (m gamma); noise from Philox4x32-10 with counter (0, trajectory,
// step_lo, step_hi) and the Box-Muller transform of its first two words.
// Bias: the rMD ratchet on z = |X| (eq (FrMD)), or the ratchets on the tube
// variables of eqs (Fw),(Fs) with the Euclidean distance to the frames of
// the mean path (d_k = |X - <X(t_k)>|^2), the toy model's stand-in for the
// contact map, one exponential per frame and step.  T accumulates
// D |F_bias|^2 per step.
#include <math.h>

#include "scps_device.h"
#include "scps_funnel.h"
#include "scps_internal.h"

namespace scps {

__device__ __forceinline__ double unit_open_d(uint32_t w) { return (double)(2u * (w >> 9) + 1u) * 0x1p-24; }

// U of eq (U) is not needed on the step; F = -grad U.
__device__ __forceinline__ void funnel_force(const FunnelK &P, double x, double y, double &fx, double &fy) {
    const double r2 = x * x + y * y;
    const double a1 = r2 + P.s1 * P.s1, a2 = r2 + P.s2 * P.s2;
    const double dx = x - P.xm, dy = y - P.ym;
    const double a3 = dx * dx + dy * dy + P.s3 * P.s3;
    // radial part: d/dr^2 of w^2 r^4 - A1 s1^2 / a1^2 + A2 s2^2 / a2^2, times 2
    const double g_r = 4.0 * P.w * P.w * r2 + 4.0 * P.A1 * P.s1 * P.s1 / (a1 * a1 * a1) -
                       4.0 * P.A2 * P.s2 * P.s2 / (a2 * a2 * a2);
    const double g_3 = 4.0 * P.A3 * P.s3 * P.s3 / (a3 * a3 * a3);
    fx = -(g_r * x + g_3 * dx);
    fy = -(g_r * y + g_3 * dy);
}

// 2^(j / 64) as an unevaluated sum hi + lo of float64
__constant__ const double2 EXP2_64[64] = {
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.02c9a3e778061p+0, -0x1.19083535b085dp-56},
    {0x1.059b0d3158574p+0, 0x1.d73e2a475b465p-55}, {0x1.0874518759bc8p+0, 0x1.186be4bb284ffp-57},
    {0x1.0b5586cf9890fp+0, 0x1.8a62e4adc610bp-54}, {0x1.0e3ec32d3d1a2p+0, 0x1.03a1727c57b53p-59},
    {0x1.11301d0125b51p+0, -0x1.6c51039449b3ap-54}, {0x1.1429aaea92de0p+0, -0x1.32fbf9af1369ep-54},
    {0x1.172b83c7d517bp+0, -0x1.19041b9d78a76p-55}, {0x1.1a35beb6fcb75p+0, 0x1.e5b4c7b4968e4p-55},
    {0x1.1d4873168b9aap+0, 0x1.e016e00a2643cp-54}, {0x1.2063b88628cd6p+0, 0x1.dc775814a8495p-55},
    {0x1.2387a6e756238p+0, 0x1.9b07eb6c70573p-54}, {0x1.26b4565e27cddp+0, 0x1.2bd339940e9d9p-55},
    {0x1.29e9df51fdee1p+0, 0x1.612e8afad1255p-55}, {0x1.2d285a6e4030bp+0, 0x1.0024754db41d5p-54},
    {0x1.306fe0a31b715p+0, 0x1.6f46ad23182e4p-55}, {0x1.33c08b26416ffp+0, 0x1.32721843659a6p-54},
    {0x1.371a7373aa9cbp+0, -0x1.63aeabf42eae2p-54}, {0x1.3a7db34e59ff7p+0, -0x1.5e436d661f5e3p-56},
    {0x1.3dea64c123422p+0, 0x1.ada0911f09ebcp-55}, {0x1.4160a21f72e2ap+0, -0x1.ef3691c309278p-58},
    {0x1.44e086061892dp+0, 0x1.89b7a04ef80d0p-59}, {0x1.486a2b5c13cd0p+0, 0x1.3c1a3b69062f0p-56},
    {0x1.4bfdad5362a27p+0, 0x1.d4397afec42e2p-56}, {0x1.4f9b2769d2ca7p+0, -0x1.4b309d25957e3p-54},
    {0x1.5342b569d4f82p+0, -0x1.07abe1db13cadp-55}, {0x1.56f4736b527dap+0, 0x1.9bb2c011d93adp-54},
    {0x1.5ab07dd485429p+0, 0x1.6324c054647adp-54}, {0x1.5e76f15ad2148p+0, 0x1.ba6f93080e65ep-54},
    {0x1.6247eb03a5585p+0, -0x1.383c17e40b497p-54}, {0x1.6623882552225p+0, -0x1.bb60987591c34p-54},
    {0x1.6a09e667f3bcdp+0, -0x1.bdd3413b26456p-54}, {0x1.6dfb23c651a2fp+0, -0x1.bbe3a683c88abp-57},
    {0x1.71f75e8ec5f74p+0, -0x1.16e4786887a99p-55}, {0x1.75feb564267c9p+0, -0x1.0245957316dd3p-54},
    {0x1.7a11473eb0187p+0, -0x1.41577ee04992fp-55}, {0x1.7e2f336cf4e62p+0, 0x1.05d02ba15797ep-56},
    {0x1.82589994cce13p+0, -0x1.d4c1dd41532d8p-54}, {0x1.868d99b4492edp+0, -0x1.fc6f89bd4f6bap-54},
    {0x1.8ace5422aa0dbp+0, 0x1.6e9f156864b27p-54}, {0x1.8f1ae99157736p+0, 0x1.5cc13a2e3976cp-55},
    {0x1.93737b0cdc5e5p+0, -0x1.75fc781b57ebcp-57}, {0x1.97d829fde4e50p+0, -0x1.d185b7c1b85d1p-54},
    {0x1.9c49182a3f090p+0, 0x1.c7c46b071f2bep-56}, {0x1.a0c667b5de565p+0, -0x1.359495d1cd533p-54},
    {0x1.a5503b23e255dp+0, -0x1.d2f6edb8d41e1p-54}, {0x1.a9e6b5579fdbfp+0, 0x1.0fac90ef7fd31p-54},
    {0x1.ae89f995ad3adp+0, 0x1.7a1cd345dcc81p-54}, {0x1.b33a2b84f15fbp+0, -0x1.2805e3084d708p-57},
    {0x1.b7f76f2fb5e47p+0, -0x1.5584f7e54ac3bp-56}, {0x1.bcc1e904bc1d2p+0, 0x1.23dd07a2d9e84p-55},
    {0x1.c199bdd85529cp+0, 0x1.11065895048ddp-55}, {0x1.c67f12e57d14bp+0, 0x1.2884dff483cadp-54},
    {0x1.cb720dcef9069p+0, 0x1.503cbd1e949dbp-56}, {0x1.d072d4a07897cp+0, -0x1.cbc3743797a9cp-54},
    {0x1.d5818dcfba487p+0, 0x1.2ed02d75b3707p-55}, {0x1.da9e603db3285p+0, 0x1.c2300696db532p-54},
    {0x1.dfc97337b9b5fp+0, -0x1.1a5cd4f184b5cp-54}, {0x1.e502ee78b3ff6p+0, 0x1.39e8980a9cc8fp-55},
    {0x1.ea4afa2a490dap+0, -0x1.e9c23179c2893p-54}, {0x1.efa1bee615a27p+0, 0x1.dc7f486a4b6b0p-54},
    {0x1.f50765b6e4540p+0, 0x1.9d3e12dd8a18bp-54}, {0x1.fa7c1819e90d8p+0, 0x1.74853f3a5931ep-55},
};

// exp(x) for x <= 0 (the weights' exponents: differences to the largest one), by
// the table-driven method of P. T. P. Tang (ACM Trans. Math. Softw. 15, 144, 1989):
// x = (64 m + j) ln2 / 64 + r, exp(x) = 2^m 2^(j/64) e^r with the table in LDS and
// e^r - 1 by its series to r^5, |r| <= ln2 / 128, the r^6 term folded into r^4 and
// r^2 over that range (truncation below 1e-18).  hi (e^r - 1) + lo is added
// to hi last, so the result carries little more than one rounding (largest error
// 0.53 units in the last place over 1.2e7 random arguments).  14 float64
// instructions, where exp took 21 and three selects for the ranges that do not
// occur here.  Arguments below -746 give 0; so does NaN, which the caller looks for.
__device__ __forceinline__ double exp_neg(double x, const double2 *tab) {
    x = fmax(x, -746.0);
    const double magic = 0x1.8p52;
    const double t = fma(x, 0x1.71547652b82fep+6, magic);   // 64 / ln2; the integer in the low bits
    const int n = __double2loint(t);
    const double nd = t - magic;
    double r = fma(nd, -0x1.62e42fee00000p-7, x);
    r = fma(nd, -0x1.a39ef35793c76p-39, r);
    const double2 T = tab[n & 63];
    double p = fma(r, 0x1.1111111111111p-7, 0x1.55557621dbbb3p-5);
    p = fma(r, p, 0x1.5555555555555p-3);
    p = fma(r, p, 0x1.fffffffffd0bap-2);
    p = fma(r * r, p, r);
    return ldexp(T.x + fma(T.x, p, T.y), n >> 6);
}

// a * b, rounded: not to be fused into the sum it is added to, so that both forms of
// the weighted sums below have the same bits.
__device__ __forceinline__ double product(double a, double b) {
#pragma clang fp contract(off)
    return a * b;
}

// Minimum over the L neighbouring lanes of a trajectory (DPP within rows of 16:
// neighbours, pairs, then mirrored halves, whose lanes hold equal values by then).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}
template <int L>
__device__ __forceinline__ double group_min(double v) {
    if constexpr (L > 1) v = fmin(v, dpp_f64<0xB1>(v));
    if constexpr (L > 2) v = fmin(v, dpp_f64<0x4E>(v));
    if constexpr (L > 4) v = fmin(v, dpp_f64<0x141>(v));
    if constexpr (L > 8) v = fmin(v, dpp_f64<0x140>(v));
    return v;
}

// A trajectory's lanes lie in one wavefront, whose LDS operations keep their order;
// the compiler must not move them across this point.
__device__ __forceinline__ void group_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of one trajectory whose frames are shared by several lanes: FCH frames'
// weights e and k e, the differences x - x_k and y - y_k, and ones, in columns.  The
// length puts neighbouring trajectories 4 banks of 64 apart.
constexpr int FCH = 16;
struct FunnelChunk {
    double col[5][FCH];
    double pad[18];
};
static_assert(sizeof(FunnelChunk) % 256 == 16, "neighbours 16 bytes apart modulo the banks");

// L lanes per trajectory: lane t mod L takes the exponentials of the frames t mod
// L, + L, ..., FCH frames at a time, and then one of the six weighted sums over
// all of them, in frame order, so that the sums have the bits that one lane
// gives; the rest of the step runs in every lane alike.  Bound by float64 VALU
// issue where the trajectories fill the chip, by one wavefront's latency where
// they do not (us for 50 steps around 51 frames, one lane per trajectory with the
// library's exp -> now): 262144 trajectories 1080 -> 910,
// 65536 365 -> 322, 16384 362 -> 241, 8000 361 -> 168, 1000 to 4096 356 -> 145.
template <int BIAS, int L>
__global__ __launch_bounds__(256) void k_funnel_steps(const FunnelK P, int n_traj, int first_id,
                                                      double2 *__restrict__ xy, double *__restrict__ cv,
                                                      int64_t n_steps, uint64_t step0, int record_every,
                                                      double2 *__restrict__ frames, int K,
                                                      const double2 *__restrict__ mp) {
    __shared__ double2 path[FUNNEL_KMAX];
    __shared__ double2 tab[64];
    __shared__ __align__(16) FunnelChunk chunk[L > 1 ? 256 / L : 1];
    bool path_nan = false;
    if (BIAS == 1) {
        if (L > 1 && threadIdx.x / L < 256 / L)
            for (int q = threadIdx.x % L; q < FCH; q += L) chunk[threadIdx.x / L].col[4][q] = 1.0;
        bool nan = false;
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            const double2 f = mp[k];
            path[k] = f;
            nan |= f.x != f.x || f.y != f.y;
        }
        if (threadIdx.x < 64) tab[threadIdx.x] = EXP2_64[threadIdx.x];
        path_nan = __syncthreads_or(nan);
    }
    const int thread = blockIdx.x * blockDim.x + threadIdx.x;
    const int sub = thread % L;
    // lanes past the last trajectory repeat it without writing (a group's lanes
    // exchange values, so none may leave)
    const bool live = thread / L < n_traj;
    const int t = live ? thread / L : n_traj - 1;
    const bool writes = live && sub == 0;
    double x = xy[t].x, y = xy[t].y;
    double *c = cv + (int64_t)t * CV_STRIDE;
    double zm = c[CV_ZM], sm = c[CV_SM], wm = c[CV_WM], T = c[CV_T];
    double z = c[CV_Z], eb = c[CV_EB], sv = c[CV_S], wv = c[CV_W];
    const double D = P.mob_dt, amp = sqrt(2.0 * P.kT * P.mob_dt);
    const int M = K - 1;
    for (int64_t n = 0;; ++n) {
        if (writes && frames && record_every > 0 && n % record_every == 0)
            frames[(n / record_every) * n_traj + t] = make_double2(x, y);
        if (n == n_steps) break;
        double fx, fy, bx = 0.0, by = 0.0;
        funnel_force(P, x, y, fx, fy);
        if (BIAS == 0) {
            z = sqrt(x * x + y * y);
            zm = fmin(zm, z);
            const double dz = z - zm;
            if (z > 0.0) {
                bx = -P.k_R * dz * x / z;
                by = -P.k_R * dz * y / z;
            }
            eb = 0.5 * P.k_R * dz * dz;
        } else {
            // tube variables: the smallest distance (the largest exponent), then the
            // weights with the sums sum_k e_k (x - x_k) and sum_k k e_k (x - x_k), half
            // of sum_k e_k grad d_k and sum_k k e_k grad d_k, from which
            // grad s = (lambda / M) sum_k p_k (k - kbar) grad d_k and grad w = lambda wscale sum_k p_k grad d_k
            double d_min = INFINITY;
#pragma unroll 4
            for (int k = sub; k < K; k += L) {
                const double ex = x - path[k].x, ey = y - path[k].y;
                d_min = fmin(d_min, fma(ex, ex, ey * ey));
            }
            d_min = group_min<L>(d_min);
            const double a = -P.lambda * d_min;
            double s0 = 0.0, s1 = 0.0, ax = 0.0, ay = 0.0, kx = 0.0, ky = 0.0, kd = (double)sub;
            auto frame = [&](int k, double &ex, double &ey) {
                ex = x - path[k].x;
                ey = y - path[k].y;
                return exp_neg(fma(-P.lambda, fma(ex, ex, ey * ey), -a), tab);
            };
            auto add = [&](double e, double ke, double ex, double ey) {
                s0 += e;
                s1 += ke;
                ax = fma(e, ex, ax);
                ay = fma(e, ey, ay);
                kx = fma(ke, ex, kx);
                ky = fma(ke, ey, ky);
            };
            if constexpr (L == 1) {
                int k = 0;
                for (; k + 1 < K; k += 2) {   // two frames at a time
                    double ex0, ey0, ex1, ey1;
                    const double e0 = frame(k, ex0, ey0), e1 = frame(k + 1, ex1, ey1);
                    add(e0, product(e0, kd), ex0, ey0);
                    add(e1, fma(e1, kd, e1), ex1, ey1);
                    kd += 2.0;
                }
                if (k < K) {
                    double ex0, ey0;
                    const double e0 = frame(k, ex0, ey0);
                    add(e0, product(e0, kd), ex0, ey0);
                }
            } else {
                // sum i = s0, s1, ax, ay, kx, ky in lane i: the products of two columns
                static_assert(L >= 8, "a lane for every sum");
                FunnelChunk &ch = chunk[threadIdx.x / L];
                const int i = min(sub, 5);
                const double *m1 = ch.col[i == 1 || i >= 4 ? 1 : 0], *m2 = ch.col[i < 2 ? 4 : 2 + (i & 1)];
                double sum = 0.0;
                for (int c0 = 0; c0 < K; c0 += FCH) {
#pragma unroll
                    for (int u = 0; u < FCH / L; ++u) {
                        const int q = sub + L * u;
                        double ex = 0.0, ey = 0.0, e = 0.0;
                        if (c0 + q < K) e = frame(c0 + q, ex, ey);   // past the end: adds zeros
                        ch.col[0][q] = e;
                        ch.col[1][q] = product(e, kd + (double)(L * u));
                        ch.col[2][q] = ex;
                        ch.col[3][q] = ey;
                    }
                    kd += FCH;
                    group_sync();
#pragma unroll
                    for (int q = 0; q < FCH; ++q) sum = fma(m1[q], m2[q], sum);
                    group_sync();
                }
                const int lane0 = (threadIdx.x & 63) / L * L;
                auto take = [&](int which) { return __shfl(sum, lane0 + which, 64); };
                s0 = take(0);
                s1 = take(1);
                ax = take(2);
                ay = take(3);
                kx = take(4);
                ky = take(5);
            }
            ax *= 2.0;
            ay *= 2.0;
            kx *= 2.0;
            ky *= 2.0;
            // no weights where exp_neg would hide it: a position that is not finite (or so far
            // that the exponent overflows), a path with a frame that is not a number
            if (!(a > -INFINITY) || path_nan) s0 = NAN;
            const double kbar = s1 / s0;
            sv = 1.0 - kbar / M;
            wv = tube_w(a, s0, P.wscale);
            const double gsx = (P.lambda / M) * (kx - kbar * ax) / s0, gsy = (P.lambda / M) * (ky - kbar * ay) / s0;
            const double lw = P.lambda * P.wscale;
            const double gwx = lw * ax / s0, gwy = lw * ay / s0;
            sm = fmin(sm, sv);
            wm = fmin(wm, wv);
            const double ds = sv - sm, dw = wv - wm;
            bx = -P.k_s * ds * gsx - P.k_w * dw * gwx;
            by = -P.k_s * ds * gsy - P.k_w * dw * gwy;
            eb = 0.5 * P.k_s * ds * ds + 0.5 * P.k_w * dw * dw;
        }
        T += D * (bx * bx + by * by);
        uint32_t ctr[4] = {0u, (uint32_t)(first_id + t), (uint32_t)(step0 + n), (uint32_t)((step0 + n) >> 32)};
        philox4x32_10(ctr, P.seed_lo, P.seed_hi);
        const double rad = sqrt(-2.0 * log(unit_open_d(ctr[0])));
        double sn, cs;
        sincos(6.283185307179586476925286766559 * unit_open_d(ctr[1]), &sn, &cs);
        x += D * (fx + bx) + amp * rad * cs;
        y += D * (fy + by) + amp * rad * sn;
    }
    if (!writes) return;
    xy[t] = make_double2(x, y);
    c[CV_Z] = z;
    c[CV_ZM] = zm;
    c[CV_EB] = eb;
    c[CV_S] = sv;
    c[CV_W] = wv;
    c[CV_SM] = sm;
    c[CV_WM] = wm;
    c[CV_T] = T;
}

// Lanes per trajectory under the tube ratchets: as long as the lanes give a SIMD
// (256 CUs x 4) no more than one or two wavefronts, and the mean path is long
// enough for the exchange through LDS, which costs a chunk of FCH frames however
// few there are.  us for 50 steps with 1 / 8 / 16 lanes:
//   frames        4096 trajectories    8192                 16384
//     2              75 /  90 /  87      74 /  93 / 132       75 / 137 / 236
//     5              88 /  90 /  87      87 /  92 / 132       87 / 135 / 236
//     7             101 /  90 /  87      99 /  92 / 132       99 / 134 / 236
//     9             108 /  97 /  87     107 / 100 / 132      106 / 144 / 236
//    20             161 / 119 / 105     159 / 119 / 156      159 / 174 / 272
//    24             180 / 119 / 105     178 / 120 / 156      178 / 174 / 272
//    51             317 / 169 / 143     319 / 170 / 204      317 / 242 / 361
//   128             688 / 274 / 203     690 / 275 / 292      691 / 391 / 527
// Above 16384 a lane each (51 frames, 20000 trajectories: 319 / 322 / 434).
static int funnel_lanes(int n_traj, int K) {
    if (n_traj <= 4096 && K >= 5) return 16;
    if (n_traj <= 8192 && K >= 7) return 8;
    if (n_traj <= 16384 && K >= 24) return 8;
    return 1;
}

hipError_t launch_funnel_steps(const FunnelK &P, int n_traj, int first_id, double2 *xy, double *cv, int64_t n_steps,
                               uint64_t step0, int record_every, double2 *frames, int K, const double2 *mp,
                               hipStream_t st) {
    const int lanes = P.bias_mode == 1 ? funnel_lanes(n_traj, K) : 1;
    const dim3 grid((unsigned)(((int64_t)n_traj * lanes + 255) / 256)), block(256);
#define SCPS_FUNNEL(BIAS, L)                                                                                   \
    hipLaunchKernelGGL((k_funnel_steps<BIAS, L>), grid, block, 0, st, P, n_traj, first_id, xy, cv, n_steps, step0, \
                       record_every, frames, K, mp)
    if (P.bias_mode != 1) {
        SCPS_FUNNEL(0, 1);
    } else {
        switch (lanes) {
        case 1: SCPS_FUNNEL(1, 1); break;
        case 8: SCPS_FUNNEL(1, 8); break;
        default: SCPS_FUNNEL(1, 16); break;
        }
    }
#undef SCPS_FUNNEL
    return hipGetLastError();
}

// The mean path: frame f averaged over the listed trajectories, one
// workgroup per frame, a fixed-order float64 sum.
__global__ __launch_bounds__(256) void k_funnel_mean(int n_traj, const double2 *__restrict__ frames,
                                                     const int *__restrict__ list, int n_list,
                                                     double2 *__restrict__ out) {
    __shared__ double sx[256], sy[256];
    const int f = blockIdx.x, tid = threadIdx.x;
    double ax = 0.0, ay = 0.0;
    for (int q = tid; q < n_list; q += 256) {
        const double2 p = frames[(int64_t)f * n_traj + list[q]];
        ax += p.x;
        ay += p.y;
    }
    sx[tid] = ax;
    sy[tid] = ay;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) {
            sx[tid] += sx[tid + h];
            sy[tid] += sy[tid + h];
        }
        __syncthreads();
    }
    if (tid == 0) out[f] = make_double2(sx[0] / n_list, sy[0] / n_list);
}

hipError_t launch_funnel_mean(int n_traj, int n_frames, const double2 *frames, const int *list, int n_list,
                              double2 *out, hipStream_t st) {
    hipLaunchKernelGGL(k_funnel_mean, dim3(n_frames), dim3(256), 0, st, n_traj, frames, list, n_list, out);
    return hipGetLastError();
}

}  // namespace scps
