// HIP kernels for gfx950: reference contact maps and the SCPS tube-variable
// passes on matrix cores.
//
// Contact maps are stored per system as float32 tiles of 64 x 64 contact
// pairs in the diagonal-major layout of the stepping kernels: element [s][l]
// of tile (I, J) is the pair (64 I + l, 64 J + ((l + s) mod 64)) of the
// contact set's internal order.  A stack of K frame maps is tile-major,
// [tile][K][4096]; the SCPS passes read a pair-major copy [tile][4096][K4]
// (K4 = K rounded up to a multiple of 4, zero-padded).
//
// Reference maps, eq (avCij) of Orioli, a Beccara, Faccioli
// (arXiv:1705.02180): R_k(i, j) is the mean over the successful paths of the
// contact function C at frame k, with C(q) = (1 + q + q^2) / (1 + q + q^2 +
// q^3 + q^4), q = (r/r0)^2.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "scps_device.h"
#include "scps_internal.h"

namespace scps {

// ---------------------------------------------------------------------------
// reference maps
// ---------------------------------------------------------------------------
__device__ __forceinline__ double contact_f64(double r2, double r0, double r_cut) {
    if (r_cut > 0.0 && r2 > r_cut * r_cut) return 0.0;
    const double q = r2 / (r0 * r0);
    const double q2 = q * q;
    const double num = 1.0 + q + q2;
    return num / (num + q2 * (q + q2));
}

__device__ __forceinline__ int64_t packed_index(int nc, int a, int b) {
    return (int64_t)a * nc - (int64_t)a * (a + 1) / 2 + (b - a - 1);
}

// One workgroup of 256 threads per contact tile pair; thread (w, l) fills
// rows k = w, w+4, ... of the diagonal-major layout element [k][l] =
// R(64I + l, 64J + ((l + k) mod 64)).  Internal contact positions equal the
// positions in contact_idx, so tiles and packed maps share indices.
__global__ void k_native_map(int n, int nc, int ncb, const int *__restrict__ perm, const double *__restrict__ xyz,
                             double r0, double r_cut, float *__restrict__ tiles, double *__restrict__ packed) {
    int I, J;
    tile_decode(blockIdx.x, ncb, I, J);
    const int l = threadIdx.x & 63;
    const int a = I * 64 + l;
    float *t = tiles + (int64_t)blockIdx.x * 4096;
    for (int k = threadIdx.x >> 6; k < 64; k += 4) {
        const int b = J * 64 + ((l + k) & 63);
        double C = 0.0;
        if (a < nc && b < nc && a != b) {
            const int oa = perm[a], ob = perm[b];
            const double dx = xyz[oa] - xyz[ob];
            const double dy = xyz[n + oa] - xyz[n + ob];
            const double dz = xyz[2 * n + oa] - xyz[2 * n + ob];
            C = contact_f64(dx * dx + dy * dy + dz * dz, r0, r_cut);
            if (packed && a < b) packed[packed_index(nc, a, b)] = C;
        }
        t[k * 64 + l] = (float)C;
    }
}

hipError_t launch_native_map(int n, int n_pad, int nc, int ncb, const int *perm_dev, const double *xyz_dev,
                             double r0, double r_cut, float *tiles, double *packed, hipStream_t st) {
    (void)n_pad;
    const int nt = ncb * (ncb + 1) / 2;
    if (nt == 0) return hipSuccess;
    hipLaunchKernelGGL(k_native_map, dim3(nt), dim3(256), 0, st, n, nc, ncb, perm_dev, xyz_dev, r0, r_cut, tiles,
                       packed);
    return hipGetLastError();
}

__global__ void k_pack_to_tiles(int nc, int ncb, int ntile, const double *__restrict__ packed,
                                float *__restrict__ tiles) {
    const int tile = blockIdx.x;
    const int map = blockIdx.y;
    int I, J;
    tile_decode(tile, ncb, I, J);
    const int64_t P = (int64_t)nc * (nc - 1) / 2;
    const double *pm = packed + (int64_t)map * P;
    float *t = tiles + ((int64_t)tile * gridDim.y + map) * 4096;   // [tile][map][4096]
    const int l = threadIdx.x & 63;
    const int a = I * 64 + l;
    for (int k = threadIdx.x >> 6; k < 64; k += 4) {
        const int b = J * 64 + ((l + k) & 63);
        float v = 0.f;
        if (a < nc && b < nc && a != b) v = (float)pm[a < b ? packed_index(nc, a, b) : packed_index(nc, b, a)];
        t[k * 64 + l] = v;
    }
}

hipError_t launch_pack_to_tiles(int n_maps, int nc, int ncb, const double *packed, float *tiles, hipStream_t st) {
    const int nt = ncb * (ncb + 1) / 2;
    if (nt == 0 || n_maps == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_to_tiles, dim3(nt, n_maps), dim3(256), 0, st, nc, ncb, nt, packed, tiles);
    return hipGetLastError();
}

// sum_i v_i^2 in two fixed-order phases: SUMSQ_BLOCKS workgroups each reduce
// a contiguous chunk into part[], then one workgroup adds the partials.
constexpr int SUMSQ_BLOCKS = 256;
__global__ void k_sum_squares(int64_t m, const double *__restrict__ v, double *__restrict__ part,
                              double *__restrict__ out) {
    __shared__ double red[4];
    const int64_t chunk = (m + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < m ? lo + chunk : m;
    double s = 0.0;
    for (int64_t e = lo + threadIdx.x; e < hi; e += blockDim.x) s += v[e] * v[e];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void k_sum_parts(int n, const double *__restrict__ part, double *__restrict__ out) {
    __shared__ double red[4];
    double s = 0.0;
    for (int e = threadIdx.x; e < n; e += blockDim.x) s += part[e];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *out = red[0] + red[1] + red[2] + red[3];
}

int sum_squares_scratch() { return SUMSQ_BLOCKS; }

hipError_t launch_sum_squares(int64_t m, const double *v, double *part, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_squares, dim3(SUMSQ_BLOCKS), dim3(256), 0, st, m, v, part, out);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, st, SUMSQ_BLOCKS, part, out);
    return hipGetLastError();
}

// The sum over the packed contact pairs a < b with |perm[a] - perm[b]| >
// min_sep of v^2: one workgroup per row a into part[a], then the rows in
// order.  perm[a] is the chain index of contact position a.
__global__ void k_sum_squares_sep(int nc, int min_sep, const int *__restrict__ perm, const double *__restrict__ v,
                                  double *__restrict__ part) {
    __shared__ double red[4];
    const int a = blockIdx.x;
    const int oa = perm[a];
    const double *row = v + (packed_index(nc, a, a + 1) - (a + 1));   // row[b] = v(a, b) for b > a
    double s = 0.0;
    for (int b = a + 1 + threadIdx.x; b < nc; b += blockDim.x)
        if (abs(oa - perm[b]) > min_sep) s += row[b] * row[b];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[a] = red[0] + red[1] + red[2] + red[3];
}

hipError_t launch_sum_squares_sep(int nc, int min_sep, const int *perm, const double *v, double *part, double *out,
                                  hipStream_t st) {
    if (nc < 2) {
        hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, st, 0, part, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_sum_squares_sep, dim3(nc), dim3(256), 0, st, nc, min_sep, perm, v, part);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(256), 0, st, nc, part, out);
    return hipGetLastError();
}

// num / den in float64 from the hardware reciprocal estimate (about 24 bits):
// one Newton step r <- r (2 - den r) doubles them, and the residual correction
// of c = num r is exact to another doubling, so the quotient is correctly
// rounded but for rare ties; a second Newton step changed nothing.  den >= 1
// here, so no scaling or special cases are needed.
__device__ __forceinline__ double quotient_f64(double num, double den) {
    double r = __builtin_amdgcn_rcp(den);
    r = fma(r, fma(-den, r, 1.0), r);
    const double c = num * r;
    return fma(fma(-den, c, num), r, c);
}

// eq (avCij): mean over successful paths of C(X_p(t_k)), float64 sums.
// Grid (contact tile pair, frame).  Thread (w, l) owns, for the 8 partners
// j = (l + 8 w + kk) mod 64 of block J, the pairs with particles l and l + 32
// mod 64 of block I: rows 8 w + kk and 8 w + kk + 32 of the diagonal-major
// tile, so that one read of j's position serves two pairs.  The positions of
// blocks I and J of UPDREF_PATHS paths at a time are staged in LDS as float64
// components (the differences of float32 coordinates are then exact).
//
// Bound by float64 VALU issue.  The contact values of UPDREF_QUAD paths of a
// pair are added over their common denominator, n1/d1 + n2/d2 = (n1 d2 +
// n2 d1)/(d1 d2) twice over, so that one reciprocal and its refinement serve
// four values: 11 + 19/4 float64 instructions a value where a quotient each
// takes 11 + 10.  The error of the mean went down with the number of roundings
// (1.06e-16 rms relative to 80-bit arithmetic against 1.62e-16 at distances
// around 5 A, 1.25e-16 against 1.72e-16 at 20 A).  d ~ q^4, so four factors
// stay finite below q = 1e18: a batch of paths with a coordinate beyond
// 3e8 r0, or a NaN, takes its values one by one instead.  32 paths x 51 frames
// x 6000 particles: 16.5 ms (22.2 ms with a quotient each and one row of
// pairs a lane).
constexpr int UPDREF_PATHS = 8, UPDREF_QUAD = 4;
static_assert(UPDREF_PATHS % UPDREF_QUAD == 0, "whole groups but for the last batch");
template <bool CUT>
__global__ __launch_bounds__(256) void k_update_reference(int n, int nc, int ncb, const int *__restrict__ perm,
                                                          const float *__restrict__ frames, int n_paths,
                                                          const int *__restrict__ succ, int n_succ,
                                                          double inv_r0sq, double r_cut2, float far_limit,
                                                          float *__restrict__ tiles, double *__restrict__ packed) {
    constexpr int PB = UPDREF_PATHS;
    __shared__ double pos[2][3][PB][64];   // [block I/J][component][path][particle]
    const int tile = blockIdx.x, f = blockIdx.y;
    int I, J;
    tile_decode(tile, ncb, I, J);
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
    const int li[2] = {l, (l + 32) & 63};
    double sum[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 8; ++k) sum[h][k] = 0.0;
    // numerator and denominator of C at a difference vector (beyond the cutoff 0 / 1)
    auto ratio = [&](double dx, double dy, double dz, double &num, double &den) {
        const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
        const double q = r2 * inv_r0sq;
        const double q2 = q * q;
        const double t = q + q2;
        num = t + 1.0;
        den = fma(q2, t, num);
        if (CUT && r2 > r_cut2) {
            num = 0.0;
            den = 1.0;
        }
    };
    // the values of paths pp .. pp + N - 1, over one denominator
    auto add_paths = [&](auto count, int pp) {
        constexpr int N = decltype(count)::value;
        double a[2][N][3];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int c = 0; c < 3; ++c) a[h][u][c] = pos[0][c][pp + u][li[h]];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int j = (l + w * 8 + kk) & 63;
            double num[2][N], den[2][N];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const double bx = pos[1][0][pp + u][j], by = pos[1][1][pp + u][j], bz = pos[1][2][pp + u][j];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    ratio(a[h][u][0] - bx, a[h][u][1] - by, a[h][u][2] - bz, num[h][u], den[h][u]);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int s = 1; s < N; s *= 2)
#pragma unroll
                    for (int u = 0; u + s < N; u += 2 * s) {
                        num[h][u] = fma(num[h][u], den[h][u + s], num[h][u + s] * den[h][u]);
                        den[h][u] *= den[h][u + s];
                    }
                sum[h][kk] += quotient_f64(num[h][0], den[h][0]);
            }
        }
    };
    for (int s0 = 0; s0 < n_succ; s0 += PB) {
        const int np = min(PB, n_succ - s0);
        bool far = false;
        __syncthreads();
        for (int e = tid; e < 2 * PB * 64; e += 256) {
            const int which = e / (PB * 64), pp = (e >> 6) % PB, c = (which ? J : I) * 64 + (e & 63);
            float x = 0.f, y = 0.f, z = 0.f;
            if (pp < np && c < nc) {
                const float *X = frames + ((int64_t)f * n_paths + succ[s0 + pp]) * 3 * (int64_t)n;
                const int o = perm[c];
                x = X[o];
                y = X[n + o];
                z = X[2 * n + o];
                far = far || !(fabsf(x) <= far_limit && fabsf(y) <= far_limit && fabsf(z) <= far_limit);
            }
            pos[which][0][pp][e & 63] = x;
            pos[which][1][pp][e & 63] = y;
            pos[which][2][pp][e & 63] = z;
        }
        int pp = 0;
        if (!__syncthreads_or(far)) {
            for (; pp + UPDREF_QUAD <= np; pp += UPDREF_QUAD) add_paths(std::integral_constant<int, UPDREF_QUAD>{}, pp);
            if (pp + 2 <= np) {
                add_paths(std::integral_constant<int, 2>{}, pp);
                pp += 2;
            }
        }
        for (; pp < np; ++pp) add_paths(std::integral_constant<int, 1>{}, pp);
    }
    float *t = tiles + ((int64_t)tile * gridDim.y + f) * 4096;     // [tile][frame][4096]
    const int64_t P = (int64_t)nc * (nc - 1) / 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int k = w * 8 + kk + 32 * h;
            const int a = I * 64 + li[h], b = J * 64 + ((li[h] + k) & 63);
            double mean = 0.0;
            if (a < nc && b < nc && a != b) {
                mean = sum[h][kk] / (double)n_succ;
                if (packed && a < b) packed[(int64_t)f * P + packed_index(nc, a, b)] = mean;
            }
            t[k * 64 + li[h]] = (float)mean;
        }
}

hipError_t launch_update_reference(int n, int n_pad, int nc, int ncb, const int *perm_dev, const float *frames,
                                   int n_paths, int n_frames, const int *succ_idx, int n_succ, double r0,
                                   double r_cut, float *tiles, double *packed, hipStream_t st) {
    (void)n_pad;
    const int nt = ncb * (ncb + 1) / 2;
    if (nt == 0) return hipSuccess;
    const double inv_r0sq = 1.0 / (r0 * r0);
    const float far_limit = (float)std::min(3.0e8 * r0, 3.0e38);   // NaN and inf coordinates compare as beyond it
    if (r_cut > 0.0)
        hipLaunchKernelGGL(k_update_reference<true>, dim3(nt, n_frames), dim3(256), 0, st, n, nc, ncb, perm_dev,
                           frames, n_paths, succ_idx, n_succ, inv_r0sq, r_cut * r_cut, far_limit, tiles,
                           packed);
    else
        hipLaunchKernelGGL(k_update_reference<false>, dim3(nt, n_frames), dim3(256), 0, st, n, nc, ncb, perm_dev,
                           frames, n_paths, succ_idx, n_succ, inv_r0sq, 0.0, far_limit, tiles, packed);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// SCPS on matrix cores.  The squared distance of replica r to frame k,
// d_k Z0 = sum_p (C_rp - R_kp)^2, splits into sum_p C_rp^2 - 2 X_rk +
// sum_p R_kp^2 with X_rk = sum_p C_rp R_kp: for a group of up to 32 replicas
// of one system that is a dense contraction over the contact pairs p, done
// here with float32 MFMA whose sums are moved into float64 every 64 pairs
// (the three terms are then accurate to float64 rounding of float32-exact
// partial sums, which keeps the cancellation in Q - 2X + R2 harmless).  The
// bias pass needs each replica's effective reference E_rp = sum_k c_rk R_kp, a
// contraction over the frames, also float32 MFMA (the same rounding as a
// float32 dot product).  Both read every stack tile once per group instead of
// once per replica.
// ---------------------------------------------------------------------------
typedef float fvec16 __attribute__((ext_vector_type(16)));


// Unordered contact pair (64 I + l, 64 J + ((l + s) mod 64)) of a tile in the
// diagonal-major layout: in a diagonal tile every pair appears twice; the
// copy at sub-steps 1..31, or at 32 for l < 32, is the one that counts.
__device__ __forceinline__ bool tile_pair_counts(bool diag, int s, int l) {
    return !diag || (s >= 1 && (s < 32 || (s == 32 && l < 32)));
}

// Per contact tile of a map [tile][4096]: the float64 sum of the squared
// entries over the tile's counted pairs (both in the contact set, beyond
// min_seq_sep, each unordered pair once).  One workgroup per tile; thread
// (w, l) takes sub-steps s = w, w + 4, ... of column l.
__global__ __launch_bounds__(256) void k_tile_sumsq(int nc, int ncb, int min_sep, const int *__restrict__ perm,
                                                    const float *__restrict__ tiles, double *__restrict__ out) {
    __shared__ double ws[4];
    const int tile = blockIdx.x;
    int I, J;
    tile_decode(tile, ncb, I, J);
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
    const int a = I * 64 + l;
    const float *t = tiles + (int64_t)tile * 4096;
    double sum = 0.0;
    for (int s = w; s < 64; s += 4) {
        const int b = J * 64 + ((l + s) & 63);
        if (a < nc && b < nc && tile_pair_counts(I == J, s, l) && abs(perm[a] - perm[b]) > min_sep) {
            const double v = t[s * 64 + l];
            sum = fma(v, v, sum);
        }
    }
    sum = wave_sum(sum);
    if (l == 0) ws[w] = sum;
    __syncthreads();
    if (tid == 0) out[tile] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

hipError_t launch_tile_sumsq(int nc, int ncb, int min_sep, const int *perm, const float *tiles, double *out,
                             hipStream_t st) {
    const int nt = ncb * (ncb + 1) / 2;
    if (nt == 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_sumsq, dim3(nt), dim3(256), 0, st, nc, ncb, min_sep, perm, tiles, out);
    return hipGetLastError();
}

// What the SCPS passes need of a new frame stack, in one pass over it: the
// pair-major copy stack_pm[tile][p][k] = stack[tile][k][p] (k < K; zero for
// K <= k < K4), and the frame distances G[j][k] = sum over the counted contact
// pairs (both in the contact set, beyond min_seq_sep, each unordered pair
// once) of (R_jp - R_kp)^2, in float64 from the float32 frames (differences of
// float32 values are exact in float64), the diagonal 0.  part
// (stack_finish_scratch doubles) must be zero on entry.
//
// A work unit is `per` sub-steps of a tile; workgroups stride over the units.
// 64 pairs (32 when K > 64) at a time are staged twice in LDS: as float32 rows
// to be written out pair by pair, and as float64 rows, zero for a pair that
// does not count (so it adds nothing without a branch); the next batch's
// loads are in flight meanwhile.  Frame k = r + N a has residue r mod N and
// digit a < SF_B; thread t holds the SF_B x SF_B frame pairs of the residues
// (r1, r2), r1 <= r2, number t mod n_blocks in registers and takes the pairs
// p = t / n_blocks mod n_slices: 12 values read from LDS feed 36
// subtract-and-FMA pairs (one frame pair per thread and read was bound by LDS
// reads), neighbouring threads read neighbouring residues, and the rows have
// odd lengths, so neither reads nor staging stores meet on a bank (blocks of
// neighbouring frames in rows of even length did, and took twice the time).
// Small stacks take short units (a tile of 10 frames in one workgroup was a
// chain of 64 load-and-wait rounds).
// Bound by float64 VALU issue.  6000 particles, 51 frames: 3.7 ms, 1.6 ms with
// the distances left out (the copy and the distances in a kernel each took 3.1 +
// 7.9 ms); 585 contact particles, 10 frames: 29 us (79 + 940 us).
constexpr int SF_B = 6;
constexpr int SF_COPIES = 64;
constexpr int SF_STAGE = 16;   // 64 pairs x 64 frames or 32 x 128 over 256 threads
static_assert(64 * 64 <= 256 * SF_STAGE && 32 * KMAX <= 256 * SF_STAGE, "a batch fits the staging registers");
size_t stack_finish_scratch(int K) { return (size_t)SF_COPIES * K * (K - 1) / 2; }
struct StackFinishShape {
    int pairs;          // pairs per batch
    int N;              // residues
    int kf, kd;         // row lengths of the float32 and the float64 rows (odd)
    size_t bytes;
};
static StackFinishShape stack_finish_shape(int K) {
    StackFinishShape L;
    L.pairs = K <= 64 ? 64 : 32;
    L.N = (K + SF_B - 1) / SF_B;
    L.kf = K | 1;
    L.kd = (L.N * SF_B) | 1;
    L.bytes = std::max((size_t)L.pairs * (L.kd * sizeof(double) + L.kf * sizeof(float)),
                       (size_t)K * (K - 1) / 2 * sizeof(double));   // also the sums' meeting place
    return L;
}
static_assert(((KMAX + SF_B - 1) / SF_B) * ((KMAX + SF_B - 1) / SF_B + 1) / 2 <= 256, "a thread for every block");

template <int PAIRS>
__global__ __launch_bounds__(256, 3) void k_stack_finish(int nc, int ncb, int K, int min_sep, int n_units, int per,
                                                         int N, int kf, int kd, const int *__restrict__ perm,
                                                         const float *__restrict__ stack,
                                                         float *__restrict__ stack_pm, double *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int pairs = PAIRS, kstep = 256 / PAIRS;
    double *rd = reinterpret_cast<double *>(smem);                    // [pairs][kd]
    float *rf = reinterpret_cast<float *>(rd + (size_t)pairs * kd);   // [pairs][kf]
    const int tid = threadIdx.x;
    const int K4 = stack_pm_width(K);
    const int n_blocks = N * (N + 1) / 2, n_slices = 256 / n_blocks;
    const int slice = tid / n_blocks;
    const bool on = slice < n_slices;
    int r1, r2;
    tile_decode(tid % n_blocks, N, r1, r2);
    double acc[SF_B][SF_B];
#pragma unroll
    for (int a = 0; a < SF_B; ++a)
#pragma unroll
        for (int b = 0; b < SF_B; ++b) acc[a][b] = 0.0;
    for (int e = tid; e < pairs * kd; e += 256) rd[e] = 0.0;   // the columns past K stay zero
    // thread tid stages pair p0 + tid mod pairs of frames tid / pairs, + 256 / pairs, ...:
    // SF_STAGE values at most, loaded a batch ahead into registers
    const int pl = tid & (pairs - 1), kt = tid / pairs;
    const int upt = 64 / per, bpu = per * 64 / pairs;   // units of a tile, batches of a unit
    float ahead[SF_STAGE];
    bool cnt_ahead = false;
    auto load = [&](int u, int q) {
        const int tile = u / upt, p = (u - tile * upt) * per * 64 + q * pairs + pl, l = p & 63, sub = p >> 6;
        int I, J;
        tile_decode(tile, ncb, I, J);
        const int a = I * 64 + l, b = J * 64 + ((l + sub) & 63);
        cnt_ahead = a < nc && b < nc && tile_pair_counts(I == J, sub, l) && abs(perm[a] - perm[b]) > min_sep;
        // (frames past K re-read frame 0: loads without branches)
        const float *src = stack + (int64_t)tile * K * 4096;
#pragma unroll
        for (int s = 0; s < SF_STAGE; ++s) {
            const int k = kt + s * kstep;
            ahead[s] = src[(uint32_t)((k < K ? k : 0) * 4096 + p)];
        }
    };
    // the pair-major rows go out four frames at a time
    const int w4 = K4 >> 2, dp = 256 / w4, dk = 256 - dp * w4;
    int u = blockIdx.x, q = 0;
    if (u < n_units) load(u, 0);
    while (u < n_units) {
        __syncthreads();
#pragma unroll
        for (int s = 0; s < SF_STAGE; ++s) {
            const int k = kt + s * kstep;
            if (k < K) {
                rf[pl * kf + k] = ahead[s];
                rd[pl * kd + k] = cnt_ahead ? (double)ahead[s] : 0.0;
            }
        }
        __syncthreads();
        const int tile = u / upt, p0 = (u - tile * upt) * per * 64 + q * pairs;
        if (++q == bpu) {
            q = 0;
            u += gridDim.x;
        }
        if (u < n_units) load(u, q);
        {
            float4 *out = reinterpret_cast<float4 *>(stack_pm + ((int64_t)tile * 4096 + p0) * K4);
            int po = tid / w4, ko = tid - po * w4;
            while (po < pairs) {
                const float *row = rf + po * kf + 4 * ko;
                const int left = K - 4 * ko;
                out[po * w4 + ko] = make_float4(row[0], left > 1 ? row[1] : 0.f, left > 2 ? row[2] : 0.f,
                                                left > 3 ? row[3] : 0.f);
                po += dp;
                ko += dk;
                if (ko >= w4) {
                    ko -= w4;
                    ++po;
                }
            }
        }
        if (on)
#pragma unroll 1
            for (int p = slice; p < pairs; p += n_slices) {
                const double *row1 = rd + p * kd + r1, *row2 = rd + p * kd + r2;
                double rj[SF_B], rk[SF_B];
#pragma unroll
                for (int a = 0; a < SF_B; ++a) {
                    rj[a] = *row1;
                    rk[a] = *row2;
                    row1 += N;
                    row2 += N;
                }
#pragma unroll
                for (int a = 0; a < SF_B; ++a)
#pragma unroll
                    for (int b = 0; b < SF_B; ++b) {
                        const double d = rj[a] - rk[b];
                        acc[a][b] = fma(d, d, acc[a][b]);
                    }
            }
    }
    // The slices' sums meet in LDS (packed upper triangle; a residue with itself
    // holds every pair twice, of which one counts), then go to one of SF_COPIES
    // sets of partial sums: atomics on one address wait for each other (about
    // 0.4 us each when workgroups of every XCD meet there).
    const int E = K * (K - 1) / 2;
    auto packed = [&](int j, int k) { return j * K - j * (j + 1) / 2 + k - j - 1; };
    __syncthreads();
    for (int e = tid; e < E; e += 256) rd[e] = 0.0;
    __syncthreads();
    if (on) {
#pragma unroll
        for (int a = 0; a < SF_B; ++a)
#pragma unroll
            for (int b = 0; b < SF_B; ++b) {
                const int f1 = r1 + a * N, f2 = r2 + b * N, j = min(f1, f2), k = max(f1, f2);
                if (f1 == f2 || k >= K || (r1 == r2 && a > b)) continue;
                unsafeAtomicAdd(&rd[packed(j, k)], acc[a][b]);
            }
    }
    __syncthreads();
    double *Gp = part + (int64_t)(blockIdx.x % SF_COPIES) * E;
    for (int e = tid; e < E; e += 256) unsafeAtomicAdd(&Gp[e], rd[e]);
}

// G[j][k] = G[k][j] = the sum of the partial sets, in order; the diagonal 0
__global__ void k_gram_sum(int K, const double *__restrict__ part, double *__restrict__ G) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x, j = e / K, k = e - j * K, E = K * (K - 1) / 2;
    if (j >= K || j > k) return;
    double t = 0.0;
    if (j < k) {
        const double *p = part + (j * K - j * (j + 1) / 2 + k - j - 1);
#pragma unroll 8
        for (int c = 0; c < SF_COPIES; ++c) t += p[(int64_t)c * E];
    }
    G[j * K + k] = t;
    G[k * K + j] = t;
}

hipError_t launch_stack_finish(int nc, int ncb, int K, int min_sep, const int *perm, const float *stack,
                               float *stack_pm, double *part, double *G, hipStream_t st) {
    const int nt = ncb * (ncb + 1) / 2;
    if (nt == 0 || K == 0) return hipSuccess;
    if (K > KMAX) return hipErrorInvalidValue;
    const StackFinishShape L = stack_finish_shape(K);
    // the workgroups that are resident at once (256 CUs), each taking at least 8
    // units where there are tiles enough, of one sub-step (64 pairs) at least; no
    // more workgroups than leave each 4 units (their sums are K^2/2 atomics each)
    const int resident = 256 * (int)std::min<size_t>(4, 160 * 1024 / L.bytes);
    int per = 64;
    while (per > 1 && (int64_t)nt * (64 / per) < 8 * resident) per /= 2;
    const int64_t n_units = (int64_t)nt * (64 / per);
    if (n_units > INT32_MAX) return hipErrorInvalidValue;
    const int grid = (int)std::min<int64_t>((n_units + 3) / 4, resident);
    if (L.pairs == 64)
        hipLaunchKernelGGL(k_stack_finish<64>, dim3(grid), dim3(256), L.bytes, st, nc, ncb, K, min_sep, (int)n_units,
                           per, L.N, L.kf, L.kd, perm, stack, stack_pm, part);
    else
        hipLaunchKernelGGL(k_stack_finish<32>, dim3(grid), dim3(256), L.bytes, st, nc, ncb, K, min_sep, (int)n_units,
                           per, L.N, L.kf, L.kd, perm, stack, stack_pm, part);
    hipLaunchKernelGGL(k_gram_sum, dim3((K * K + 63) / 64), dim3(64), 0, st, K, part, G);
    return hipGetLastError();
}

// Contact value of one replica-pair for the MFMA operand (0 when the pair
// does not count).  CUT: test the contact cutoff (a cutoff marks every
// contact tile MASK, so the other tiles need no test).
template <bool CUT>
__device__ __forceinline__ float contact_operand(const KParams &P, const float4 &pi, const float4 &pj, bool ok) {
    float dx, dy, dz;
    const float r2 = pair_r2(pi, pj, dx, dy, dz);
    const float q = r2 * P.inv_r0sq;
    const float q2 = q * q;
    const float t = q + q2;   // num = 1 + t, den = num + q^2 t
    const float num = 1.f + t;
    const float den = fmaf(q2, t, num);
    const bool inside = CUT ? (!P.has_cut | (r2 <= P.r_cut2)) : true;
    return (ok & inside) ? num * frcp(den) : 0.f;
}

// Pass 1, around each replica's reference frame j_r (see tube_sums): with
// u_rp = C_rp - R_{j_r}p, X[r][k] += sum_p u_rp R_kp and Q[r] += sum_p u_rp^2
// over the contact pairs of each work item (group of replicas, tile);
// workgroups stride over the items and flush their sums when the group
// changes and at the end.
//
// 16x16x4 float32 MFMAs: NR row groups of 16 replicas (2, or 1 where no group
// has more than 16) against NB blocks of 16 frames (NB the smallest of 1 .. 6
// and 8 that holds the stack), so the matrix and the pair work go with the
// replicas and the frames.  (32x32x2 blocks, 32 replicas x 64 frames a pass
// over the tile, ran 128 frames for 65, in two passes that each took the
// contact values again, and 32 replicas for 8.)  The pairs of a tile are taken
// row by row: wavefront w takes rows i = w, w + NW, ... of block I and, per row,
// 16 steps of 4 pairs (i, 4m + (l >> 4)); lane l evaluates u of that pair for
// replicas 16 g + (l & 15) (A operands, one per row group) with particle i's
// positions in registers (loaded a row ahead) and particle j's from the block-J
// positions in LDS, and loads its frames of the pair (min(NB, 4) (l & 15) ...,
// and from 64 on (NB - 4) (l & 15) ...) with one or two vector loads
// DIST_AHEAD steps ahead of their use.  A wavefront writes the frames of its
// next 4 pairs to LDS, where each lane finds R_j of its replicas (LDS
// operations of a wavefront keep their order, so one buffer is enough; cross-
// lane moves of the same took one per row group and vector component).  A
// diagonal tile counts the pairs j > i.  The float32 accumulators hold one row
// (64 pairs per element) and are added after every row into the workgroup's
// float64 sums xl in LDS; u^2 goes to float64 term by term (a Q that carries
// float32 partial sums moves w by more than the ratchets near the appendix
// limit allow).  Element v of lane l in row group g, block b is replica slot
// 16 g + 4 (l >> 4) + v, frame dist_frame(b, l & 15).
// Addressing: pair (i, j) sits at s * 64 + i in the tile, s = (j - i) mod 64.
// Lanes of slots without a replica compute finite values from zero positions
// that reach only their own output rows and Q sums, which the flush drops;
// MASK tiles (diagonal ones among them) zero u of pairs that do not count.
// Bound by MFMA and VALU issue, which do not overlap on a SIMD here (about 35
// VALU instructions a step of 4 pairs and 32 replicas beside its 8 MFMAs; 42
// with the 32x32x2 form).  us a pass, 32x32x2 form -> now: 32 replicas x 6000
// particles x 51 frames 1117 -> 1041 (in the map update), 20 x 1501 x 72 232 ->
// 111, 15 x 1700 x 70 242 -> 106, 30 x 2100 x 50 213 -> 165, 32 x 3000 x 12 319
// -> 157.
constexpr int DIST_AHEAD = 4;   // 2: 1.07 against 1.00 ms at 6000 particles; 8 spills (1.45 ms)
constexpr int DIST_NW = 8;   // wavefronts per workgroup, sharing block J and the float64 sums

template <int NR, int NB>
struct DistLds {
    static constexpr int SCW = 16 * NB + 4;      // frames of a pair, rows 16-byte aligned
    float4 posj[64][16 * NR];                    // block J of every replica slot
    double xl[16 * NR][16 * NB];                 // float64 sums of the current group, columns 16 b + (l & 15)
    float sc[DIST_NW][4][SCW];                   // each wavefront's next 4 pairs, by frame
    double qs[16 * NR];
    int orgj[64];
    int rep[16 * NR];
    int jref[16 * NR];                           // reference frame of every replica slot
};
template <int NR, int NB>
constexpr int dist_resident() { return sizeof(DistLds<NR, NB>) <= 80 * 1024 ? 2 : 1; }   // workgroups per CU

// frame of column c (0 .. 15) of block b
template <int NB>
__device__ __forceinline__ int dist_frame(int b, int c) {
    constexpr int W0 = NB < 4 ? NB : 4, W1 = NB - W0;
    return b < W0 ? W0 * c + b : 64 + W1 * c + (b - W0);
}

template <bool MASK, int NR, int NB>
__device__ __forceinline__ void scps_dist_tile(const KParams &P, const SysDesc &S, const int nrep,
                                               const ScpsItem &it, DistLds<NR, NB> &L, const float4 *__restrict__ xs,
                                               const RepDesc *__restrict__ reps, const int lane, const int wave,
                                               const int r0, const int r1, double q[NR]) {
    constexpr int W0 = NB < 4 ? NB : 4, W1 = NB - W0, D = DIST_AHEAD;
    static_assert(16 % D == 0, "the ring keeps its phase over a row");
    typedef float vec0 __attribute__((ext_vector_type(W0), aligned(W0 == 3 ? 4 : 4 * W0)));
    typedef float vec1 __attribute__((ext_vector_type(W1 > 0 ? W1 : 1), aligned(W1 > 0 ? 4 * W1 : 4)));
    typedef float acc4 __attribute__((ext_vector_type(4)));
    const int I = it.IJ >> 16, J = it.IJ & 0xFFFF;
    const bool diag = I == J;
    const int K4 = stack_pm_width(S.K);
    const int col = lane & 15, quad = lane >> 4;
    // global (not flat) loads from a uniform base with 32-bit lane offsets: flat
    // loads would also count against the LDS wait counter and drain the ring
    typedef const __attribute__((address_space(1))) char *gbytes;
    const gbytes tile_base = (gbytes)(S.stack_pm + (int64_t)it.tile * 4096 * K4);
    const uint32_t row_bytes = 4u * (uint32_t)K4;   // one pair of the tile, all frames
    // lanes past the stack width re-read the pair's first frames (a lane across its
    // end reads on into the next pair); the flush drops their columns
    const uint32_t f0 = W0 * col < K4 ? 4u * (uint32_t)(W0 * col) : 0u;
    const uint32_t f1 = W1 > 0 && 64 + W1 * col < K4 ? 4u * (uint32_t)(64 + W1 * col) : 0u;
    const float4 *xr[NR];
    int jr[NR];
    bool rep[NR];
#pragma unroll
    for (int g = 0; g < NR; ++g) {
        const int slot = 16 * g + col;
        rep[g] = slot < nrep;
        xr[g] = xs + 2 * reps[L.rep[slot]].poff + I * 128;
        jr[g] = L.jref[slot];
    }
    struct Frames {
        vec0 a;
        vec1 b;
    };
    // step m of row i (a row past the last is never consumed: clamped to 63)
    auto load = [&](int i_, int m_) {
        const int ic = i_ < 64 ? i_ : 63;
        const int b = (4 * m_ - ic) & 63;   // uniform; s = (b + quad) mod 64
        const uint32_t lo = __umul24((uint32_t)(b + quad) & 63u, 64u * row_bytes);
        const gbytes base = tile_base + (uint32_t)ic * row_bytes;
        Frames r;
        r.a = *(const __attribute__((address_space(1))) vec0 *)(base + (lo + f0));
        if constexpr (W1 > 0) r.b = *(const __attribute__((address_space(1))) vec1 *)(base + (lo + f1));
        return r;
    };
    auto *sc = L.sc[wave];
    auto publish = [&](const Frames &r) {
        *reinterpret_cast<vec0 *>(&sc[quad][W0 * col]) = r.a;
        if constexpr (W1 > 0) *reinterpret_cast<vec1 *>(&sc[quad][64 + W1 * col]) = r.b;
    };
    Frames ring[D];
#pragma unroll
    for (int u = 0; u < D; ++u) ring[u] = load(r0 + wave, u);
    float rj[NR];
    publish(ring[0]);
#pragma unroll
    for (int g = 0; g < NR; ++g) rj[g] = sc[quad][jr[g]];
    typedef float vec3 __attribute__((ext_vector_type(3), aligned(16)));
    vec3 pn[NR];   // the next row's particle i
    auto particle = [&](int g, int i_) {
        typedef const __attribute__((address_space(1))) vec3 *gvec3;
        return *(gvec3)(xr[g] + min(i_, 63));
    };
#pragma unroll
    for (int g = 0; g < NR; ++g) pn[g] = particle(g, r0 + wave);
#pragma unroll 1
    for (int i = r0 + wave; i < r1; i += DIST_NW) {
        float4 pi[NR];
#pragma unroll
        for (int g = 0; g < NR; ++g) {
            pi[g] = make_float4(rep[g] ? pn[g].x : 0.f, rep[g] ? pn[g].y : 0.f, rep[g] ? pn[g].z : 0.f, 0.f);
            pn[g] = particle(g, i + DIST_NW);
        }
        const int oi = MASK ? S.perm[I * 64 + i] : 0;
        const bool icon = I * 64 + i < S.nc;
        acc4 acc[NR][NB];
#pragma unroll
        for (int g = 0; g < NR; ++g)
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[g][b] = acc4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int mg = 0; mg < 16 / D; ++mg) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int m = D * mg + u;
                const Frames f = ring[u];
                float rc[NR];
#pragma unroll
                for (int g = 0; g < NR; ++g) rc[g] = rj[g];
                publish(ring[(u + 1) % D]);   // the next step's frames (u = D - 1: loaded D - 1 steps ago)
#pragma unroll
                for (int g = 0; g < NR; ++g) rj[g] = sc[quad][jr[g]];
                ring[u] = m + D < 16 ? load(i, m + D) : load(i + DIST_NW, m + D - 16);
                const int jl = 4 * m + quad;
                bool ok0 = true;
                if constexpr (MASK)
                    ok0 = icon & (J * 64 + jl < S.nc) & (abs(oi - L.orgj[jl]) > P.min_sep) & (!diag | (jl > i));
#pragma unroll
                for (int g = 0; g < NR; ++g) {
                    const float4 pj = L.posj[jl][16 * g + col];
                    float c;
                    if constexpr (MASK) {
                        const bool ok = ok0 & rep[g];
                        const float cv = contact_operand<true>(P, pi[g], pj, ok);
                        c = ok ? cv - rc[g] : 0.f;   // u = C - R_j of a counted pair
                    } else {
                        c = contact_operand<false>(P, pi[g], pj, true) - rc[g];
                    }
                    q[g] = fma((double)c, (double)c, q[g]);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float bv = b < W0 ? f.a[b < W0 ? b : 0] : f.b[b < W0 ? 0 : b - W0];
                        acc[g][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(c, bv, acc[g][b], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int g = 0; g < NR; ++g)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) atomicAdd(&L.xl[16 * g + 4 * quad + v][16 * b + col], (double)acc[g][b][v]);
    }
}

// Work unit t: rows [r0, r0 + 64 / nsplit) of item t / nsplit.  The sums are
// flushed when the group changes.
template <int NR, int NB>
__global__ __launch_bounds__(64 * DIST_NW)
__attribute__((amdgpu_waves_per_eu(dist_resident<NR, NB>() * DIST_NW / 4, dist_resident<NR, NB>() * DIST_NW / 4)))
void k_scps_dist(const KParams P, const SysDesc *__restrict__ sysd, const RepDesc *__restrict__ reps,
                 const ScpsGroup *__restrict__ groups, const ScpsItem *__restrict__ items, const int n_items,
                 const int nsplit, const int *__restrict__ jref, const float4 *__restrict__ xs,
                 double *__restrict__ X, double *__restrict__ Q, const int sets, const int kmax,
                 const int stack_sys) {
    __shared__ __align__(16) DistLds<NR, NB> L;
    constexpr int WG = 64 * DIST_NW, SLOTS = 16 * NR, COLS = 16 * NB;
    // the wavefront index is uniform: in a scalar register, the row and step
    // arithmetic of the tile loop (and its load bases) stay scalar
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < SLOTS * COLS; e += WG) L.xl[e / COLS][e % COLS] = 0.0;
    if (tid < SLOTS) L.qs[tid] = 0.0;
    double q[NR];
#pragma unroll
    for (int g = 0; g < NR; ++g) q[g] = 0.0;
    int cur = -1, nrep = 0;
    SysDesc S;
    const int n_units = n_items * nsplit, rows = 64 / nsplit;
    const int set = blockIdx.x & (sets - 1);
    for (int t = blockIdx.x;; t += gridDim.x) {
        const bool more = t < n_units;
        const int u = t / nsplit, r0 = (t - u * nsplit) * rows;
        const ScpsItem it = more ? items[u] : ScpsItem{-1, 0, 0, 0};
        const bool change = it.group != cur;
        if (cur >= 0 && change) {
            // flush the group's sums to one set of the replicas' float64 totals
#pragma unroll
            for (int g = 0; g < NR; ++g) {
                unsafeAtomicAdd(&L.qs[16 * g + (lane & 15)], q[g]);
                q[g] = 0.0;
            }
            __syncthreads();
            for (int e = tid; e < SLOTS * COLS; e += WG) {
                const int slot = e / COLS, c = e % COLS, k = dist_frame<NB>(c >> 4, c & 15);
                if (slot < nrep && k < S.K)
                    unsafeAtomicAdd(&X[(int64_t)(L.rep[slot] * sets + set) * kmax + k], L.xl[slot][c]);
                L.xl[slot][c] = 0.0;
            }
            if (tid < SLOTS) {
                if (tid < nrep) unsafeAtomicAdd(&Q[L.rep[tid] * sets + set], L.qs[tid]);
                L.qs[tid] = 0.0;
            }
        }
        if (!more) break;
        __syncthreads();
        if (change) {
            cur = it.group;
            const ScpsGroup *gp = groups + cur;
            nrep = gp->nrep;
            S = sysd[gp->sys];
            if (stack_sys >= 0) {   // another system's stack (same chain and contact set)
                S.stack_pm = sysd[stack_sys].stack_pm;
                S.K = sysd[stack_sys].K;
            }
            if (tid < SLOTS) {
                L.rep[tid] = tid < nrep ? gp->rep[tid] : gp->rep[0];
                L.jref[tid] = tid < nrep ? ref_frame(jref, gp->rep[tid], S.K) : 0;
            }
            __syncthreads();
        }
        // stage block J of every replica of the group
        const int J = it.IJ & 0xFFFF;
        for (int e = tid; e < 64 * SLOTS; e += WG) {
            const int pl = e / SLOTS, slot = e % SLOTS;
            float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
            if (slot < nrep) p = xs[2 * reps[L.rep[slot]].poff + J * 128 + pl];
            L.posj[pl][slot] = p;
        }
        if (tid < 64) L.orgj[tid] = S.perm[J * 64 + tid];
        __syncthreads();
        if ((it.flags & TILE_MASK) || (it.IJ >> 16) == J)
            scps_dist_tile<true, NR, NB>(P, S, nrep, it, L, xs, reps, lane, wave, r0, r0 + rows, q);
        else
            scps_dist_tile<false, NR, NB>(P, S, nrep, it, L, xs, reps, lane, wave, r0, r0 + rows, q);
    }
}

// Pass 2 operand of the two-pass form (exec mode 2; the default forms it inside
// k_scps_bias): E[eoff_r + tile * 4096 + p] = sum_k c_rk R_kp for every
// pair p of each work item's tile and replica r of its group (coef holds
// c_rk).  Wavefront w takes chunks of 32 EFF_NB pairs w, w+4, ...; a chunk is
// EFF_NB 32-pair MFMA blocks interleaved so that block b holds pairs
// EFF_NB j + b: lane l reads pairs EFF_NB (l & 31) .. +EFF_NB-1 of frame
// 2 kk + (l >> 5) with one load (component b is its B operand of block b)
// and supplies c of replica l & 31 for that frame (A operand, 32x32x2
// float32 MFMA).  Result element v of lane l in block b is replica
// 8 (v >> 2) + 4 (l >> 5) + (v & 3), pair EFF_NB (l & 31) + b: the blocks give
// one EFF_NB-wide store per replica.
#ifndef SCPS_EFF_BLOCKS
#define SCPS_EFF_BLOCKS 4
#endif
#ifndef SCPS_EFF_WPE
#define SCPS_EFF_WPE (SCPS_EFF_BLOCKS == 4 ? 2 : 3)
#endif
#ifndef SCPS_EFF_NT
#define SCPS_EFF_NT 3   // bit 0: non-temporal stores of E, bit 1: non-temporal loads of the stack
#endif                  // (each is used once per step; measured 1.7 % faster per SCPS step with both)
constexpr int EFF_NB = SCPS_EFF_BLOCKS;
static_assert(EFF_NB == 2 || EFF_NB == 4, "chunks of 2 or 4 MFMA blocks");
typedef float effvec __attribute__((ext_vector_type(EFF_NB)));

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SCPS_EFF_WPE, SCPS_EFF_WPE))) void k_scps_eff(
    const SysDesc *__restrict__ sysd, const RepDesc *__restrict__ reps, const ScpsGroup *__restrict__ groups,
    const ScpsItem *__restrict__ items, const int n_items, const float *__restrict__ coef, const int kmax,
    float *__restrict__ E) {
    __shared__ int64_t sh_eoff[SCPS_GROUP];   // -1 for an empty slot
    constexpr int CH = 32 * EFF_NB;            // pairs per chunk
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slot = lane & 31, half = lane >> 5;
    int cur = -1;
    SysDesc S;
    float creg[KMAX / 2];
    for (int t = blockIdx.x; t < n_items; t += gridDim.x) {
        const ScpsItem it = items[t];
        if (it.group != cur) {
            cur = it.group;
            const ScpsGroup *gp = groups + cur;
            const int nrep = gp->nrep;
            S = sysd[gp->sys];
            const int myrep = slot < nrep ? gp->rep[slot] : 0;
#pragma unroll
            for (int kk = 0; kk < KMAX / 2; ++kk) {
                const int k = 2 * kk + half;
                creg[kk] = (slot < nrep && k < S.K) ? coef[(int64_t)myrep * kmax + k] : 0.f;
            }
            __syncthreads();
            if (tid < SCPS_GROUP) sh_eoff[tid] = tid < nrep ? reps[gp->rep[tid]].eoff : -1;
            __syncthreads();
        }
        const int K = S.K;
        const float *Rt = S.stack + (int64_t)it.tile * K * 4096;
#pragma unroll 1
        for (int ch = wave; ch < 4096 / CH; ch += 4) {
            const int p = ch * CH + EFF_NB * slot;
            fvec16 acc[EFF_NB];
#pragma unroll
            for (int bl = 0; bl < EFF_NB; ++bl)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[bl][v] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KMAX / 2; ++kk) {
                if (2 * kk < K) {
                    const int k = 2 * kk + half;
                    effvec b;
                    if (k < K) {
#if SCPS_EFF_NT & 2
                        b = __builtin_nontemporal_load(reinterpret_cast<const effvec *>(Rt + k * 4096 + p));
#else
                        b = *reinterpret_cast<const effvec *>(Rt + k * 4096 + p);
#endif
                    } else
#pragma unroll
                        for (int bl = 0; bl < EFF_NB; ++bl) b[bl] = 0.f;
#pragma unroll
                    for (int bl = 0; bl < EFF_NB; ++bl)
                        acc[bl] = __builtin_amdgcn_mfma_f32_32x32x2f32(creg[kk], b[bl], acc[bl], 0, 0, 0);
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t eo = sh_eoff[8 * (v >> 2) + 4 * half + (v & 3)];
                if (eo >= 0) {
                    effvec o;
#pragma unroll
                    for (int bl = 0; bl < EFF_NB; ++bl) o[bl] = acc[bl][v];
#if SCPS_EFF_NT & 1
                    __builtin_nontemporal_store(o, reinterpret_cast<effvec *>(E + eo + (int64_t)it.tile * 4096 + p));
#else
                    *reinterpret_cast<effvec *>(E + eo + (int64_t)it.tile * 4096 + p) = o;
#endif
                }
            }
        }
    }
}

// Pass 2 fused with the bias forces: the effective references never leave
// the chip.  A workgroup takes one work item (group of replicas, contact tile
// pair I, J) at a time, with blocks I and J of every replica slot in LDS, and
// walks the tile's sub-steps (lane i of block I meets particle (i + k) mod 64
// of block J) in chunks of BIAS_CH.  Its wavefronts split into a producer
// and a consumer half that work on neighbouring chunks at the same time
// (double-buffered E in LDS, one barrier per chunk):
//  - matrix wavefront w forms E[slot][i] = sum_f c_f,slot R_f,(i, k) of
//    sub-step k = chunk + w with 32x32x2 float32 MFMAs (rows: the pairs
//    i = 2 row + b of block b, read with one 8-byte load per lane from frames
//    2 kk + (l >> 5); columns: the slots, B operand c of slot l & 31 as in
//    k_scps_eff), stores it, and issues the stack loads of its next sub-step;
//  - pair wavefront p takes slots p, p + BIAS_NPW, ... with lane = i, as the
//    tile kernels do: the contact gradient term (csum C - E) C' of the bias
//    goes to the lane's i-side partials and to j-side partials that rotate
//    with the j partner (DPP), over every sub-step of the tile.
// The partials of each slot go to the replica's float64 bias accumulators
// (components 3..5) once per item, 64 consecutive particles per atomic
// instruction.  A diagonal tile takes sub-steps 1..32 (lanes i < 32 at
// k = 32), so each pair is met once; MASK tiles evaluate the contact
// predicate and the cutoff per pair.  Nonbonded forces and bonds are not
// computed here.
constexpr int BIAS_WG = 768;
constexpr int BIAS_NMW = 4;                      // matrix wavefronts = sub-steps per chunk
constexpr int BIAS_NPW = BIAS_WG / 64 - BIAS_NMW;  // pair wavefronts
constexpr int BIAS_CH = BIAS_NMW;
constexpr int BIAS_SPW = SCPS_GROUP / BIAS_NPW;  // replica slots per pair wavefront

struct BiasLds {
    float4 pos[2][SCPS_GROUP][64];        // blocks I, J: [slot][particle]
    float E[2][BIAS_CH][SCPS_GROUP][65];  // two chunks: [sub-step][slot][i], padded for the matrix stores
    float c[KMAX / 2][64];                // B operand: c of slot l & 31, frame 2 kk + (l >> 5)
    float cs[SCPS_GROUP];
    int org[2][64];
    int rep[SCPS_GROUP];                  // -1: empty slot
    int64_t poff[SCPS_GROUP];
};
static_assert(BIAS_WG % 64 == 0 && BIAS_NPW > 0 && SCPS_GROUP % BIAS_NPW == 0,
              "every pair wavefront takes the same number of replica slots");
static_assert(sizeof(BiasLds) <= 160 * 1024, "the fused bias pass keeps one workgroup's state in LDS");

typedef float bias_f2 __attribute__((ext_vector_type(2)));

// Frames 2 (f0 + kk) + half of pairs 2 slot, 2 slot + 1 of sub-step k: a
// uniform tile base and a 32-bit lane offset per load.
template <int KKN>
__device__ __forceinline__ void bias_loads(const float *tile_base, const int k, const int f0, const int K,
                                           const int slot, const int half, bias_f2 r[KKN]) {
    typedef const __attribute__((address_space(1))) bias_f2 *gptr;
    const gptr gb = (gptr)tile_base;
    const int o = (half * 4096 + k * 64 + 2 * slot) >> 1;   // in float pairs
#pragma unroll
    for (int kk = 0; kk < KKN; ++kk) {
        r[kk] = bias_f2{0.f, 0.f};
        if (2 * (f0 + kk) + half < K) r[kk] = __builtin_nontemporal_load(gb + (o + (f0 + kk) * 4096));
    }
}

// KKN frame pairs per MFMA chain, NH chains per sub-step (2 KKN NH >= K;
// frames beyond K have zero coefficients and are not loaded), fixed at
// compile time so that a chain has no branches and its loads are issued
// together.  With NH = 2 (stacks of more than 64 frames) the loads of the
// next half are issued after the MFMAs of the current one.
template <int KKN, int NH>
__device__ __forceinline__ void scps_bias_produce(const SysDesc &S, const ScpsItem &it, const int lane,
                                                  const int wave, const int kb, const int ke, BiasLds &L) {
    const int nch = (ke - kb + BIAS_CH - 1) / BIAS_CH;
    // ---- E of sub-step kb + BIAS_CH st + wave, chunk st -> buffer st & 1
    const int K = S.K;
    const int slot = lane & 31, half = lane >> 5;
    const float *Rt = S.stack + (int64_t)it.tile * K * 4096;   // uniform
    bias_f2 r[KKN];
    if (kb + wave < ke) bias_loads<KKN>(Rt, kb + wave, 0, K, slot, half, r);
#pragma unroll 1
    for (int st = 0; st <= nch; ++st) {
        const int k = kb + BIAS_CH * st + wave;
        if (st < nch && k < ke) {
            fvec16 acc[2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
            // one chain per KKN frame pairs; a second chain's loads go out after
            // the first chain's MFMAs, into the same registers
#pragma unroll
            for (int h = 0; h < NH; ++h) {
#pragma unroll
                for (int kk = 0; kk < KKN; ++kk) {
                    const float c = L.c[KKN * h + kk][lane];
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(r[kk].x, c, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(r[kk].y, c, acc[1], 0, 0, 0);
                }
                if (h + 1 < NH) bias_loads<KKN>(Rt, k, KKN * (h + 1), K, slot, half, r);
            }
            float(*E)[65] = L.E[st & 1][wave];
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int b = 0; b < 2; ++b) E[slot][16 * (v >> 2) + 8 * half + 2 * (v & 3) + b] = acc[b][v];
            if (k + BIAS_CH < ke) bias_loads<KKN>(Rt, k + BIAS_CH, 0, K, slot, half, r);
        }
        __syncthreads();
    }
}

// The same for a group of at most 16 replicas, with 16x16x4 float32 MFMAs
// (half the matrix time): rows pairs 4 row + b of block b, read with one
// 16-byte load per lane from frame 4 kk + (l >> 4); columns the slots l & 15.
// Element v of lane l in block b is pair 16 (l >> 4) + 4 v + b.
typedef float bias_f4 __attribute__((ext_vector_type(4)));
template <int KKN>
__device__ __forceinline__ void bias_loads16(const float *tile_base, const int k, const int f0, const int K,
                                             const int lane, bias_f4 r[KKN]) {
    typedef const __attribute__((address_space(1))) bias_f4 *gptr;
    const gptr gb = (gptr)tile_base;
    const int o = (lane >> 4) * 1024 + k * 16 + (lane & 15);   // in groups of four floats
#pragma unroll
    for (int kk = 0; kk < KKN; ++kk) {
        r[kk] = bias_f4{0.f, 0.f, 0.f, 0.f};
        if (4 * (f0 + kk) + (lane >> 4) < K) r[kk] = __builtin_nontemporal_load(gb + (o + (f0 + kk) * 4096));
    }
}

template <int KKN, int NH>
__device__ __forceinline__ void scps_bias_produce16(const SysDesc &S, const ScpsItem &it, const int lane,
                                                    const int wave, const int kb, const int ke, BiasLds &L) {
    const int nch = (ke - kb + BIAS_CH - 1) / BIAS_CH;
    const int K = S.K;
    const int slot = lane & 15, quad = lane >> 4;
    const float *Rt = S.stack + (int64_t)it.tile * K * 4096;   // uniform
    // c of frame 4 kk + quad: row 2 kk + quad / 2 of L.c, its lower or upper half
    const float *cl = &L.c[quad >> 1][(quad & 1) * 32 + slot];
    bias_f4 r[KKN];
    if (kb + wave < ke) bias_loads16<KKN>(Rt, kb + wave, 0, K, lane, r);
#pragma unroll 1
    for (int st = 0; st <= nch; ++st) {
        const int k = kb + BIAS_CH * st + wave;
        if (st < nch && k < ke) {
            bias_f4 acc[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[b] = bias_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < NH; ++h) {
#pragma unroll
                for (int kk = 0; kk < KKN; ++kk) {
                    const float c = cl[128 * (KKN * h + kk)];
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[kk][b], c, acc[b], 0, 0, 0);
                }
                if (h + 1 < NH) bias_loads16<KKN>(Rt, k, KKN * (h + 1), K, lane, r);
            }
            float(*E)[65] = L.E[st & 1][wave];
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int b = 0; b < 4; ++b) E[slot][16 * quad + 4 * v + b] = acc[b][v];
            if (k + BIAS_CH < ke) bias_loads16<KKN>(Rt, k + BIAS_CH, 0, K, lane, r);
        }
        __syncthreads();
    }
}

// Pair wavefront pw: chunk st - 1 from buffer (st - 1) & 1, for its first SPW
// slots (the wavefronts of a group of fewer than SCPS_GROUP replicas have fewer).
template <bool MASK, int SPW>
__device__ __forceinline__ void scps_bias_consume(const KParams &P, const SysDesc &S, const ScpsItem &it,
                                                  const int lane, const int pw, const int kb, const int ke,
                                                  BiasLds &L, float fi[][3], float fj[][3]) {
    const int I = it.IJ >> 16, J = it.IJ & 0xFFFF;
    const bool diag = it.flags & TILE_DIAG;
    const int nch = (ke - kb + BIAS_CH - 1) / BIAS_CH;
    const int nc = S.nc, min_sep = P.min_sep;
    const bool has_cut = P.has_cut;
    const float inv_r0sq = P.inv_r0sq, r_cut2 = P.r_cut2;
    const float cp0 = P.cp[0], cp1 = P.cp[1], cp2 = P.cp[2], cp3 = P.cp[3];
    const bool icon = I * 64 + lane < nc;
    const int oi = L.org[0][lane];
    constexpr int SA = SPW > 0 ? SPW : 1;
    float px[SA], py[SA], pz[SA], csm[SA];
#pragma unroll
    for (int m = 0; m < SPW; ++m) {
        const float4 p = L.pos[0][pw + BIAS_NPW * m][lane];
        px[m] = p.x;
        py[m] = p.y;
        pz[m] = p.z;
        csm[m] = L.cs[pw + BIAS_NPW * m];
    }
#pragma unroll 1
    for (int st = 0; st <= nch; ++st) {
        if (st > 0) {
            const int c0 = kb + BIAS_CH * (st - 1), nk = min(BIAS_CH, ke - c0);
            float(*E)[SCPS_GROUP][65] = L.E[(st - 1) & 1];
            // sub-steps in order (the j-side partials rotate once per sub-step);
            // the slots of one sub-step are independent, so they run interleaved
#pragma unroll
            for (int u = 0; u < BIAS_CH; ++u) {
                if (u < nk) {
                    const int k = c0 + u, jl = (lane + k) & 63;
                    const bool con0 = !diag | (k != 32) | (lane < 32);
                    bool conm = true;
                    if constexpr (MASK) conm = icon & (J * 64 + jl < nc) & (abs(oi - L.org[1][jl]) > min_sep);
#pragma unroll
                    for (int m = 0; m < SPW; ++m) {
                        const int sl = pw + BIAS_NPW * m;
                        const float4 pj = L.pos[1][sl][jl];
                        const float dx = px[m] - pj.x, dy = py[m] - pj.y, dz = pz[m] - pj.z;
                        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                        bool inside = true;
                        if constexpr (MASK) inside = !has_cut | (r2 <= r_cut2);
                        const float q = r2 * inv_r0sq;
                        const float q2 = q * q;
                        const float t = q + q2;
                        const float num = 1.f + t;
                        const float den = fmaf(q2, t, num);
                        const float inv_den = inside ? frcp(den) : 0.f;
                        float diff = fmaf(csm[m], num * inv_den, -E[u][sl][lane]);
                        diff = (con0 & conm) ? diff : 0.f;
                        const float poly = fmaf(q, fmaf(q, fmaf(q, cp0, cp1), cp2), cp3);
                        const float g = (diff * (q2 * inv_den)) * (poly * inv_den);
                        fi[m][0] = fmaf(g, dx, fi[m][0]);
                        fi[m][1] = fmaf(g, dy, fi[m][1]);
                        fi[m][2] = fmaf(g, dz, fi[m][2]);
                        fj[m][0] = rot1(fmaf(-g, dx, fj[m][0]));
                        fj[m][1] = rot1(fmaf(-g, dy, fj[m][1]));
                        fj[m][2] = rot1(fmaf(-g, dz, fj[m][2]));
                    }
                }
            }
        }
        __syncthreads();
    }
}

// BIG: stacks of 65 .. KMAX frames, HALF: no group of more than 16 replicas, in
// kernels of their own so that each keeps its register allocation.  A sub-step's
// matrix work is cut to the smallest of a few frame counts that holds the stack and
// to 16 or 32 replicas, and a pair wavefront's to its replicas.  The counts are steps
// of 8 to 32 frames, with one at 52 and one at 72, where the paths of the protocol
// lie (10^4 steps with a frame every 200; about 72 frames to a path): each more is
// another form of the producer to compile and to hold in the instruction cache.  us
// a pass as 32 replicas x 64 or 128 frames -> so cut -> with the workgroups per tile
// of launch_scps_bias: 20 replicas x 1501 particles, 72 frames 230 -> 168 -> 142; 8 x
// 2500 (1252 in contact), 33 frames 71 -> 33; 15 x 1700, 70 frames 241 -> 122 -> 108.
// A step of 32 x 1500 particles: 72 frames 311 us, 73 320, 96 344, 97 399, 128 402.
template <bool BIG, bool HALF>
__device__ __forceinline__ void scps_bias_produce_any(const SysDesc &S, const ScpsItem &it, const int lane,
                                                      const int wave, const int kb, const int ke, BiasLds &L) {
    // KKN frame pairs, or half as many groups of four frames
#define SCPS_PRODUCE(KKN, NH)                                                     \
    do {                                                                           \
        if constexpr (HALF)                                                        \
            scps_bias_produce16<KKN / 2, NH>(S, it, lane, wave, kb, ke, L);        \
        else                                                                       \
            scps_bias_produce<KKN, NH>(S, it, lane, wave, kb, ke, L);              \
    } while (0)
    static_assert(KMAX / 2 == 64, "frame pairs of the largest stack");
    if constexpr (BIG) {
        if (S.K <= 72)
            SCPS_PRODUCE(18, 2);
        else if (S.K <= 96)
            SCPS_PRODUCE(24, 2);
        else
            SCPS_PRODUCE(32, 2);
    } else {
        if (S.K <= 16)
            SCPS_PRODUCE(8, 1);
        else if (S.K <= 32)
            SCPS_PRODUCE(16, 1);
        else if (S.K <= 40)
            SCPS_PRODUCE(20, 1);
        else if (S.K <= 52)
            SCPS_PRODUCE(26, 1);
        else
            SCPS_PRODUCE(32, 1);
    }
#undef SCPS_PRODUCE
}

template <bool MASK>
__device__ __forceinline__ void scps_bias_consume_any(const KParams &P, const SysDesc &S, const ScpsItem &it,
                                                      const int lane, const int pw, const int n_slots, const int kb,
                                                      const int ke, BiasLds &L, float fi[][3], float fj[][3]) {
#define SCPS_CONSUME(SPW) scps_bias_consume<MASK, SPW>(P, S, it, lane, pw, kb, ke, L, fi, fj)
    static_assert(BIAS_SPW == 4, "one case per number of slots");
    switch (n_slots) {
    case 0: SCPS_CONSUME(0); break;
    case 1: SCPS_CONSUME(1); break;
    case 2: SCPS_CONSUME(2); break;
    case 3: SCPS_CONSUME(3); break;
    default: SCPS_CONSUME(4); break;
    }
#undef SCPS_CONSUME
}

template <bool BIG, bool HALF>
__global__ __launch_bounds__(BIAS_WG) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_scps_bias(
    const KParams P, const SysDesc *__restrict__ sysd, const RepDesc *__restrict__ reps,
    const ScpsGroup *__restrict__ groups, const ScpsItem *__restrict__ items, const int n_items,
    const float4 *__restrict__ xs, const float *__restrict__ coef, const double *__restrict__ csum, const int kmax,
    const int ksplit, double *__restrict__ acc) {
    __shared__ BiasLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int cur = -1, nrep = 0;
    SysDesc S;
    // work unit t: a range of the sub-steps of item t / ksplit (ksplit > 1
    // when there are too few items to fill the chip), in whole chunks
    for (int t = blockIdx.x; t < n_items * ksplit; t += gridDim.x) {
        const ScpsItem it = items[t / ksplit];
        const bool tdiag = it.flags & TILE_DIAG;
        const int kb0 = tdiag ? 1 : 0, ke0 = tdiag ? 33 : 64;   // a diagonal tile meets each pair by sub-step 32
        const int per = ((ke0 - kb0 + ksplit - 1) / ksplit + BIAS_CH - 1) / BIAS_CH * BIAS_CH;
        const int kb = min(ke0, kb0 + (t % ksplit) * per), ke = min(ke0, kb + per);
        __syncthreads();   // the previous item's positions are no longer read
        if (it.group != cur) {
            cur = it.group;
            const ScpsGroup *gp = groups + cur;
            nrep = gp->nrep;
            S = sysd[gp->sys];
            for (int e = tid; e < KMAX / 2 * 64; e += BIAS_WG) {
                const int kk = e >> 6, l = e & 63, sl = l & 31, k = 2 * kk + (l >> 5);
                L.c[kk][l] = (sl < nrep && k < S.K) ? coef[(int64_t)gp->rep[sl] * kmax + k] : 0.f;
            }
            if (tid < SCPS_GROUP) {
                const bool live = tid < nrep;
                L.rep[tid] = live ? gp->rep[tid] : -1;
                L.poff[tid] = live ? reps[gp->rep[tid]].poff : 0;
                L.cs[tid] = live ? (float)csum[gp->rep[tid]] : 0.f;
            }
            __syncthreads();
        }
        const int I = it.IJ >> 16, J = it.IJ & 0xFFFF;
        for (int e = tid; e < 2 * SCPS_GROUP * 64; e += BIAS_WG) {
            const int pl = e & 63, sl = (e >> 6) & 31, side = e >> 11;
            float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
            if (L.rep[sl] >= 0) p = xs[2 * L.poff[sl] + (side ? J : I) * 128 + pl];
            L.pos[side][sl][pl] = p;
        }
        if (tid < 128) L.org[tid >> 6][tid & 63] = S.perm[((tid >> 6) ? J : I) * 64 + (tid & 63)];
        __syncthreads();
        float fi[BIAS_SPW][3], fj[BIAS_SPW][3];
#pragma unroll
        for (int m = 0; m < BIAS_SPW; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c) fi[m][c] = fj[m][c] = 0.f;
        if (wave < BIAS_NMW) {
            scps_bias_produce_any<BIG, HALF>(S, it, lane, wave, kb, ke, L);
        } else {
            const int pw = wave - BIAS_NMW, n_slots = (nrep - pw + BIAS_NPW - 1) / BIAS_NPW;   // <= 0: none
            if (it.flags & TILE_MASK)
                scps_bias_consume_any<true>(P, S, it, lane, pw, max(n_slots, 0), kb, ke, L, fi, fj);
            else
                scps_bias_consume_any<false>(P, S, it, lane, pw, max(n_slots, 0), kb, ke, L, fi, fj);
        }
        if (wave < BIAS_NMW || kb == ke) continue;
        // after sub-steps kb .. ke-1 lane l holds the j-side partials of particle (l + ke) mod 64
        const int jo = J * 64 + ((lane + ke) & 63);
        const int n_pad = S.n_pad;
#pragma unroll
        for (int m = 0; m < BIAS_SPW; ++m) {
            const int sl = (wave - BIAS_NMW) + BIAS_NPW * m;
            if (L.rep[sl] >= 0) {
                double *ar = acc + 6 * L.poff[sl];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    unsafeAtomicAdd(&ar[(3 + c) * n_pad + I * 64 + lane], (double)fi[m][c]);
                    unsafeAtomicAdd(&ar[(3 + c) * n_pad + jo], (double)fj[m][c]);
                }
            }
        }
    }
}

// Each tile's rows are split over up to 16 workgroups where that shortens the
// pass: the CU with the most units takes them one after the other, each 8 / k
// rows of a wavefront and the staging and first loads of a unit (about 0.7 rows);
// where it holds two at a time (all but stacks of more than 96 frames with more
// than 16 replicas) the two together take 0.8 of that.  16 ranges leave half the
// wavefronts without a row and are still the best at 15 tiles.  us a step for 1 / 2 /
// 4 / 8 / 16 workgroups a tile, 51 frames (32 x 560: 45 tiles, and so on):
//   45 tiles   132 /  99 /  84 /  82 /  88      136 tiles  186 / 173 / 162 / 159 / 166
//   66         153 / 120 / 116 / 114 / 118      240        200 / 192 / 197 / 206 / 227
//   120        158 / 127 / 122 / 124 / 135      300        298 / 272 / 257 / 268 / 287
int scps_dist_splits(int n_items, int resident) {
    int ns = 1;
    double best = 1e30;
    for (int k = 1; k <= 16; k *= 2) {
        const double units = std::ceil(n_items * (double)k / 256.0);   // of the fullest CU
        const double t = units * (8.0 / k + 0.7) * (units > 1.0 && resident > 1 ? 0.8 : 1.0);
        if (t < 0.97 * best) {
            best = t;
            ns = k;
        }
    }
    return ns;
}

template <int NR, int NB>
static void launch_scps_dist_as(const KParams &P, const SysDesc *sysd, const RepDesc *reps, const ScpsGroup *groups,
                                const ScpsItem *items, int n_items, const int *jref, const float4 *xs, double *X,
                                double *Q, int sets, int kmax, int stack_sys, hipStream_t st) {
    const int ns = scps_dist_splits(n_items, dist_resident<NR, NB>());
    const int grid = std::min(n_items * ns, 256 * dist_resident<NR, NB>());
    hipLaunchKernelGGL((k_scps_dist<NR, NB>), dim3(grid), dim3(64 * DIST_NW), 0, st, P, sysd, reps, groups, items,
                       n_items, ns, jref, xs, X, Q, sets, kmax, stack_sys);
}

hipError_t launch_scps_dist(const KParams &P, const SysDesc *sysd, const RepDesc *reps, const ScpsGroup *groups,
                            const ScpsItem *items, int n_items, int max_frames, int max_group, const int *jref,
                            const float4 *xs, double *X, double *Q, int sets, int kmax, int stack_sys,
                            hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    if (sets != 1 && sets != XQ_SETS) return hipErrorInvalidValue;
    if (max_frames < 1 || max_frames > KMAX || max_frames > kmax) return hipErrorInvalidValue;
#define SCPS_DIST(NB)                                                                                           \
    do {                                                                                                        \
        const auto launch = max_group <= 16 ? launch_scps_dist_as<1, NB> : launch_scps_dist_as<2, NB>;          \
        launch(P, sysd, reps, groups, items, n_items, jref, xs, X, Q, sets, kmax, stack_sys, st);               \
    } while (0)
    switch ((max_frames + 15) / 16) {
    case 1: SCPS_DIST(1); break;
    case 2: SCPS_DIST(2); break;
    case 3: SCPS_DIST(3); break;
    case 4: SCPS_DIST(4); break;
    case 5: SCPS_DIST(5); break;
    case 6: SCPS_DIST(6); break;
    default: SCPS_DIST(8); break;
    }
#undef SCPS_DIST
    return hipGetLastError();
}

// Tube variables of every replica against the frame stack of system
// stack_sys (-1: its own system's), from the sums k_scps_dist left in X and
// Q around the reference frames jref_in, which are cleared for the next
// pass.  s, w: nullable [R]; sigma: nullable [R], set to weight (1 - s) when
// first, else incremented by it (the mean of 1 - s over several stacks is
// the progress coordinate sigma); jref_out: nullable [R], each replica's
// frame of largest weight.
template <int SETS>
__global__ void k_tube_eval(double lam, double wscale, const int *__restrict__ jref_in, int *__restrict__ jref_out,
                            const SysDesc *__restrict__ sysd, const RepDesc *__restrict__ reps, int kmax,
                            int stack_sys, double *__restrict__ X, double *__restrict__ Q, double *__restrict__ s,
                            double *__restrict__ w, double *__restrict__ sigma, double weight, int first) {
    const int r = blockIdx.x, lane = threadIdx.x;
    const SysDesc S = sysd[stack_sys >= 0 ? stack_sys : reps[r].sys];
    const int K = S.K;
    const int j = ref_frame(jref_in, r, K);
    double yk[2];
    const double q = take_xq<SETS>(lane, K, kmax, r, X, Q, yk);
    const TubeSums ts = tube_sums(lane, K, q, yk, j, S.G + (int64_t)j * K, S.Z0, lam);
    const double sv = 1.0 - (ts.s1 / ts.s0) / (double)(K - 1);
    const double wv = tube_w(ts.a, ts.s0, wscale);
    if (lane == 0) {
        if (s) s[r] = sv;
        if (w) w[r] = wv;
        if (sigma) sigma[r] = (first ? 0.0 : sigma[r]) + weight * (1.0 - sv);
        if (jref_out) jref_out[r] = ts.kmax;
    }
}

hipError_t launch_tube_eval(double lam, double wscale, const int *jref_in, int *jref_out, const SysDesc *sysd,
                            const RepDesc *reps, int R, int kmax, int stack_sys, double *X, double *Q, int sets,
                            double *s, double *w, double *sigma, double weight, int first, hipStream_t st) {
    const auto kernel = sets == 1 ? k_tube_eval<1> : k_tube_eval<XQ_SETS>;
    hipLaunchKernelGGL(kernel, dim3(R), dim3(64), 0, st, lam, wscale, jref_in, jref_out, sysd, reps, kmax, stack_sys,
                       X, Q, s, w, sigma, weight, first);
    return hipGetLastError();
}

hipError_t launch_scps_eff(const SysDesc *sysd, const RepDesc *reps, const ScpsGroup *groups, const ScpsItem *items,
                           int n_items, const float *coef, int kmax, float *E, hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    const int grid = n_items < 1024 ? n_items : 1024;
    hipLaunchKernelGGL(k_scps_eff, dim3(grid), dim3(256), 0, st, sysd, reps, groups, items, n_items, coef, kmax,
                       E);
    return hipGetLastError();
}

hipError_t launch_scps_bias(const KParams &P, const SysDesc *sysd, const RepDesc *reps, const ScpsGroup *groups,
                            const ScpsItem *items, int n_items, int max_frames, int max_group, const float4 *xs,
                            const float *coef, const double *csum, int kmax, double *acc, hipStream_t st) {
    if (n_items == 0) return hipSuccess;
    if (max_frames < 1 || max_frames > KMAX || max_frames > kmax) return hipErrorInvalidValue;
    // one workgroup per compute unit (LDS).  Each tile's sub-steps are split over
    // up to 8 workgroups (whole chunks) where that shortens the pass: rounds of
    // 256 units, each 64 / ks sub-steps and the staging and first chunk of a unit
    // (about 7 sub-steps more).  15 tiles take 8 ranges, and 300 tiles, whose
    // second round of 44 left the chip idle, 4 (20 replicas x 72
    // frames: 168 -> 142 us).
    int ks = 1;
    double best = 1e30;
    for (int k = 1; k <= 8; k *= 2) {
        const double t = std::ceil(n_items * (double)k / 256.0) * (64.0 / k + 7.0);
        if (t < 0.97 * best) {
            best = t;
            ks = k;
        }
    }
    const int grid = std::min(n_items * ks, 256);
#define SCPS_LAUNCH(BIG, HALF)                                                                                  \
    hipLaunchKernelGGL((k_scps_bias<BIG, HALF>), dim3(grid), dim3(BIAS_WG), 0, st, P, sysd, reps, groups, items, \
                       n_items, xs, coef, csum, kmax, ks, acc)
    if (max_frames > 64) {
        if (max_group <= 16)
            SCPS_LAUNCH(true, true);
        else
            SCPS_LAUNCH(true, false);
    } else if (max_group <= 16) {
        SCPS_LAUNCH(false, true);
    } else {
        SCPS_LAUNCH(false, false);
    }
#undef SCPS_LAUNCH
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// convergence measure between iterations
// ---------------------------------------------------------------------------
// Occupancy of an nx x ny grid of square cells (side cell, lower corner
// (x0, y0), half-open) by 2-D points xy [n][2]: occ[cy * nx + cx] = 1 for
// every cell holding a point; points outside the grid are ignored.  Cell
// indices are taken in float64.  occ must be zero on entry.
__global__ void k_occupancy(const float *__restrict__ xy, int64_t n, double x0, double y0, double cell, int nx, int ny,
                            int *__restrict__ occ) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const double u = floor(((double)xy[2 * e] - x0) / cell), v = floor(((double)xy[2 * e + 1] - y0) / cell);
        if (u >= 0.0 && u < (double)nx && v >= 0.0 && v < (double)ny) occ[(int)v * nx + (int)u] = 1;
    }
}

// Counts of occupied cells in a, in b, and in both (one workgroup).
__global__ __launch_bounds__(256) void k_occupancy_overlap(const int *__restrict__ a, const int *__restrict__ b,
                                                           int m, long long *__restrict__ out) {
    __shared__ long long sh[3][256];
    long long na = 0, nb = 0, nab = 0;
    for (int e = threadIdx.x; e < m; e += 256) {
        na += a[e];
        nb += b[e];
        nab += a[e] & b[e];
    }
    sh[0][threadIdx.x] = na;
    sh[1][threadIdx.x] = nb;
    sh[2][threadIdx.x] = nab;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h)
            for (int q = 0; q < 3; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x < 3) out[threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void k_fill_int(int *__restrict__ v, int m) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < m; e += gridDim.x * blockDim.x) v[e] = 0;
}

// Scratch of the convergence measure for callers that cannot allocate: the
// four counts (long long) first, then the two occupancy grids, in a file-scope
// device array each GPU holds until the process ends.  Host code must not
// pass `scratch` itself to a kernel (in host code the name is a stand-in, not
// a device address): path_scratch() returns this GPU's address of it.
static __device__ __align__(256) int scratch[8 + 2 * PATH_NOALLOC_MAX_CELLS];

hipError_t path_scratch(int **occ, long long **counts) {
    static std::mutex lock;
    static void *addr[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(lock);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // with this device current: its own copy
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *counts = reinterpret_cast<long long *>(addr[dev]);
    *occ = reinterpret_cast<int *>(addr[dev]) + 8;
    return hipSuccess;
}

hipError_t launch_path_occupancy(const float *xy_a, int64_t n_a, const float *xy_b, int64_t n_b, double x0,
                                 double y0, double cell, int nx, int ny, int *occ, long long *counts,
                                 hipStream_t st) {
    const int m = nx * ny;
    hipLaunchKernelGGL(k_fill_int, dim3((2 * m + 255) / 256), dim3(256), 0, st, occ, 2 * m);
    if (n_a > 0)
        hipLaunchKernelGGL(k_occupancy, dim3((unsigned)std::min<int64_t>((n_a + 255) / 256, 4096)), dim3(256), 0, st,
                           xy_a, n_a, x0, y0, cell, nx, ny, occ);
    if (n_b > 0)
        hipLaunchKernelGGL(k_occupancy, dim3((unsigned)std::min<int64_t>((n_b + 255) / 256, 4096)), dim3(256), 0, st,
                           xy_b, n_b, x0, y0, cell, nx, ny, occ + m);
    hipLaunchKernelGGL(k_occupancy_overlap, dim3(1), dim3(256), 0, st, occ, occ + m, m, counts);
    return hipGetLastError();
}

}  // namespace scps
