// Direct Gaussian-kernel products (a7), the plain O(n_t n_s) path:
//   out_i = sum_j v_j exp(-|x_i - y_j|^2 / eta)      (Sec. 5, eq. fastsum-sum)
//
// Small products (direct_small_targets) run in one launch whose blocks split the sources among their
// sixteen wavefronts.  Above, both precisions split a job's sources into dsplit equal ranges, so
// that products with few targets still spread over the chip: an item is a group of targets and
// one range; with dsplit > 1 it writes its partial sums to the job's partial buffer, and
// direct_reduce_kernel adds the ranges in order.
//
// FP64 variant: one target per lane, a block's four wavefronts summing quarters of a
// source range in ascending source order, the quarters (and ranges) then added in order
// (details at direct_fp64_kernel).
//
// Mixed variant: FP32 transcendental with FP64 accumulation.  With c = log2(e) / eta and
// coordinates taken relative to the point cloud's centre,
//   exp(-|x - y|^2 / eta) = exp2(a_x + x.y' + a_y),  a_x = -c|x|^2, a_y = -c|y|^2, y' = 2 c y,
// and x.y' + a_y is a contraction of length four, one MFMA for 16 sources x 16 targets
// (details at direct_mixed_kernel).  The exponent is a sum of terms up to c r^2 (r the
// cloud's radius) that cancel to -c|x - y|^2, so its FP32 rounding error grows like
// 6e-8 c r^2; when c r^2 exceeds 8 (small eta) the kernel forms the same exponent on the FP64
// MFMA and rounds only the result to FP32 for v_exp_f32.  Source values are scaled by 2^-e
// (e = exponent of max v) so FP32 never under- or overflows.
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "mot_internal.h"

namespace mot {

// Uniform reads through the scalar unit: the sources of a product are written by earlier
// launches only.
#define MOT_CONST __attribute__((address_space(4)))

constexpr int kDirectT = 64;    // targets per FP64 item
constexpr int kMixedT = 256;    // targets per mixed item, 64 per wavefront
constexpr int kMixedS = 256;    // sources staged in LDS at a time

constexpr int kSmallWaves = 16, kSmallT = 16;  // small products: wavefronts, targets of a block at most

int direct_targets_per_item(int precision) { return precision == MOT_PREC_FP64 ? kDirectT : kMixedT; }

// Targets of a block of the small form, for about 256 blocks of the `width` products that run
// together (FP64: 2 to 16, mixed: a tile of 16), or 0 for products that take source ranges: a
// second launch costs 3 us, but the small form reads a source once per block.  Paths of three
// marginals in 2-D, 20 sweeps, FP64: 250 points 0.89 ms small, 1.11 with ranges; 1000 points
// 1.06 and 1.21; 1500 points 1.28 and 1.36; 2500 points 2.09 and 1.78; mixed: 1000 points 1.04
// and 1.30; 4000 points 1.32 and 1.64.
int direct_small_targets(int precision, int64_t nt, int64_t ns, int width)
{
    if ((double)nt * ns * width > (precision == MOT_PREC_FP64 ? 2.6e6 : 3.2e7)) return 0;
    int t = precision == MOT_PREC_FP64 ? 2 : kSmallT;
    while (t < kSmallT && width * nt > 256 * t) t *= 2;
    return width * nt > 256 * t && precision == MOT_PREC_FP64 ? 0 : t;
}

// Items a job is split into at least, while its sources last: two 256-thread blocks per CU in
// mixed precision, four in FP64.  Without the split a star of four 3-D marginals of 3000
// points ran a mixed product on 3 blocks: 760 us per sweep against 74 us with it (20000
// points: 5.3 ms against 0.53 ms); 1024 mixed items measured the same as 512, 2048 FP64 items
// the same as 1024.
int direct_items_wanted(int precision) { return precision == MOT_PREC_FP64 ? 1024 : 512; }

int direct_source_split(int64_t nt, int64_t ns, int precision)
{
    const int tpi = direct_targets_per_item(precision);
    const int64_t groups = (nt + tpi - 1) / tpi;
    const int64_t items = direct_items_wanted(precision), want = (items + groups - 1) / groups;
    const int64_t most = (ns + 63) / 64;               // at least 64 sources per range
    return (int)std::max<int64_t>(1, std::min<int64_t>(std::min(want, most), 64));
}

// Sources of one range.  Mixed ranges are multiples of 64 sources.
__device__ __forceinline__ void direct_range(const ProdJob &J, int range, int quantum, int64_t &a, int64_t &b)
{
    int64_t per = (J.ns + J.dsplit - 1) / J.dsplit;
    per = (per + quantum - 1) / quantum * quantum;
    a = min(J.ns, (int64_t)range * per);
    b = min(J.ns, a + per);
}

// 2^y for y = d2 c, c = -log2(e) / eta given as c_hi + c_lo, d2 >= 0.  n = rint(y) and the
// remainder f = d2 c - n by two FMAs, which keeps the low part of c, so f is exact to one
// rounding; 2^f on [-1/2, 1/2] is its Chebyshev interpolant of degree 11 (relative error
// 2e-17 with its coefficients rounded, below the FP64 rounding).  dmax = 1100 / |c| bounds y: terms below 2^-1100 are zero.
struct ExpScale {
    double c_hi, c_lo, dmax;
};

__device__ __forceinline__ ExpScale exp_scale(double eta)
{
    constexpr double L_hi = 1.4426950408889634, L_lo = 2.0355273740931033e-17;  // log2(e)
    ExpScale E;
    E.c_hi = -L_hi / eta;
    E.c_lo = -(fma(E.c_hi, eta, L_hi) + L_lo) / eta;
    if (!(E.c_hi > -DBL_MAX)) E.c_hi = -DBL_MAX;  // eta at the end of the FP64 range
    if (!(fabs(E.c_lo) < DBL_MAX)) E.c_lo = 0.0;
    E.dmax = fmin(1100.0 / -E.c_hi, DBL_MAX);
    return E;
}

__device__ __forceinline__ double exp2_scaled(double d2, const ExpScale &E)
{
    constexpr double kMagic = 6755399441055744.0;  // 1.5 2^52: adding it rounds to an integer
    d2 = fmin(d2, E.dmax);
    const double t = fma(d2, E.c_hi, kMagic);
    const int n = (int)__builtin_bit_cast(uint64_t, t);
    double f = fma(d2, E.c_hi, kMagic - t);
    f = fma(d2, E.c_lo, f);
    double p = 4.4558179475918685e-10;
    p = fma(p, f, 7.074194370937212e-09);
    p = fma(p, f, 1.017805708751313e-07);
    p = fma(p, f, 1.3215432535498108e-06);
    p = fma(p, f, 1.5252733841557202e-05);
    p = fma(p, f, 0.0001540353046372516);
    p = fma(p, f, 0.001333355814640647);
    p = fma(p, f, 0.009618129107587256);
    p = fma(p, f, 0.055504108664821625);
    p = fma(p, f, 0.24022650695910158);
    p = fma(p, f, 0.6931471805599453);
    p = fma(p, f, 1.0);
    return ldexp(p, n);
}

// FP64 variant: an item is 64 targets (one per lane) and one of the job's dsplit equal
// source ranges; the block's four wavefronts take the four quarters of that range, each
// summing its sources in ascending order, and the quarters are added in order.  Bound by
// FP64 issue (half the FP32 rate): 24 FP64 instructions per pair in 3-D, where a division and
// the library's exp took about 40.  Five marginals of up to 7000 points in 3-D: 122 -> 60 us
// per launch.
template <int D>
__global__ __launch_bounds__(256) void direct_fp64_kernel(const ProdJob *__restrict__ jobs,
                                                          const int4 *__restrict__ items, int n_items)
{
    __shared__ double red[3][kDirectT];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int64_t i = (int64_t)itm.y + lane;
        const bool act = i < J.nt;
        double x[D];
#pragma unroll
        for (int c = 0; c < D; ++c) x[c] = act ? gp(J.tgt_pts)[i * D + c] : 0.0;
        const ExpScale E = exp_scale(J.eta);
        int64_t a, b;
        direct_range(J, itm.z, 1, a, b);
        const int64_t q = (b - a + 3) / 4;
        const int64_t ja = min(b, a + wave * q), jb = min(b, ja + q);
        const MOT_CONST double *y = (const MOT_CONST double *)J.src_pts;
        const MOT_CONST double *v = (const MOT_CONST double *)J.v;
        double acc = 0.0;
#pragma unroll 4
        for (int64_t j = ja; j < jb; ++j) {
            double d2 = 0.0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const double df = x[c] - y[j * D + c];
                d2 = fma(df, df, d2);
            }
            acc = fma(v[j], exp2_scaled(d2, E), acc);
        }
        __syncthreads();  // the previous item's reads of red are done
        if (wave > 0) red[wave - 1][lane] = acc;
        __syncthreads();
        if (wave == 0 && act) {
            const double sum = ((acc + red[0][lane]) + red[1][lane]) + red[2][lane];
            if (J.dsplit > 1)
                J.dpart[(int64_t)itm.z * J.nt + i] = sum;
            else
                J.out[i] = sum;
        }
    }
}

// Small FP64 products: a block takes T = 2 to 16 targets (item: job, first target, T), lane l of
// wavefront w the target l % T and every (1024 / T)-th source from (64 w + l) / T on; the lanes of
// a target are added by lane exchanges, the wavefronts in order through LDS.  Bound by the
// latency of the launch and its loads: a path of three marginals of 500 points spent 5.9 us in a
// product's first launch and 3.7 us in adding its ranges.
template <int D>
__global__ __launch_bounds__(64 * kSmallWaves) void direct_fp64_small_kernel(const ProdJob *__restrict__ jobs,
                                                                             const int4 *__restrict__ items,
                                                                             int n_items)
{
    __shared__ double red[kSmallWaves][kSmallT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int T = itm.z, stride = 64 * kSmallWaves / T;
        const int64_t i = (int64_t)itm.y + (lane & (T - 1));
        const bool act = i < J.nt;
        const MOT_GLOBAL double *y = gp(J.src_pts), *v = gp(J.v);
        const int ns = (int)J.ns;
        constexpr int U = 4;  // sources in flight per lane
        double x[D], yv[U][D + 1], acc = 0.0;
        auto fetch = [&](int j0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + stride * u, jc = j < ns ? j : 0;
#pragma unroll
                for (int c = 0; c < D; ++c) yv[u][c] = y[jc * D + c];
                yv[u][D] = j < ns ? v[jc] : 0.0;
            }
        };
        const int first = tid / T;
        fetch(first);
#pragma unroll
        for (int c = 0; c < D; ++c) x[c] = act ? gp(J.tgt_pts)[i * D + c] : 0.0;
        const ExpScale E = exp_scale(J.eta);
        for (int j = first; j < ns; j += stride * U) {
            double w[U][D + 1];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c <= D; ++c) w[u][c] = yv[u][c];
            if (j + stride * U < ns) fetch(j + stride * U);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j + stride * u >= ns) break;
                double d2 = 0.0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const double df = x[c] - w[u][c];
                    d2 = fma(df, df, d2);
                }
                acc = fma(w[u][D], exp2_scaled(d2, E), acc);
            }
        }
        if (T <= 2) acc += lane_xor(acc, 2);
        if (T <= 4) acc += lane_xor(acc, 4);
        if (T <= 8) acc += lane_xor(acc, 8);
        acc += lane_xor(acc, 16);
        acc += lane_xor(acc, 32);
        __syncthreads();  // the previous item's reads of red are done
        if (lane < T) red[wave][lane] = acc;
        __syncthreads();
        if (tid < T && act) {
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < kSmallWaves; ++w) sum += red[w][tid];
            gp(J.out)[i] = sum;
        }
    }
}

// out_i = sum over the job's source ranges, in range order, of the partial sums.
__global__ __launch_bounds__(256) void direct_reduce_kernel(const ProdJob *__restrict__ jobs,
                                                            const int2 *__restrict__ items, int n_items)
{
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int64_t i = (int64_t)itm.y + threadIdx.x;
        if (i >= J.nt) continue;
        const MOT_GLOBAL double *p = gp(J.dpart) + i;
        const int64_t nt = J.nt;
        double acc = 0.0;
#pragma unroll 8
        for (int r = 0; r < J.dsplit; ++r) acc += p[(int64_t)r * nt];
        gp(J.out)[i] = acc;
    }
}

// Mixed variant on the MFMA.  A wavefront owns 64 targets, four tiles of 16, and runs over
// the item's sources 16 at a time: one 16x16x4 MFMA per tile gives the exponents of 256
// pairs, with the sources (y', a_y) as the A operand (lane l: source l % 16, component l / 16) and
// the targets (x, 1) as the B operand (lane l: target l % 16), so that lane l's four results
// belong to target l % 16 and four sources, whose values are one 16-byte LDS read.  A pair
// then costs the vector unit one v_exp_f32 (four issue slots) and one FMA, five slots where
// forming the exponent there too took nine; the MFMAs run beside it.
//   FP32: r = x.y' + a_y is at most c |x|^2 <= 8, so 2^r is summed and 2^(a_x) applied once per
//         target;
//   WIDE: the exponent with a_x on the FP64 MFMA, rounded to FP32 once (the D tile of the FP64
//         form holds row l / 16 + 4 r in register r).
// A lane sums 64 terms (every fourth of 256 sources) in FP32 and adds that to its FP64
// accumulator; the four lane groups of a target are added at the end.  Bound by vector issue:
// nine jobs of 1e5 x 1e5 pairs in 3-D took 19.6 ms with the exponent on the vector unit (four
// targets per lane), 13.2 ms here (9.2 ms is v_exp_f32's own rate); WIDE 27.8 -> 19.2 ms.  The
// bound of four blocks per CU makes the compiler keep the MFMA results in vector registers;
// without it they pass through accumulation registers (15 ms).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kMixedTiles = 4;

template <int D, bool WIDE>
__global__ __launch_bounds__(256, 4) void direct_mixed_kernel(const ProdJob *__restrict__ jobs,
                                                           const int4 *__restrict__ items, int n_items)
{
    typedef typename std::conditional<WIDE, double, float>::type real;
    typedef typename std::conditional<WIDE, f64x4, f32x4>::type real4;
    constexpr int kPad = WIDE ? 8 : 16;  // the four component rows start on different banks
    __shared__ real sy[2][4][kMixedS + kPad];
    __shared__ __align__(16) float sv[2][kMixedS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const double c2 = 1.4426950408889634 / J.eta;  // log2(e) / eta
        int e = *gp(J.v_exp);
        if (e == INT32_MIN) e = 0;
        const MOT_GLOBAL double *src = gp(J.src_pts), *vv = gp(J.v), *tgt = gp(J.tgt_pts);
        int64_t ja, jb;
        direct_range(J, itm.z, 64, ja, jb);
        const int64_t i0 = (int64_t)itm.y + 64 * wave;
        real xt[kMixedTiles];
        double ax[kMixedTiles], acc[kMixedTiles];
#pragma unroll
        for (int t = 0; t < kMixedTiles; ++t) {
            const int64_t i = i0 + 16 * t + li;
            double nrm = 0.0, mine = lk == 3 ? 1.0 : 0.0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const double dx = i < J.nt ? tgt[i * D + c] - J.ctr[c] : 0.0;
                if (lk == c) mine = dx;
                nrm += dx * dx;
            }
            xt[t] = (real)mine;
            ax[t] = -c2 * nrm;
            acc[t] = 0.0;
        }
        // source tid of the next stage, loaded one stage ahead; places past the range's end hold the
        // centre or a source of before, whose exponents are finite, with the value 0
        double ly[3] = {J.ctr[0], J.ctr[1], J.ctr[2]}, lv = 0.0;
        auto fetch = [&](int64_t j) {
            lv = 0.0;
            if (j < jb) {
#pragma unroll
                for (int c = 0; c < D; ++c) ly[c] = src[j * D + c];
                lv = vv[j];
            }
        };
        auto put = [&](int buf) {
            double nrm = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double dy = c < D ? ly[c] - J.ctr[c] : 0.0;
                sy[buf][c][tid] = (real)(2.0 * c2 * dy);
                nrm += dy * dy;
            }
            sy[buf][3][tid] = (real)(-c2 * nrm);
            sv[buf][tid] = (float)ldexp(lv, -e);
        };
        const int nstages = (int)((jb - ja + kMixedS - 1) / kMixedS);
        fetch(ja + tid);
        __syncthreads();  // the previous item's reads of LDS are done
        put(0);
        __syncthreads();
        for (int k = 0; k < nstages; ++k) {
            const int64_t j0 = ja + (int64_t)k * kMixedS;
            const bool more = k + 1 < nstages;
            if (more) fetch(j0 + kMixedS + tid);
            const int steps = ((int)min((int64_t)kMixedS, jb - j0) + 15) / 16;
            const real *ya = &sy[k & 1][lk][li];
            const f32x4 *va = reinterpret_cast<const f32x4 *>(sv[k & 1]);
            float part[kMixedTiles];
#pragma unroll
            for (int t = 0; t < kMixedTiles; ++t) part[t] = 0.0f;
#pragma unroll 2
            for (int m = 0; m < steps; ++m) {
                const real a = ya[16 * m];
                f32x4 w;
                if constexpr (WIDE) {
                    // register r of the FP64 tile is source l / 16 + 4 r
#pragma unroll
                    for (int r = 0; r < 4; ++r) w[r] = sv[k & 1][16 * m + lk + 4 * r];
                } else {
                    w = va[4 * m + lk];
                }
                real4 g[kMixedTiles];
#pragma unroll
                for (int t = 0; t < kMixedTiles; ++t) {
                    if constexpr (WIDE)
                        g[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, xt[t], f64x4{ax[t], ax[t], ax[t], ax[t]}, 0, 0, 0);
                    else
                        g[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, xt[t], f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
                }
#pragma unroll
                for (int t = 0; t < kMixedTiles; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        part[t] = fmaf(w[r], __builtin_amdgcn_exp2f((float)g[t][r]), part[t]);
            }
#pragma unroll
            for (int t = 0; t < kMixedTiles; ++t) acc[t] += (double)part[t];
            if (more) put((k + 1) & 1);
            __syncthreads();
        }
#pragma unroll
        for (int t = 0; t < kMixedTiles; ++t) {
            double s = acc[t];
            s += lane_xor(s, 16);
            s += lane_xor(s, 32);
            if constexpr (!WIDE) s *= exp2(ax[t]);
            const int64_t i = i0 + 16 * t + li;
            if (lk == 0 && i < J.nt) {
                const double o = ldexp(s, e);
                if (J.dsplit > 1)
                    gp(J.dpart)[(int64_t)itm.z * J.nt + i] = o;
                else
                    gp(J.out)[i] = o;
            }
        }
    }
}

// Small mixed products: a block takes one tile of 16 targets, wavefront w the w-th sixteenth of
// the sources (a multiple of 16), staged 64 at a time in its own LDS slice; the exponents as
// above, the wavefronts' sums added in order through LDS.  (64 targets to a block left most of
// the chip idle: 20 sweeps of a star of four 1000-point marginals 0.95 ms, here 0.78.)
template <int D, bool WIDE>
__global__ __launch_bounds__(64 * kSmallWaves) void direct_mixed_small_kernel(const ProdJob *__restrict__ jobs,
                                                                              const int4 *__restrict__ items,
                                                                              int n_items)
{
    typedef typename std::conditional<WIDE, double, float>::type real;
    typedef typename std::conditional<WIDE, f64x4, f32x4>::type real4;
    constexpr int kPitch = 64 + (WIDE ? 8 : 16);
    __shared__ real sy_all[kSmallWaves][4 * kPitch];
    __shared__ __align__(16) float sv_all[kSmallWaves][64];
    __shared__ double red[kSmallWaves][kSmallT];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    real *sy = sy_all[wave];
    float *sv = sv_all[wave];
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const MOT_GLOBAL double *src = gp(J.src_pts), *vv = gp(J.v), *tgt = gp(J.tgt_pts);
        const int ns = (int)J.ns;
        const int per = (ns + 16 * kSmallWaves - 1) / (16 * kSmallWaves) * 16;
        const int ja = min(ns, wave * per), jb = min(ns, ja + per);
        double ly[3] = {J.ctr[0], J.ctr[1], J.ctr[2]}, lv = 0.0;  // past the end: as above
        auto fetch = [&](int j) {
            lv = 0.0;
            if (j < jb) {
#pragma unroll
                for (int c = 0; c < D; ++c) ly[c] = src[(int64_t)j * D + c];
                lv = vv[j];
            }
        };
        fetch(ja + lane);
        const double c2 = 1.4426950408889634 / J.eta;  // log2(e) / eta
        int e = *gp(J.v_exp);
        if (e == INT32_MIN) e = 0;
        const int64_t i = (int64_t)itm.y + li;
        double nrmx = 0.0, mine = lk == 3 ? 1.0 : 0.0, acc = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double dx = i < J.nt ? tgt[i * D + c] - J.ctr[c] : 0.0;
            if (lk == c) mine = dx;
            nrmx += dx * dx;
        }
        const real xt = (real)mine;
        const double ax = -c2 * nrmx;
        // position of a source's value: register r of the FP64 tile's lane group g is source g + 4 r
        const int vpos = WIDE ? (lane & 48) | ((lane & 3) << 2) | ((lane >> 2) & 3) : lane;
        for (int j0 = ja; j0 < jb; j0 += 64) {
            const int steps = (min(64, jb - j0) + 15) >> 4;
            wave_sync();
            double nrm = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double dy = c < D ? ly[c] - J.ctr[c] : 0.0;
                sy[c * kPitch + lane] = (real)(2.0 * c2 * dy);
                nrm += dy * dy;
            }
            sy[3 * kPitch + lane] = (real)(-c2 * nrm);
            sv[vpos] = (float)ldexp(lv, -e);
            wave_sync();
            fetch(j0 + 64 + lane);
            float part = 0.0f;
            auto add = [&](auto U) {  // U tiles of 16 sources
                real4 g[U];
                f32x4 w[U];
#pragma unroll
                for (int m = 0; m < U; ++m) {
                    const real a = sy[lk * kPitch + 16 * m + li];
                    w[m] = reinterpret_cast<const f32x4 *>(sv)[4 * m + lk];
                    if constexpr (WIDE)
                        g[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, xt, f64x4{ax, ax, ax, ax}, 0, 0, 0);
                    else
                        g[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, xt, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
                }
#pragma unroll
                for (int m = 0; m < U; ++m)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        part = fmaf(w[m][r], __builtin_amdgcn_exp2f((float)g[m][r]), part);
            };
            switch (steps) {
            case 1: add(std::integral_constant<int, 1>()); break;
            case 2: add(std::integral_constant<int, 2>()); break;
            case 3: add(std::integral_constant<int, 3>()); break;
            default: add(std::integral_constant<int, 4>()); break;
            }
            acc += (double)part;
        }
        __syncthreads();  // the previous item's reads of red are done
        acc += lane_xor(acc, 16);
        acc += lane_xor(acc, 32);
        if constexpr (!WIDE) acc *= exp2(ax);
        if (lk == 0) red[wave][li] = acc;
        __syncthreads();
        if (tid < kSmallT && itm.y + tid < J.nt) {
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < kSmallWaves; ++w) sum += red[w][tid];
            gp(J.out)[(int64_t)itm.y + tid] = ldexp(sum, e);
        }
    }
}

template <int D>
static void launch_direct_d(const ProdJob *jobs, const int4 *items, int n_items, int precision, int diff, bool small,
                            hipStream_t s)
{
    const dim3 grid(n_items < 65535 ? n_items : 65535), block(small ? 64 * kSmallWaves : 256);
    if (precision == MOT_PREC_FP64) {
        if (small)
            hipLaunchKernelGGL(direct_fp64_small_kernel<D>, grid, block, 0, s, jobs, items, n_items);
        else
            hipLaunchKernelGGL(direct_fp64_kernel<D>, grid, block, 0, s, jobs, items, n_items);
    } else if (diff) {
        if (small)
            hipLaunchKernelGGL((direct_mixed_small_kernel<D, true>), grid, block, 0, s, jobs, items, n_items);
        else
            hipLaunchKernelGGL((direct_mixed_kernel<D, true>), grid, block, 0, s, jobs, items, n_items);
    } else {
        if (small)
            hipLaunchKernelGGL((direct_mixed_small_kernel<D, false>), grid, block, 0, s, jobs, items, n_items);
        else
            hipLaunchKernelGGL((direct_mixed_kernel<D, false>), grid, block, 0, s, jobs, items, n_items);
    }
}

hipError_t launch_direct(int d, const ProdJob *jobs_dev, const int4 *items, int n_items, const int2 *red_items,
                         int n_red, int precision, int diff, bool small, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (d == 1) launch_direct_d<1>(jobs_dev, items, n_items, precision, diff, small, s);
    if (d == 2) launch_direct_d<2>(jobs_dev, items, n_items, precision, diff, small, s);
    if (d == 3) launch_direct_d<3>(jobs_dev, items, n_items, precision, diff, small, s);
    if (n_red > 0)
        hipLaunchKernelGGL(direct_reduce_kernel, dim3(n_red < 16384 ? n_red : 16384), dim3(256), 0, s, jobs_dev,
                           red_items, n_red);
    return hipGetLastError();
}

}  // namespace mot
