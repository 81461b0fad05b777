// Truncated direct products for small eta (the truncation suggested at the end of
// Sec. 6.1):
//   out_i = sum over sources j in the cells near target i's cell of v_j exp(-|x_i - y_j|^2 / eta).
// Both point sets are sorted by cubic cells of side h (the a1 binning with tile edge 1).
// The sources summed for a target are those of every cell whose box distance to the
// target's cell is at most r_c, so every source within r_c of the target is included and
// the terms left out are below exp(-r_c^2 / eta) v_j.  In the row-major cell order the
// cells of one row of the neighbourhood (fixed leading coordinates, a range along the last
// one) are one contiguous range of sorted sources.
//
// One wavefront takes one item: up to 64 targets (FP64: 64 R, R per lane) from a run of B
// consecutive cells of one row (consecutive in the sorted order; B > 1 fills the lanes
// when cells hold few points).  The neighbourhood rows of a run are those of its first
// cell, widened by B - 1 cells along the row.  The wave first lists the item's non-empty
// rows in LDS with the prefix sum of their lengths, so its sources form one list; it then
// stages that list 64 entries at a time through its own LDS slice (every stage full but
// the last) and multiplies a stage while the next one's sources are loaded.  The waves of a
// block take different items and synchronise only within themselves.
//
// Mixed precision: the exponents of 16 sources x 16 targets are one 16x16x4 FP64 MFMA.  With
// c = log2(e) / eta and coordinates relative to the centre of the item's run of cells,
//   -c |x - y|^2 = -c |x|^2 + x.(2 c y) - c |y|^2
// is the contraction of (x, 1) with (2 c y, -c |y|^2) on top of the target's -c |x|^2, the MFMA's
// addend; it is rounded to FP32 once, for v_exp_f32.  It is formed in full, without a part kept
// back for a factor per target: the largest terms of a sum have exponents near 0 and little
// rounding, and the smallest, log2(eps) (about -41 at the default target), leave 2^-85 of
// FP32's range to the values.  (A shift common to a run, half the largest c |x|^2 of its cells,
// rounds every exponent at the shift's size and takes as much off that range: sparse clouds have
// shifts up to 98.  It saves registers, 0.5 to 2 % of a launch in 3-D and nothing in 2-D.)
// Values are scaled by 2^-e (e = exponent of max v); a lane sums 16 of a stage's 64 sources in
// FP32 and adds that to its FP64 accumulator.  A pair costs the vector unit a conversion,
// v_exp_f32 and an FMA, and targets come in tiles of 16 where one per lane left half of the
// lanes idle in sparse cells.  Star trees in 3-D, time
// per launch against FP32 coordinate differences with a target per lane: nine jobs of 1e5
// points, eta = 1e-3 5.1 -> 5.0 ms, eta = 3e-4 2.0 -> 1.85 ms; three jobs of 20000 points 0.45 -> 0.27
// ms, of 5000 points at eta = 3e-4 0.12 -> 0.06 ms.  Bound by vector issue (about 160 cycles per
// 16 x 16 pairs with the staging, 131 without); a bound of three or five blocks per CU measured
// 2 % slower.
// In 1-D and 2-D the contraction has one or two empty terms of four, and exponents of FP32
// coordinate differences, scaled by sqrt(c) and relative to the run's centre, take fewer cycles than
// the MFMA and the conversion; they are used for runs within a half-diagonal of 3, where rounding
// the coordinates moves a term that counts by about 1e-7.  Sweeps of star trees, differences and
// MFMA: 2-D, six marginals of 60000 points, eta = 3e-4 0.96 and 1.21 ms, 1e-3 2.23 and 2.88, 3e-3
// 4.5 and 5.8; 1-D, four of 60000, 1e-4 0.81 and 1.24 ms.  (In 3-D, three differences: 44 cycles a
// wavefront and source of 64 targets against 40 with the MFMA, which fills its tiles better.)
// FP64: plain exp(-|x - y|^2 / eta) with FP64 sums in source order.
#include <type_traits>

#include "mot_internal.h"

namespace mot {

// Sorted source range [a, b) of neighbour row ri of the run of B cells starting at cc;
// false when the row lies outside the grid or farther than r_c from the run.
template <int D>
__device__ __forceinline__ bool trunc_row(const ProdJob &J, const int cc[3], int B, int ri, int64_t &a,
                                          int64_t &b)
{
    const int w = J.tw, nc = J.nc, span = 2 * w + 1;
    int del[2] = {0, 0};
    if (D == 3) {
        del[0] = ri / span - w;
        del[1] = ri % span - w;
    } else if (D == 2) {
        del[0] = ri - w;
    }
    double used = 0.0;
    int64_t base = 0;
#pragma unroll
    for (int c = 0; c < D - 1; ++c) {
        const int x = cc[c] + del[c];
        if (x < 0 || x >= nc) return false;
        const int e = abs(del[c]) - 1;
        if (e > 0) used += (double)e * e;
        base = base * nc + x;
    }
    const double rem = J.q2 - used;
    if (rem < 0.0) return false;
    const int wl = min(w, 1 + (int)floor(sqrt(rem)));
    const int xa = max(cc[D - 1] - wl, 0), xb = min(cc[D - 1] + B - 1 + wl, nc - 1);
    const MOT_GLOBAL int32_t *off = gp(J.src_cell_off);
    a = off[base * nc + xa];
    b = off[base * nc + xb + 1];
    return b > a;
}

template <int D>
__device__ __forceinline__ void trunc_cell(const ProdJob &J, int cell, int cc[3])
{
    cc[0] = cc[1] = cc[2] = 0;
    int rem = cell;
#pragma unroll
    for (int c = D - 1; c >= 0; --c) {
        cc[c] = rem % J.nc;
        rem /= J.nc;
    }
}

__device__ __forceinline__ int trunc_rows(int D, int w)
{
    const int span = 2 * w + 1;
    return D == 1 ? 1 : (D == 2 ? span : span * span);
}

constexpr int kTruncWaves = 4;  // independent wavefronts per block, one item each

__device__ __forceinline__ int wave_incl_scan(int v, int lane)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kSrcPitch = 64 + 8;  // staged component rows, in doubles (LDS banks)

// DIFF: exponents of FP32 coordinate differences (D < 3).
template <int D, bool DIFF>
__global__ __launch_bounds__(64 * kTruncWaves, 4) void trunc_mixed_kernel(const ProdJob *__restrict__ jobs,
                                                                          const int4 *__restrict__ items,
                                                                          int n_items)
{
    __shared__ __align__(16) double sw_all[kTruncWaves][4 * kSrcPitch];  // 2c y, -c |y|^2
    __shared__ __align__(16) float sv_all[kTruncWaves][64];
    __shared__ int32_t ra_all[kTruncWaves][kMaxTruncRows];      // first sorted source of each row
    __shared__ int32_t rp_all[kTruncWaves][kMaxTruncRows + 1];  // sources before each row
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    double *sw = sw_all[wave];
    float *sv = sv_all[wave];
    int32_t *ra = ra_all[wave], *rp = rp_all[wave];
    for (int it = blockIdx.x * kTruncWaves + wave; it < n_items; it += gridDim.x * kTruncWaves) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int cnt = itm.w & 0xffff, B = itm.w >> 16;
        int cc[3];
        trunc_cell<D>(J, itm.y, cc);
        const double c2 = 1.4426950408889634 / J.eta;  // log2(e) / eta
        double ctr[3] = {0.0, 0.0, 0.0};  // centre of the run
#pragma unroll
        for (int c = 0; c < D; ++c) ctr[c] = J.glo[c] + (cc[c] + (c == D - 1 ? 0.5 * B : 0.5)) * J.h;
        int e = *gp(J.v_exp);
        if (e == INT32_MIN) e = 0;
        const MOT_GLOBAL double *tgt = gp(J.tgt_pts);
        const MOT_GLOBAL double *src = gp(J.src_pts);
        const MOT_GLOBAL double *vv = gp(J.v);
        // the item's non-empty neighbour rows, compacted in row order with the prefix of
        // their lengths: the sources to sum are one list of `total` entries
        int nr = 0, total = 0;
        const int nrows = trunc_rows(D, J.tw);
        wave_sync();
        for (int r0 = 0; r0 < nrows; r0 += 64) {
            int64_t a = 0, b = 0;
            const bool ok = r0 + lane < nrows && trunc_row<D>(J, cc, B, r0 + lane, a, b);
            const int len = ok ? (int)(b - a) : 0;
            const int f = len > 0 ? 1 : 0;
            const int fpos = wave_incl_scan(f, lane), lpos = wave_incl_scan(len, lane);
            if (f) {
                ra[nr + fpos - 1] = (int32_t)a;
                rp[nr + fpos - 1] = total + lpos - len;
            }
            nr += __builtin_amdgcn_readlane(fpos, 63);
            total += __builtin_amdgcn_readlane(lpos, 63);
        }
        if (lane == 0) rp[nr] = total;
        wave_sync();
        // targets: 16-wide tile t, lane l has component l / 16 of target l % 16, and its -c |x|^2
        double xt[4], ax[4], acc[4];
        float xf[4][2];  // DIFF: every component of target l % 16
        const double sc = sqrt(c2);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool act = 16 * t + li < cnt;
            const int64_t i = (int64_t)itm.z + 16 * t + li;
            double nrm = 0.0;
            xt[t] = lk == 3 ? 1.0 : 0.0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const double dx = act ? tgt[i * D + c] - ctr[c] : 0.0;
                if (lk == c) xt[t] = dx;
                if (DIFF && c < 2) xf[t][c] = (float)(dx * sc);
                nrm += dx * dx;
            }
            ax[t] = -c2 * nrm;
            acc[t] = 0.0;
        }
        // stages of 64 consecutive list entries; each lane follows its entry's row with a
        // pointer that only moves forward, and loads its source one stage ahead
        int row = 0;
        double ly[3] = {ctr[0], ctr[1], ctr[2]}, lv = 0.0;
        auto fetch = [&](int q) {
            lv = 0.0;
            if (q < total) {
                while (rp[row + 1] <= q) ++row;
                const int64_t j = (int64_t)ra[row] + (q - rp[row]);
#pragma unroll
                for (int c = 0; c < D; ++c) ly[c] = src[j * D + c];
                lv = vv[j];
            }
        };
        // position of a source's value: the FP64 tile's register r of lane group g is source g + 4 r
        const int vpos = DIFF ? lane : (lane & 48) | ((lane & 3) << 2) | ((lane >> 2) & 3);
        float *sf = reinterpret_cast<float *>(sw);  // DIFF: components of the stage's sources, 64 each
        auto scan = [&](auto NT) {
            for (int s0 = 0; s0 < total; s0 += 64) {
                const int steps = (min(64, total - s0) + 15) >> 4;
                wave_sync();
                if constexpr (DIFF) {
#pragma unroll
                    for (int c = 0; c < D; ++c) sf[64 * c + lane] = (float)((ly[c] - ctr[c]) * sc);
                    sv[vpos] = (float)ldexp(lv, -e);
                } else {
                    // entries past the list's end have the value 0 and the place of the run's centre
                    // or of a source of before, whose exponents are finite
                    double nrm = 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double dy = c < D ? ly[c] - ctr[c] : 0.0;
                        sw[c * kSrcPitch + lane] = 2.0 * c2 * dy;
                        nrm += dy * dy;
                    }
                    sw[3 * kSrcPitch + lane] = -c2 * nrm;
                    sv[vpos] = (float)ldexp(lv, -e);
                }
                wave_sync();
                fetch(s0 + 64 + lane);
                float part[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) part[t] = 0.0f;
                for (int m = 0; DIFF && m < steps; ++m) {
                    const f32x4 w = reinterpret_cast<const f32x4 *>(sv)[4 * m + lk];
                    f32x4 y[2];
#pragma unroll
                    for (int c = 0; c < D && c < 2; ++c) y[c] = reinterpret_cast<const f32x4 *>(sf + 64 * c)[4 * m + lk];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float dx = xf[t][0] - y[0][r];
                            float q = dx * dx;
                            if (D > 1) {
                                const float dy = xf[t][1] - y[1][r];
                                q = fmaf(dy, dy, q);
                            }
                            part[t] = fmaf(w[r], __builtin_amdgcn_exp2f(-q), part[t]);
                        }
                }
                for (int m = 0; !DIFF && m < steps; ++m) {
                    const double a = sw[lk * kSrcPitch + 16 * m + li];
                    const f32x4 w = reinterpret_cast<const f32x4 *>(sv)[4 * m + lk];
                    f64x4 g[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        g[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, xt[t], f64x4{ax[t], ax[t], ax[t], ax[t]}, 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            part[t] = fmaf(w[r], __builtin_amdgcn_exp2f((float)g[t][r]), part[t]);
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] += (double)part[t];
            }
        };
        fetch(lane);
        switch ((cnt + 15) >> 4) {
        case 1: scan(std::integral_constant<int, 1>()); break;
        case 2: scan(std::integral_constant<int, 2>()); break;
        case 3: scan(std::integral_constant<int, 3>()); break;
        default: scan(std::integral_constant<int, 4>()); break;
        }
        MOT_GLOBAL double *out = gp(J.out);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            double s = acc[t];
            s += lane_xor(s, 16);
            s += lane_xor(s, 32);
            if (lk == 0 && 16 * t + li < cnt) out[(int64_t)itm.z + 16 * t + li] = ldexp(s, e);
        }
    }
}

template <int D, int R>
__global__ __launch_bounds__(64) void trunc_fp64_kernel(const ProdJob *__restrict__ jobs,
                                                        const int4 *__restrict__ items, int n_items)
{
    __shared__ double sy[64][4];
    const int lane = threadIdx.x;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int cnt = itm.w & 0xffff, B = itm.w >> 16;
        int cc[3];
        trunc_cell<D>(J, itm.y, cc);
        const double inv_eta = 1.0 / J.eta;
        const MOT_GLOBAL double *tgt = gp(J.tgt_pts);
        const MOT_GLOBAL double *src = gp(J.src_pts);
        const MOT_GLOBAL double *vv = gp(J.v);
        double xs[R][3], acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool act = lane + 64 * r < cnt;
            const int64_t i = (int64_t)itm.z + lane + 64 * r;
#pragma unroll
            for (int c = 0; c < 3; ++c) xs[r][c] = (c < D && act) ? tgt[i * D + c] : 0.0;
            acc[r] = 0.0;
        }
        const int nrows = trunc_rows(D, J.tw);
        for (int ri = 0; ri < nrows; ++ri) {
            int64_t a, b;
            if (!trunc_row<D>(J, cc, B, ri, a, b)) continue;
            for (int64_t j0 = a; j0 < b; j0 += 64) {
                const int nj = (int)min((int64_t)64, b - j0);
                __syncthreads();
                if (lane < nj) {
                    const int64_t j = j0 + lane;
#pragma unroll
                    for (int c = 0; c < D; ++c) sy[lane][c] = src[j * D + c];
                    sy[lane][3] = vv[j];
                }
                __syncthreads();
                for (int jj = 0; jj < nj; ++jj) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        double d2 = 0.0;
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            const double df = xs[r][c] - sy[jj][c];
                            d2 += df * df;
                        }
                        acc[r] += sy[jj][3] * exp(-d2 * inv_eta);
                    }
                }
            }
        }
        MOT_GLOBAL double *out = gp(J.out);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = (int64_t)itm.z + lane + 64 * r;
            if (lane + 64 * r < cnt) out[i] = acc[r];
        }
    }
}

template <int D>
static void launch_trunc_d(int precision, int diff, int R, const ProdJob *jobs, const int4 *items, int n_items, hipStream_t s)
{
    if (precision == MOT_PREC_FP64) {
        const dim3 grid(n_items < (1 << 20) ? n_items : (1 << 20)), block(64);
        if (R == 1) hipLaunchKernelGGL((trunc_fp64_kernel<D, 1>), grid, block, 0, s, jobs, items, n_items);
        if (R == 2) hipLaunchKernelGGL((trunc_fp64_kernel<D, 2>), grid, block, 0, s, jobs, items, n_items);
    } else {
        const int blocks = (n_items + kTruncWaves - 1) / kTruncWaves;
        const dim3 grid(blocks < (1 << 20) ? blocks : (1 << 20)), block(64 * kTruncWaves);
        if constexpr (D < 3) {
            if (!diff) {
                hipLaunchKernelGGL((trunc_mixed_kernel<D, true>), grid, block, 0, s, jobs, items, n_items);
                return;
            }
        }
        hipLaunchKernelGGL((trunc_mixed_kernel<D, false>), grid, block, 0, s, jobs, items, n_items);
    }
}

hipError_t launch_trunc(int d, int precision, int diff, int R, const ProdJob *jobs_dev, const int4 *items, int n_items,
                        hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (R != 1 && (R != 2 || precision != MOT_PREC_FP64)) return hipErrorInvalidValue;
    if (d == 1) launch_trunc_d<1>(precision, diff, R, jobs_dev, items, n_items, s);
    if (d == 2) launch_trunc_d<2>(precision, diff, R, jobs_dev, items, n_items, s);
    if (d == 3) launch_trunc_d<3>(precision, diff, R, jobs_dev, items, n_items, s);
    return hipGetLastError();
}

}  // namespace mot
