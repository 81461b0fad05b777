// Whole transform of a 1-D or 2-D fast summation job in one workgroup: fold (a2), forward
// transform, multiply, inverse transform (a3-a5), from the patches to the result grid with
// the box held in LDS.
//
// Only L_c box cells per dimension enter the transform and only the band |k_c| <= M leaves it
// (box 43 to 110, band 33 to 129 of grids of 128 to 512 points), so the pruned transforms are
// short dense contractions with the DFT matrix and run on the FP32 MFMA: a 256-point radix-2
// line on a wavefront costs about 500 vector instructions whatever it holds of zeros, and one
// workgroup doing a 70 x 70 box that way took 32 us.  With w = exp(-2 pi i / n), i' = i + lo the
// grid index of box cell i, H = M + 1:
//   rows       X[i0][k]  = sum_i1 R[i0][i1] w^(k i1'),                     k = 0..M
//   columns    P = sum_i0 cos X, Q = sum_i0 sin X at f = 0..M; the values at +-f are
//              X^(+-f) = P -+ i Q, times D(k, +-f), and only their sum and difference
//              E = X^(f) + X^(-f), O = X^(f) - X^(-f) enter the way back (f = 0: E = X^(0))
//   columns    Z[i0][k]  = sum_f (cos E + i sin O), times 2 for k > 0
//   rows       G[i0][i1] = sum_k Re(Z conj(w)^(k i1')),  the real inverse of the half spectrum
// 1-D is the first and last line, times D in between.  Powers of w come from the n-point table
// in LDS.  Jobs of small problems are bound by the launches of a pass chain (fold and three
// passes of 4 to 8 us each), those of row-by-row circles by the traffic between its passes.
#include <type_traits>

#include "nfft_device.h"

namespace mot {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Steps of four of a contraction over K entries: four steps at a time, whose operands are read
// together before their MFMAs (a loop around an MFMA is not unrolled by the compiler), then
// the rest.  f(first entry, steps as a constant).  The real cosine sums over cells (xr and pr
// below) hold the sum of all cells, whose error is common to every result of the product and
// shifts the scalings of every sweep: step u of a round goes to the u-th of four chains of
// theirs (standard deviation of a product's mean relative error over problems of 1000 to 2300
// points: 4.6e-8 with one chain, 2.6e-8 here, 2.2e-8 by radix-2 lines).
template <class F>
__device__ __forceinline__ void k_steps(int K, F f)
{
    int s = 0;
    for (; s + 12 < K; s += 16) f(s, std::integral_constant<int, 4>());
    for (; s < K; s += 4) f(s, std::integral_constant<int, 1>());
}

// The same from the last step down, for sums over frequencies: the spectrum falls by orders of
// magnitude over the band, and a chain of FP32 sums that starts with its small terms rounds at
// their size until the large ones come (spread of a 2-D product's relative errors about their
// mean, bands of 12, 28 and 40: upward 7.9e-8, 8.5e-8 and 8.3e-8, downward 6.5e-8, 6.4e-8 and
// 6.4e-8; by radix-2 lines 6.4e-8, 6.2e-8 and 6.2e-8).
template <class F>
__device__ __forceinline__ void k_steps_down(int K, F f)
{
    int s = (K + 3) / 4 * 4 - 4;
    for (; s >= 12; s -= 16) f(s, std::integral_constant<int, 4>());
    for (; s >= 0; s -= 4) f(s, std::integral_constant<int, 1>());
}

// LDS layout of a 2-D job: R[L0p][p1] then E, O (real, imaginary) [4][H4][py] in one place, X[L0p][px]
// then Z[L0p][pz] in another.  Rows read as A operands (16 rows x 4 columns of a wavefront) have
// pitches of 4 x odd, rows read as B operands (4 rows x 16 columns) of 16 x odd: no bank conflicts.
__device__ __forceinline__ void plane2(const ProdJob &J, const float2 *tw, float *ry, float *xz)
{
    const PlaneGeom P(J.L[0], J.L[1], J.M);
    const int nw = (int)(blockDim.x >> 6), wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int M = J.M, B = 2 * M + 1, H = M + 1, L0 = J.L[0], L1 = J.L[1], lo0 = J.lo[0], lo1 = J.lo[1];
    const int mask = J.n - 1;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const int m_tiles = P.L0p / 16, k_tiles = P.Hp / 16;
    // rows: X real in columns [0, Hp), imaginary in [Hp, 2 Hp)
    for (int t = wave; t < m_tiles * k_tiles; t += nw) {
        const int m0 = t % m_tiles * 16, k0 = t / m_tiles * 16;
        const int k = k0 + li;
        const float *a = ry + (m0 + li) * P.p1 + lk;
        int idx = k * (lk + lo1);
        f32x4 xr4[4] = {zero, zero, zero, zero}, xi = zero;
        k_steps(L1, [&](int s, auto U) {
            float2 w[U];
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = tw[(idx + 4 * k * u) & mask];
                v[u] = a[s + 4 * u];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                xr4[u] = mfma4(v[u], w[u].x, xr4[u]);
                xi = mfma4(v[u], w[u].y, xi);
            }
            idx += 4 * k * U;
        });
        const f32x4 xr = (xr4[0] + xr4[1]) + (xr4[2] + xr4[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float *x = xz + (m0 + 4 * lk + r) * P.px + k;
            x[0] = k < H ? xr[r] : 0.0f;
            x[P.Hp] = k < H ? xi[r] : 0.0f;
        }
    }
    __syncthreads();
    // columns forward and the multiplier: tiles of 16 frequencies f x 16 columns k
    const int f_tiles = (H + 15) / 16, yst = P.H4 * P.py;
    const MOT_GLOBAL float *D = gp(J.D);
    for (int t = wave; t < f_tiles * k_tiles; t += nw) {
        const int f0 = t % f_tiles * 16, k0 = t / f_tiles * 16;
        const int k = k0 + li, f = f0 + li;
        float dp[4], dn[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int fr = f0 + 4 * lk + r;
            const bool in = fr < H && k < H;
            dp[r] = in ? D[k * B + M + fr] : 0.0f;
            dn[r] = in && fr > 0 ? D[k * B + M - fr] : 0.0f;
        }
        const float *b = xz + lk * P.px + k;
        int idx = f * (lk + lo0);
        // cos X and sin X, w = cos - i sin
        f32x4 pr4[4] = {zero, zero, zero, zero}, pi = zero, qr = zero, qi = zero;
        k_steps(L0, [&](int s, auto U) {
            float2 w[U];
            float xr[U], xi[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = tw[(idx + 4 * f * u) & mask];
                xr[u] = b[(s + 4 * u) * P.px];
                xi[u] = b[(s + 4 * u) * P.px + P.Hp];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pr4[u] = mfma4(w[u].x, xr[u], pr4[u]);
                pi = mfma4(w[u].x, xi[u], pi);
                qr = mfma4(-w[u].y, xr[u], qr);
                qi = mfma4(-w[u].y, xi[u], qi);
            }
            idx += 4 * f * U;
        });
        const f32x4 pr = (pr4[0] + pr4[1]) + (pr4[2] + pr4[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int fr = f0 + 4 * lk + r;
            if (fr >= P.H4) continue;
            // E and O of X(+-f) = P -+ i Q times dp, dn; t = 0 but at the band's edge and f = 0
            const float s = dp[r] + dn[r], t = dp[r] - dn[r];
            float *y = ry + fr * P.py + k;
            y[0] = fmaf(qi[r], t, pr[r] * s);
            y[yst] = fmaf(-qr[r], t, pi[r] * s);
            y[2 * yst] = fmaf(pr[r], t, qi[r] * s);
            y[3 * yst] = fmaf(pi[r], t, -qr[r] * s);
        }
    }
    __syncthreads();
    // columns back: tiles of 16 rows i0 x 16 columns k; conj(w)^(f i) = cos + i sin
    for (int t = wave; t < m_tiles * k_tiles; t += nw) {
        const int m0 = t % m_tiles * 16, k0 = t / m_tiles * 16;
        const int k = k0 + li, i = m0 + li + lo0;
        const float *b = ry + lk * P.py + k;
        int idx = (P.H4 - 4 + lk) * i;
        f32x4 zr = zero, zi = zero;
        k_steps_down(H, [&](int s, auto U) {
            float2 w[U];
            float er[U], ei[U], orr[U], oi[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float *y = b + (s - 4 * u) * P.py;
                w[u] = tw[(idx - 4 * i * u) & mask];
                er[u] = y[0];
                ei[u] = y[yst];
                orr[u] = y[2 * yst];
                oi[u] = y[3 * yst];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                zr = mfma4(w[u].x, er[u], zr);
                zi = mfma4(w[u].x, ei[u], zi);
                zr = mfma4(w[u].y, oi[u], zr);     // -sin O_i
                zi = mfma4(-w[u].y, orr[u], zi);   // +sin O_r
            }
            idx -= 4 * i * U;
        });
        const float wk = k == 0 ? 1.0f : 2.0f;
        if (k < P.H4)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float *z = xz + (m0 + 4 * lk + r) * P.pz + k;
                z[0] = wk * zr[r];
                z[P.H4] = wk * zi[r];
            }
    }
    __syncthreads();
    // rows back: tiles of 16 rows x 16 cells, Re(Z conj(w)) = Z_r cos - Z_i sin
    MOT_GLOBAL float *grid = gp(J.grid);
    const int n_tiles = (L1 + 15) / 16;
    for (int t = wave; t < m_tiles * n_tiles; t += nw) {
        const int m0 = t % m_tiles * 16, c0 = t / m_tiles * 16;
        const int i1 = c0 + li, i = i1 + lo1;
        const float *a = xz + (m0 + li) * P.pz + lk;
        int idx = (P.H4 - 4 + lk) * i;
        f32x4 g = zero, h = zero;
        k_steps_down(H, [&](int s, auto U) {
            float2 w[U];
            float zr[U], zi[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = tw[(idx - 4 * i * u) & mask];
                zr[u] = a[s - 4 * u];
                zi[u] = a[s - 4 * u + P.H4];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                g = mfma4(zr[u], w[u].x, g);
                h = mfma4(zi[u], w[u].y, h);
            }
            idx -= 4 * i * U;
        });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i0 = m0 + 4 * lk + r;
            if (i0 < L0 && i1 < L1) grid[i0 * L1 + i1] = g[r] + h[r];
        }
    }
}

// 1-D: eight lanes per output, each every eighth term; the same chains and order of sums.
__device__ __forceinline__ void plane1(const ProdJob &J, const float2 *tw, const float *R, float2 *Y)
{
    const int M = J.M, L0 = J.L[0], lo0 = J.lo[0], mask = J.n - 1;
    const int q = threadIdx.x & 7, step = (int)(blockDim.x >> 3);
    for (int k0 = 0; k0 <= M; k0 += step) {  // uniform trip count: the lane sums need every lane
        const int k = k0 + (int)(threadIdx.x >> 3);
        float yr4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, yi = 0.0f;
        auto term = [&](int i, int u) {
            const float2 w = tw[(k * (i + lo0)) & mask];
            yr4[u] = fmaf(R[i], w.x, yr4[u]);
            yi = fmaf(R[i], w.y, yi);
        };
        if (k <= M) {
            int i = q;
            for (; i + 24 < L0; i += 32)
#pragma unroll
                for (int u = 0; u < 4; ++u) term(i + 8 * u, u);
            for (; i < L0; i += 8) term(i, 0);
        }
        float yr = (yr4[0] + yr4[1]) + (yr4[2] + yr4[3]);
#pragma unroll
        for (int h = 1; h <= 4; h <<= 1) {
            yr += lane_xor(yr, h);
            yi += lane_xor(yi, h);
        }
        if (q == 0 && k <= M) {
            const float d = gp(J.D)[k] * (k == 0 ? 1.0f : 2.0f);
            Y[k] = make_float2(yr * d, yi * d);
        }
    }
    __syncthreads();
    for (int i0 = 0; i0 < L0; i0 += step) {
        const int i = i0 + (int)(threadIdx.x >> 3);
        float g = 0.0f;
        if (i < L0)
#pragma unroll 4
            for (int k = ((M - q) >> 3) * 8 + q; k >= 0; k -= 8) {  // downward, as k_steps_down
                const float2 w = tw[(k * (i + lo0)) & mask], y = Y[k];
                g = fmaf(y.x, w.x, fmaf(y.y, w.y, g));
            }
#pragma unroll
        for (int h = 1; h <= 4; h <<= 1) g += lane_xor(g, h);
        if (q == 0 && i < L0) gp(J.grid)[i] = g;
    }
}

__global__ __launch_bounds__(1024) void plane_kernel(const ProdJob *__restrict__ jobs, const int2 *__restrict__ items,
                                                     int n_items)
{
    __shared__ int32_t s_tab[kFoldTab];
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int d = J.d, n = J.n, L0 = J.L[0], L1 = d == 2 ? J.L[1] : 1;
        const PlaneGeom P(L0, L1, J.M);
        float2 *tw = reinterpret_cast<float2 *>(smem);
        float *R = reinterpret_cast<float *>(tw + n);
        const int pitch = d == 2 ? P.p1 : 1;
        const float rL1 = 1.0f / (float)L1;
        for (int j = tid; j < n; j += blockDim.x) {
            const float2 w = ld2(J.twiddle, j & (n / 2 - 1));
            tw[j] = j < n / 2 ? w : make_float2(-w.x, -w.y);
        }
        if (d == 2)  // the padding of R enters the contractions as zeros
            for (int f = tid; f < P.L0p * P.p1; f += blockDim.x) {
                const int row = div_small(f, 1.0f / (float)P.p1), i = f - row * P.p1;
                if (row >= L0 || i >= L1) R[f] = 0.0f;
            }
        if (itm.y == 0) {  // folded by a launch of its own
            const MOT_GLOBAL float *grid = gp(J.grid);
            const int cells = L0 * L1, step = (int)blockDim.x;
            for (int f0 = tid; f0 < cells; f0 += 8 * step) {
                float v[8];  // loads in flight together; past the end entry 0 is read and dropped
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = grid[f0 + u * step < cells ? f0 + u * step : 0];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int f = f0 + u * step, row = div_small(f, rL1);
                    if (f < cells) R[row * pitch + f - row * L1] = v[u];
                }
            }
        } else {
            const int ntab = (d == 2 ? J.ntile[0] * J.ntile[1] : J.ntile[0]) + 1;
            const MOT_GLOBAL int32_t *tg = gp(J.src_tile_chunks);
            const bool staged = ntab <= kFoldTab;
            if (staged)
                for (int i = tid; i < ntab; i += blockDim.x) s_tab[i] = tg[i];
            __syncthreads();
            const int32_t *lt = s_tab;
            for (int f = tid; f < L0 * L1; f += blockDim.x) {
                const int row = div_small(f, rL1), i = f - row * L1, gu[2] = {row, 0};
                float v;
                if (d == 2)
                    v = staged ? fold_cell<2>(J, gu, i, lt) : fold_cell<2>(J, gu, i, tg);
                else
                    v = staged ? fold_cell<1>(J, gu, row, lt) : fold_cell<1>(J, gu, row, tg);
                R[row * pitch + i] = v;
            }
        }
        __syncthreads();
        if (d == 2)
            plane2(J, tw, R, R + P.ry);
        else
            plane1(J, tw, R, reinterpret_cast<float2 *>(R + (L0 + 1) / 2 * 2));
        __syncthreads();  // LDS is rewritten by the next item
    }
}

// Threads per job: blocks of four wavefronts fill the chip from 512 jobs on; fewer jobs are
// bound by the rounds of a job's tiles and take sixteen wavefronts each.
hipError_t launch_plane(const ProdJob *jobs, const int2 *items, int n_items, int lds_bytes, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (lds_bytes > kPlaneLds) return hipErrorInvalidValue;
    hipLaunchKernelGGL(plane_kernel, dim3(n_items < 65535 ? n_items : 65535), dim3(n_items >= 512 ? 256 : 1024),
                       lds_bytes, s, jobs, items, n_items);
    return hipGetLastError();
}

}  // namespace mot
