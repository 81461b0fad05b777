// NFFT fast-summation kernels for gfx950: point binning, window rows, spreading into
// per-tile patches, the deterministic patch fold, and grid-to-point interpolation.
//
// Fast summation (Sec. 5, Algorithm 4) evaluates beta = F_t (kappa_hat (.) F*_s v).
// The adjoint NDFT F*_s is approximated by spreading v onto an oversampled grid of n
// cells per dimension with a Kaiser-Bessel window followed by an FFT; the NDFT F_t by an
// inverse FFT followed by interpolation with the same window.  Grid coordinates of a
// point x are u = x * s + o with s = n / (2 tau) (the 2 tau-periodic kernel becomes
// n-periodic); each point touches the 2m grid cells l = cell - m + 1 .. cell + m per
// dimension, cell = floor(u).
//
// Work decomposition: points are stable-sorted by tile (T^d cells).  A spreading work
// item is a chunk of points of one tile; it produces the tile's 16^d patch as a matrix
// product on the MFMA units and writes it once to global memory.  A fold pass sums the
// overlapping patches of neighbouring tiles into the box grid in a fixed order -- no
// atomics anywhere (gfx950 executes LDS float atomics lane by lane, far below LDS
// read rates), and the grid does not depend on which other jobs share a launch.
// Interpolation keeps a tile's patch of the result grid in registers and contracts it
// with the points' windows, again on the MFMA units.
#include "nfft_device.h"

namespace mot {

// ---------------------------------------------------------------------------------------
// Binning

__global__ void bin_cells_kernel(int d, int64_t npts, const double *__restrict__ x, double s0,
                                 double s1, double s2, double o0, double o1, double o2, int n,
                                 int T, int32_t *__restrict__ cell, int32_t *__restrict__ tile)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npts) return;
    const double sc[3] = {s0, s1, s2}, oc[3] = {o0, o1, o2};
    int tpd = (n + T - 1) / T;
    int32_t t = 0;
    for (int c = 0; c < d; ++c) {
        // u = x*s + o with both operations rounded separately (no FMA contraction)
        double u = __dadd_rn(__dmul_rn(x[i * d + c], sc[c]), oc[c]);
        double f = floor(u);
        int ci = !(f >= 0.0) ? 0 : (f > (double)(n - 1) ? n - 1 : (int)f);
        cell[i * d + c] = ci;
        t = t * tpd + ci / T;
    }
    tile[i] = t;
}

hipError_t launch_bin_cells(int d, int64_t npts, const double *x, double s0, double s1, double s2,
                            double o0, double o1, double o2, int n, int T, int32_t *cell,
                            int32_t *tile, hipStream_t st)
{
    if (npts == 0) return hipSuccess;
    int blocks = (int)((npts + 255) / 256);
    hipLaunchKernelGGL(bin_cells_kernel, dim3(blocks), dim3(256), 0, st, d, npts, x, s0, s1, s2,
                       o0, o1, o2, n, T, cell, tile);
    return hipGetLastError();
}

// Stable sort by tile: bitonic sort of the unique 64-bit keys (tile << 32 | index).  With
// a sub-key (cell != nullptr) the key is ((tile << kSubBits | r) << 32 | index), where r
// is the point's tile-relative cell in dimension sub_dim: points of a tile then come in
// ascending r, ties in index order.
constexpr int kSubBits = 4;

__global__ void make_keys_kernel(int64_t npts, int64_t npad, const int32_t *__restrict__ tile,
                                 const int32_t *__restrict__ cell, int d, int sub_dim, int T,
                                 uint64_t *__restrict__ keys)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= npad) return;
    uint64_t hi = i < npts ? (uint64_t)(uint32_t)tile[i] : 0;
    if (cell != nullptr && i < npts) hi = (hi << kSubBits) | (uint64_t)(cell[i * d + sub_dim] % T);
    keys[i] = i < npts ? (hi << 32) | (uint64_t)i : ~0ull;
}

// The bitonic network over npad keys: blocks of kSortBlock keys in LDS, wider strides in global
// memory, two to a launch.  A sort of this size is bound by its launches and barriers (npad = 32768:
// 17 launches, 22 with one stride to a launch).  Wider blocks save launches but leave most of the
// chip idle in the long chain of strides inside a block: creating a tree plan of 46000 points and
// sweeping it took 10.1 ms with 4096 or 2048 keys, 9.7 with 1024.
constexpr int kSortBlock = 1024, kSortThreads = 512;

__device__ __forceinline__ void order_keys(uint64_t &a, uint64_t &b, bool up)
{
    const uint64_t x = a, y = b;
    const bool swap = (x > y) == up;
    a = swap ? y : x;
    b = swap ? x : y;
}

// The strides j and, with TWO, j / 2 of stage k in global memory: a thread holds the two or four keys
// that they join.
template <bool TWO>
__global__ __launch_bounds__(256) void bitonic_global_kernel(uint64_t *keys, int64_t threads, int64_t k, int64_t j)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= threads) return;
    const int64_t s = TWO ? j / 2 : j;                            // the smaller stride
    const int64_t i = (q & ~(s - 1)) * (TWO ? 4 : 2) + (q & (s - 1));  // s is a power of two
    const bool up = (i & k) == 0;
    if constexpr (TWO) {
        uint64_t a = keys[i], b = keys[i + s], c = keys[i + 2 * s], d = keys[i + 3 * s];
        order_keys(a, c, up);
        order_keys(b, d, up);
        order_keys(a, b, up);
        order_keys(c, d, up);
        keys[i] = a;
        keys[i + s] = b;
        keys[i + 2 * s] = c;
        keys[i + 3 * s] = d;
    } else {
        uint64_t a = keys[i], b = keys[i + s];
        order_keys(a, b, up);
        keys[i] = a;
        keys[i + s] = b;
    }
}

// Stages k_lo .. k_hi inside LDS, from stride min(k, nb) / 2 on; a block holds nb <= kSortBlock keys.
// A wavefront's pairs of strides up to 64 lie in its own 128 keys, so those strides need no
// barrier between them.
__global__ __launch_bounds__(kSortThreads) void bitonic_local_kernel(uint64_t *keys, int nb, int64_t k_lo, int64_t k_hi)
{
    __shared__ uint64_t sk[kSortBlock];
    const int64_t base = (int64_t)blockIdx.x * nb;
    for (int t = threadIdx.x; t < nb; t += kSortThreads) sk[t] = keys[base + t];
    __syncthreads();
    for (int64_t k = k_lo; k <= k_hi; k <<= 1) {
        for (int j = (int)(k < nb ? k : nb) / 2; j > 0; j >>= 1) {
            for (int q = threadIdx.x; q < nb / 2; q += kSortThreads) {
                const int i = 2 * (q & ~(j - 1)) + (q & (j - 1));
                order_keys(sk[i], sk[i + j], ((base + i) & k) == 0);
            }
            // the next stride: j / 2, or the next stage's widest
            if (j > 64 || (j == 1 && k >= 128 && k < k_hi))
                __syncthreads();
            else
                wave_sync();
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nb; t += kSortThreads) keys[base + t] = sk[t];
}

// perm[i] = index of the i-th sorted key (i < npts); tile_off[t] = first sorted position
// whose tile is >= t (t <= ntiles), by binary search over the sorted keys, so empty
// stretches of tiles cost nothing extra.
__global__ void keys_to_perm_kernel(int64_t npts, int64_t ntiles, const uint64_t *__restrict__ keys,
                                    int shift, int32_t *__restrict__ perm, int32_t *__restrict__ tile_off)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < npts) perm[i] = (int32_t)(keys[i] & 0xffffffffull);
    if (tile_off != nullptr && i <= ntiles) {
        int64_t lo = 0, hi = npts;  // first position with tile >= i in [lo, hi]
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)(keys[mid] >> shift) < i)
                lo = mid + 1;
            else
                hi = mid;
        }
        tile_off[i] = (int32_t)lo;
    }
}

// Sorted ranges of the tiles of an active box after stable_tile_sort (whose sorted keys are
// still in the scratch buffer): box tile b (row-major over nt[0] x nt[1] x nt[2] tiles,
// coordinate 0 slowest, offset by t0 in the grid of tpd tiles per dimension) holds sorted
// positions [lo[b], hi[b]).  Binary searches as in keys_to_perm_kernel.
__global__ void box_tile_ranges_kernel(int64_t npts, const uint64_t *__restrict__ keys, int shift, int d, int tpd,
                                       int t00, int t01, int t02, int nt0, int nt1, int nt2, int64_t nbox,
                                       int32_t *__restrict__ lo, int32_t *__restrict__ hi)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nbox) return;
    const int t0[3] = {t00, t01, t02}, nt[3] = {nt0, nt1, nt2};
    int tc[3] = {0, 0, 0};
    int64_t rem = b;
    for (int c = d - 1; c >= 0; --c) {
        tc[c] = (int)(rem % nt[c]);
        rem /= nt[c];
    }
    int64_t gt = 0;
    for (int c = 0; c < d; ++c) gt = gt * tpd + (t0[c] + tc[c]);
    int64_t out[2];
    for (int q = 0; q < 2; ++q) {
        int64_t a = 0, e = npts;
        while (a < e) {
            const int64_t mid = (a + e) >> 1;
            if ((int64_t)(keys[mid] >> shift) < gt + q)
                a = mid + 1;
            else
                e = mid;
        }
        out[q] = a;
    }
    lo[b] = (int32_t)out[0];
    hi[b] = (int32_t)out[1];
}

hipError_t launch_box_tile_ranges(int64_t npts, const void *scratch, bool sub_keyed, int d, int tpd, const int *t0,
                                  const int *nt, int32_t *lo, int32_t *hi, hipStream_t st)
{
    int64_t nbox = 1;
    for (int c = 0; c < d; ++c) nbox *= nt[c];
    if (nbox == 0) return hipSuccess;
    hipLaunchKernelGGL(box_tile_ranges_kernel, dim3((unsigned)((nbox + 255) / 256)), dim3(256), 0, st, npts,
                       (const uint64_t *)scratch, sub_keyed ? 32 + kSubBits : 32, d, tpd, t0[0], d > 1 ? t0[1] : 0,
                       d > 2 ? t0[2] : 0, nt[0], d > 1 ? nt[1] : 1, d > 2 ? nt[2] : 1, nbox, lo, hi);
    return hipGetLastError();
}

size_t stable_tile_sort_scratch(int64_t npts, int64_t /*ntiles*/)
{
    int64_t npad = 1024;
    while (npad < npts) npad <<= 1;
    return (size_t)npad * sizeof(uint64_t);
}

hipError_t stable_tile_sort(int64_t npts, const int32_t *tile, int64_t ntiles, int32_t *perm,
                            int32_t *tile_off, void *scratch, size_t scratch_bytes, hipStream_t st,
                            const int32_t *cell, int d, int sub_dim, int T)
{
    int64_t npad = 1024;
    while (npad < npts) npad <<= 1;
    if (scratch_bytes < (size_t)npad * sizeof(uint64_t)) return hipErrorInvalidValue;
    if (cell != nullptr && (T > (1 << kSubBits) || sub_dim < 0 || sub_dim >= d ||
                            ntiles >= ((int64_t)1 << (32 - kSubBits))))
        return hipErrorInvalidValue;
    uint64_t *keys = (uint64_t *)scratch;
    int blocks = (int)((npad + 255) / 256);
    hipLaunchKernelGGL(make_keys_kernel, dim3(blocks), dim3(256), 0, st, npts, npad, tile, cell, d, sub_dim,
                       T, keys);
    const int nb = (int)std::min<int64_t>(npad, kSortBlock);
    const dim3 lblocks((unsigned)(npad / nb));
    hipLaunchKernelGGL(bitonic_local_kernel, lblocks, dim3(kSortThreads), 0, st, keys, nb, (int64_t)2, (int64_t)nb);
    for (int64_t k = 2 * (int64_t)nb; k <= npad; k <<= 1) {
        for (int64_t j = k / 2; j >= nb;) {
            if (j / 2 >= nb) {
                hipLaunchKernelGGL(bitonic_global_kernel<true>, dim3((unsigned)(npad / 4 / 256)), dim3(256), 0, st, keys,
                                   npad / 4, k, j);
                j /= 4;
            } else {
                hipLaunchKernelGGL(bitonic_global_kernel<false>, dim3((unsigned)(npad / 2 / 256)), dim3(256), 0, st,
                                   keys, npad / 2, k, j);
                j /= 2;
            }
        }
        hipLaunchKernelGGL(bitonic_local_kernel, lblocks, dim3(kSortThreads), 0, st, keys, nb, k, k);
    }
    const int64_t nthr = std::max<int64_t>(npts, ntiles + 1);
    int pblocks = (int)((nthr + 255) / 256);
    hipLaunchKernelGGL(keys_to_perm_kernel, dim3(pblocks), dim3(256), 0, st, npts, ntiles, keys,
                       cell != nullptr ? 32 + kSubBits : 32, perm, tile_off);
    return hipGetLastError();
}

constexpr int kPatch = 16;  // patch edge T + 2m - 1 in cells

// ---------------------------------------------------------------------------------------
// Kaiser-Bessel window in grid units, normalised to 1 at s = 0:
//   psi(s) = (m / r) sinh(b r) / sinh(b m),  r = sqrt(m^2 - s^2),  |s| <= m,
// b = pi (2 - 1/sigma).  Its Fourier transform is I0(m sqrt(b^2 - w^2)), which the host
// uses for the spectral multiplier.
//
// Window rows.  A tile holds T = 17 - 2m cells per dimension, so the patch of cells its
// points touch is exactly 16 wide (T + 2m - 1).  For a point with tile-relative cell r
// and fractional offset f in dimension c, its row is the 16-vector
//   w_c[q] = psi(f + m - 1 + r - q)  if 0 <= q - r < 2m,  else 0,
// the weights of patch cells q = 0..15.  The rows depend on the points only, so they are
// evaluated once per plan in FP64 (rounded to FP32) and stored per point in binned
// order, rows[(i d + c) 16 + q]: every later product reads them instead of
// re-evaluating the window.
__global__ void window_rows_kernel(int d, int64_t npts, const double *__restrict__ pts, double s,
                                   double o0, double o1, double o2, int T, int m, double b,
                                   double inv_sinh_bm, float *__restrict__ rows)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= npts * d) return;
    const int64_t i = t / d;
    const int c = (int)(t - i * d);
    const double oc = c == 0 ? o0 : (c == 1 ? o1 : o2);
    // the binning's operations, so the cell is the one the point was sorted by
    const double u = __dadd_rn(__dmul_rn(pts[i * d + c], s), oc);
    const double fl = floor(u);
    const double f = u - fl;
    const int r = (int)fl % T;
    const double dm = m;
    float w[kPatch];
#pragma unroll
    for (int q = 0; q < kPatch; ++q) {
        const int j = q - r;
        float val = 0.0f;
        if (j >= 0 && j < 2 * m) {
            const double a = f + (dm - 1.0 - j);
            const double rr = sqrt(fmax(dm * dm - a * a, 0.0));
            const double br = b * rr;
            // sinh(b r) / r, with its series near r = 0 (the support edge)
            const double sr = br < 1e-4 ? b * (1.0 + br * br / 6.0) : sinh(br) / rr;
            val = (float)(dm * sr * inv_sinh_bm);
        }
        w[q] = val;
    }
    float4 *dst = reinterpret_cast<float4 *>(rows + t * kPatch);
#pragma unroll
    for (int q = 0; q < kPatch / 4; ++q) dst[q] = make_float4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
}

hipError_t launch_window_rows(int d, int64_t npts, const double *pts, double s, const double *o, int T,
                              int m, double b, float *rows, hipStream_t st)
{
    if (npts == 0) return hipSuccess;
    const int64_t work = npts * d;
    const int blocks = (int)((work + 255) / 256);
    hipLaunchKernelGGL(window_rows_kernel, dim3(blocks), dim3(256), 0, st, d, npts, pts, s, o[0],
                       d > 1 ? o[1] : 0.0, d > 2 ? o[2] : 0.0, T, m, b, 1.0 / sinh(b * m), rows);
    return hipGetLastError();
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int source_exponent(const ProdJob &J)
{
    const int e = *gp(J.v_exp);
    return e == INT32_MIN ? 0 : e;
}

// ---------------------------------------------------------------------------------------
// Spreading (a2) as a dense tile contraction on FP32 MFMA.
//
// For a chunk of points of one tile, the patch is
//   G[a][(b,c')] = sum_p X[a][p] Y[p][(b,c')],   X[a][p] = v_p w_0,p[a],
//   Y[p][(b,c')] = w_1,p[b] w_2,p[c'],
// a 16 x 256 x P product done with v_mfma_f32_16x16x4_f32: a step takes 4 points (the K
// dimension), one MFMA per b (16 output tiles of 16 x 16 over (a, c')).  Lane l holds
// A[a = l % 16][k = l / 16] and B[k = l / 16][c' = l % 16]; accumulator r of tile b holds
// G[a = 4 (l / 16) + r][b][c' = l % 16].  In 2-D the product is one 16 x 16 tile per step,
// in 1-D a plain sum over points.
//
// A block of kSpreadWaves wavefronts takes one chunk, which owns its patch: no atomics.
// In 1-D and 2-D wave w takes the 4-point steps w, w + kSpreadWaves, ... and the wave
// partials are added through LDS in a fixed order (pairwise halving); in 3-D the waves
// split the b tiles instead (spread3_kernel).  Either way a patch is the same whatever
// else shares the launch.
constexpr int kSpreadWaves = 4;
constexpr int kInterpWaves = 4;

// Points are staged through LDS kStage at a time: all threads of the block copy the
// stage's window rows (contiguous in memory for consecutive points) with 16-byte loads,
// one stage ahead of the MFMA work, so the row stream overlaps the contractions.
constexpr int kStage = 64;

// Staged 3-D window rows: a point's 48 floats are its rows for dimensions 0, 1, 2.  The
// dimension-1 row w_1[0..15] is stored transposed, position 4 i + q holding w_1[4 q + i], so
// that the four values w_1[w], w_1[w + 4], w_1[w + 8], w_1[w + 12] a wavefront w takes are
// one 16-byte read at position 4 w.  idx is the 16-byte piece (12 per point).
__device__ __forceinline__ void store_piece3(unsigned char *buf, int idx, f32x4 v)
{
    const int piece = idx % 12;
    if (piece >= 4 && piece < 8) {
        float *row = reinterpret_cast<float *>(buf) + (idx - piece + 4) * 4;
        const int q = piece - 4;
        row[q] = v[0];
        row[4 + q] = v[1];
        row[8 + q] = v[2];
        row[12 + q] = v[3];
    } else {
        reinterpret_cast<f32x4 *>(buf)[idx] = v;
    }
}

template <int D, bool WITH_V>
struct Stage {
    static constexpr int kRow4 = kStage * D * kPatch / 4;  // 16-byte row pieces per stage
    static constexpr int kPer = (kRow4 + 255) / 256;        // per thread (256 threads)
    static constexpr int kBytes = kRow4 * 16 + (WITH_V ? kStage * 4 : 0);
    f32x4 r[kPer];
    double v, w;  // source value and factor, joined only when stored, so that the loads stay in flight

    // Registers <- global: points pb .. pb + kStage - 1 (zeros past p1), and for
    // spreading the source values.
    __device__ __forceinline__ void load(const float *rows, const double *vsrc, const double *wsrc, int64_t pb,
                                         int64_t p1)
    {
        const MOT_GLOBAL f32x4 *g = reinterpret_cast<const MOT_GLOBAL f32x4 *>(gp(rows)) + pb * (D * 4);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int idx = threadIdx.x + 256 * i;
            r[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (idx < kRow4 && pb + idx / (D * 4) < p1) r[i] = g[idx];
        }
        if constexpr (WITH_V) {
            v = 0.0;
            w = 1.0;
            const int64_t p = pb + threadIdx.x;
            if (threadIdx.x < kStage && p < p1) {
                v = gp(vsrc)[p];
                if (wsrc) w = gp(wsrc)[p];
            }
        }
    }
    // LDS <- registers; source values are stored as FP32 v 2^-e.  In 3-D the dimension-1
    // row of a point is stored transposed (see store_rows3).
    __device__ __forceinline__ void store(unsigned char *buf, int e) const
    {
        f32x4 *rl = reinterpret_cast<f32x4 *>(buf);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int idx = threadIdx.x + 256 * i;
            if (idx < kRow4) {
                if constexpr (D == 3)
                    store_piece3(buf, idx, r[i]);
                else
                    rl[idx] = r[i];
            }
        }
        if constexpr (WITH_V)
            if (threadIdx.x < kStage)
                reinterpret_cast<float *>(buf + kRow4 * 16)[threadIdx.x] = (float)ldexp(v * w, -e);
    }
};

template <int D>
__global__ __launch_bounds__(64 * kSpreadWaves, 4) void spread_kernel(const ProdJob *__restrict__ jobs,
                                                                   const int2 *__restrict__ items,
                                                                   int n_items)
{
    static_assert(kSpreadWaves == 4, "staging assumes 256 threads");
    static_assert(D < 3, "3-D spreading is spread3_kernel");
    using St = Stage<D, true>;
    constexpr int kRed = (kSpreadWaves / 2) * 64 * 16;
    constexpr int kSmem = 2 * St::kBytes > kRed ? 2 * St::kBytes : kRed;
    __shared__ __align__(16) unsigned char smem[kSmem];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int64_t p0 = gp(J.src_chunk_start)[itm.y], p1 = gp(J.src_chunk_start)[itm.y + 1];
        const int e = source_exponent(J);
        const int nstages = (int)((p1 - p0 + kStage - 1) / kStage);
        f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        St stg;
        stg.load(J.src_win, J.v, J.v_mul, p0, p1);
        stg.store(smem, e);
        __syncthreads();
        for (int k = 0; k < nstages; ++k) {
            const bool more = k + 1 < nstages;
            if (more) stg.load(J.src_win, J.v, J.v_mul, p0 + (int64_t)(k + 1) * kStage, p1);
            const unsigned char *buf = smem + (k & 1) * St::kBytes;
            const float *rl = reinterpret_cast<const float *>(buf);
            const float *vl = reinterpret_cast<const float *>(buf + St::kRow4 * 16);
            // this wave's 4-point steps of the stage: points 4 j + lane group, j = wave + 4 i
#pragma unroll 1
            for (int i = 0; i < kStage / 16; ++i) {
                const int pi = 4 * (wave + 4 * i) + lk;
                const float *row = rl + pi * (D * kPatch);
                const float x = vl[pi] * row[li];
                if constexpr (D == 2)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, row[kPatch + li], acc, 0, 0, 0);
                else
                    acc[0] += x;
            }
            if (more) stg.store(smem + ((k + 1) & 1) * St::kBytes, e);
            __syncthreads();
        }
        if constexpr (D == 1) {
            // sum over the four points of a step (lane groups), then over waves
            float a1 = acc[0];
            a1 += lane_xor(a1, 16);
            a1 += lane_xor(a1, 32);
            acc[0] = a1;
        }
        // wave partials: wave w < half adds wave w + half, halving until wave 0 holds the
        // patch (the staging buffers are free: the last stage ended with a barrier)
        f32x4(*red)[64] = reinterpret_cast<f32x4(*)[64]>(smem);
#pragma unroll
        for (int half = kSpreadWaves / 2; half >= 1; half >>= 1) {
            if (wave >= half && wave < 2 * half) red[wave - half][lane] = acc;
            __syncthreads();
            if (wave < half) acc += red[wave][lane];
            __syncthreads();
        }
        if (wave == 0) {
            MOT_GLOBAL float *out = gp(J.patches) + (int64_t)itm.y * (D == 2 ? 256 : 16);
            if constexpr (D == 2) {
#pragma unroll
                for (int r = 0; r < 4; ++r) out[(4 * lk + r) * 16 + li] = acc[r];
            } else {
                if (lk == 0) out[li] = acc[0];
            }
        }
    }
}

// 3-D spreading: the 16 b tiles are split over the block's waves.  Wave w accumulates
// tiles b = w, w + 4, w + 8, w + 12 over every point of the chunk (one MFMA per tile and
// 4-point step, in point order), so a wave holds 4 accumulators per job rather than 16, no
// partial patches are combined, and every wave writes its own quarter of the patch.  Any
// 2m = 12 consecutive b values hold three of each wave's four, so when the points of a step
// share their window support every wave skips one step and none waits at the stage
// barrier for the others (with quarters of consecutive b values the two middle waves
// never skip).
//
// An item is (job_0, .., job_{G-1}, chunk): G jobs that spread different values from the
// same points (the down products of a node's children).  They share the chunk's window
// rows, so the rows are staged once, and the B operand w_1,p[b] w_2,p[c'] and the test for
// a zero step are formed once for G MFMAs.  Each job's patch is accumulated exactly as it
// would be on its own.
template <int G>
struct SpreadStage3 {
    static constexpr int kRow4 = kStage * 3 * kPatch / 4;  // 16-byte row pieces per stage
    static constexpr int kPer = (kRow4 + 255) / 256;        // per thread (256 threads)
    static constexpr int kBytes = kRow4 * 16 + G * kStage * 4;
    f32x4 r[kPer];
    double v, w;  // value and factor of job q = threadIdx.x / kStage (the wave), joined only when stored

    // Registers <- global: points pb .. pb + kStage - 1 (zeros past p1); wave q < G loads
    // job q's values from vq (the job's pointer, selected by the caller), factors from wq if any.
    __device__ __forceinline__ void load(const float *rows, const double *vq, const double *wq, int64_t pb,
                                         int64_t p1)
    {
        const MOT_GLOBAL f32x4 *g = reinterpret_cast<const MOT_GLOBAL f32x4 *>(gp(rows)) + pb * 12;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int idx = threadIdx.x + 256 * i;
            r[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (idx < kRow4 && pb + idx / 12 < p1) r[i] = g[idx];
        }
        v = 0.0;
        w = 1.0;
        const int64_t p = pb + (threadIdx.x % kStage);
        if (threadIdx.x / kStage < G && p < p1) {
            v = gp(vq)[p];
            if (wq) w = gp(wq)[p];
        }
    }
    // LDS <- registers (dimension-1 rows transposed, store_piece3); job q's values are
    // stored as FP32 v 2^-eq.
    __device__ __forceinline__ void store(unsigned char *buf, int eq) const
    {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int idx = threadIdx.x + 256 * i;
            if (idx < kRow4) store_piece3(buf, idx, r[i]);
        }
        if (threadIdx.x / kStage < G)
            reinterpret_cast<float *>(buf + kRow4 * 16)[threadIdx.x] = (float)ldexp(v * w, -eq);
    }
};

template <int G>
__global__ __launch_bounds__(64 * kSpreadWaves, G == 1 ? 6 : (G == 2 ? 5 : 4)) void spread3_kernel(const ProdJob *__restrict__ jobs,
                                                                                 const int4 *__restrict__ items,
                                                                                 int n_items)
{
    static_assert(kSpreadWaves == 4 && kStage == 64 && G >= 1 && G <= 3,
                  "one wave per group of 4 b tiles and per job's stage values; up to 3 jobs");
    using St = SpreadStage3<G>;
    __shared__ __align__(16) unsigned char smem[2 * St::kBytes];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const int c = itm.w;
        const ProdJob &J = jobs[itm.x];  // the points, shared by the item's jobs
        const int64_t p0 = gp(J.src_chunk_start)[c], p1 = gp(J.src_chunk_start)[c + 1];
        // wave q < G stages job q's values: its pointer and exponent, selected by wave
        const int jq = wave == 0 ? itm.x : (wave == 1 ? itm.y : itm.z);
        const int q_job = wave < G ? jq : itm.x;
        const double *vq = jobs[q_job].v;
        const int eq = source_exponent(jobs[q_job]);
        const int nstages = (int)((p1 - p0 + kStage - 1) / kStage);
        f32x4 acc[G][4];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[g][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        St stg;
        stg.load(J.src_win, vq, J.v_mul, p0, p1);
        stg.store(smem, eq);
        __syncthreads();
        for (int k = 0; k < nstages; ++k) {
            const bool more = k + 1 < nstages;
            if (more) stg.load(J.src_win, vq, J.v_mul, p0 + (int64_t)(k + 1) * kStage, p1);
            const unsigned char *buf = smem + (k & 1) * St::kBytes;
            const float *rl = reinterpret_cast<const float *>(buf);
            const float *vl = reinterpret_cast<const float *>(buf + St::kRow4 * 16);
#pragma unroll 2
            for (int j = 0; j < kStage / 4; ++j) {
                const int pi = 4 * j + lk;  // point of lane group lk in step j
                const float *row = rl + pi * (3 * kPatch);
                const float w0 = row[li];
                float x[G];
#pragma unroll
                for (int g = 0; g < G; ++g) x[g] = vl[g * kStage + pi] * w0;
                const float w2 = row[2 * kPatch + li];
                // w_1,p[b] for the wave's b = wave + 4 u (one read of the transposed row)
                const f32x4 w1 = reinterpret_cast<const f32x4 *>(row + kPatch)[wave];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    // B is zero when b = w + 4 u is outside the window of all four points:
                    // the products would add exact zeros
                    if (__any(w1[u] != 0.0f)) {
                        const float bu = w1[u] * w2;
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[g], bu, acc[g][u], 0, 0, 0);
                    }
            }
            if (more) stg.store(smem + ((k + 1) & 1) * St::kBytes, eq);
            __syncthreads();
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int jg = g == 0 ? itm.x : (g == 1 ? itm.y : itm.z);
            MOT_GLOBAL float *out = gp(jobs[jg].patches) + (int64_t)c * 4096;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) out[((4 * lk + r) * 16 + wave + 4 * u) * 16 + li] = acc[g][u][r];
        }
    }
}

// Fold (a2, second half): box grid cell g = sum of the patches covering it in a fixed order
// (3-D: leading tile by leading tile; the covering tiles' first chunks in tile order, then
// their second chunks, and so on).  One thread folds one
// cell; an item is kFoldCellsPerItem consecutive cells of the box in row-major order
// (lines of the last dimension back to back, so every lane has a cell even when a line
// is shorter than a wavefront); item = (job, first cell).  The job's tile -> chunk table
// is staged in LDS when it fits, so the chunk lookups of a thread's covering tiles cost
// LDS rather than global latency.
// PARTS = 2: in 3-D the leading tiles that cover a cell go to two threads in turn, as each is a
// sequence of dependent lookups and loads that one thread waits for (30^3 box, tiles of 7 cells, one
// or two jobs: 12.6 us with one thread to a cell, 7.7 here, 8.8 with four).  A launch that fills
// the chip is bound by its loads and gains nothing (nine jobs on a 41^3 box: 27.2 us, 40 with four), so
// the split ends at kFoldSplitItems items.
constexpr int kFoldSplitItems = 1024;

// One item of the fold.
template <int D, int PARTS, class Tab>
__device__ __forceinline__ void fold_item(const ProdJob &J, int f0, Tab tch, float *s_part)
{
    const int Ll = J.L[D - 1];
    const int nl = D == 3 ? J.L[0] * J.L[1] : (D == 2 ? J.L[0] : 1);
    const int cell = (int)threadIdx.x % kFoldCellsPerItem, part = (int)threadIdx.x / kFoldCellsPerItem;
    if (D < 3 && part > 0) return;
    const int f = D == 3 && PARTS == 2 ? min(f0 + cell, nl * Ll - 1) : f0 + cell;
    if (f >= nl * Ll) return;
    const int line = f / Ll, g = f - line * Ll;
    int gu[2] = {0, 0};  // line coordinates in the leading dimensions
    if (D == 3) {
        gu[0] = line / J.L[1];
        gu[1] = line - gu[0] * J.L[1];
    } else if (D == 2) {
        gu[0] = line;
    }
    if constexpr (D == 3 && PARTS == 2) {
        const float sum = fold_cell<D, PARTS>(J, gu, g, tch, part);
        if (part > 0) s_part[cell] = sum;
        __syncthreads();
        if (part == 0 && f0 + cell < nl * Ll) gp(J.grid)[f] = sum + s_part[cell];
    } else {
        gp(J.grid)[f] = fold_cell<D>(J, gu, g, tch);
    }
}

// D = 0: every item takes its job's own d (batches of plans of several dimensions).
template <int D, int PARTS>
__global__ __launch_bounds__(kFoldCellsPerItem *PARTS) void fold_kernel(const ProdJob *__restrict__ jobs,
                                                                 const int2 *__restrict__ items, int n_items)
{
    __shared__ int32_t s_tab[kFoldTab];
    __shared__ float s_part[PARTS == 2 ? kFoldCellsPerItem : 1];
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int d = D > 0 ? D : J.d;
        int ntab = 1;
        for (int c = 0; c < d; ++c) ntab *= J.ntile[c];
        ++ntab;
        const bool staged = ntab <= kFoldTab;
        if (staged) {
            __syncthreads();  // the previous item's reads of the table are done
            const MOT_GLOBAL int32_t *tg = gp(J.src_tile_chunks);
            for (int i = threadIdx.x; i < ntab; i += blockDim.x) s_tab[i] = tg[i];
            __syncthreads();
        } else if (PARTS == 2) {
            __syncthreads();  // the previous item's reads of the partial sums are done
        }
        const int32_t *lt = static_cast<const int32_t *>(s_tab);
        const MOT_GLOBAL int32_t *gt = gp(J.src_tile_chunks);
        if (d == 3) {
            if (staged) fold_item<3, PARTS>(J, itm.y, lt, s_part); else fold_item<3, PARTS>(J, itm.y, gt, s_part);
        } else if (d == 2) {
            if (staged) fold_item<2, PARTS>(J, itm.y, lt, s_part); else fold_item<2, PARTS>(J, itm.y, gt, s_part);
        } else {
            if (staged) fold_item<1, PARTS>(J, itm.y, lt, s_part); else fold_item<1, PARTS>(J, itm.y, gt, s_part);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Interpolation (a6) as the transposed contraction on FP32 MFMA.
//
// For 16 target points of one tile and the 16^d patch G of the result grid over the
// tile, Z[a][p] = sum_{(b,c')} G[a][(b,c')] Y[(b,c')][p] with Y[(b,c')][p] =
// w_1,p[b] w_2,p[c'], then beta_p = sum_a w_0,p[a] Z[a][p].  Step s of the 64-step MFMA
// chain covers b = s / 4 and, for lane group g = l / 16, c' = 4 g + s % 4: lane l holds
// A[a = l % 16][k] = G[a][b][c'] and B[k][p = l % 16] = w_1,p[b] w_2,p[c'].  The grid
// values are the same for every point of the tile, so they stay in registers for the whole
// chunk.  Accumulator r holds Z[a = 4 g + r][p = l % 16], so each lane owns one point: the
// last contraction over a takes the lane's four a and then adds the four lane groups.  In
// 2-D the chain has 4 steps (k = b = 4 g + s); in 1-D one lane takes one point.
// out = 2^e beta, e the exponent the source was scaled by.
//
// A block of kInterpWaves wavefronts takes one chunk.  In 2-D wave w takes the 16-point
// groups w, w + kInterpWaves, ... (one per stage), in 1-D 64-point groups; 3-D
// interpolation splits the b values over the waves instead (interp3_kernel).
template <int D>
__global__ __launch_bounds__(64 * kInterpWaves, 4) void interp_kernel(const ProdJob *__restrict__ jobs,
                                                                   const int2 *__restrict__ items,
                                                                   int n_items)
{
    static_assert(kInterpWaves == 4 && kStage == 16 * kInterpWaves, "one 16-point group per wave and stage");
    static_assert(D < 3, "3-D interpolation is interp3_kernel");
    constexpr int NB = D == 2 ? 4 : 16;  // B values per lane
    using St = Stage<D, false>;
    __shared__ __align__(16) unsigned char smem[D == 1 ? 16 : 2 * St::kBytes];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int T = J.T;
        int tc[3] = {0, 0, 0};
        {
            int rem = gp(J.tgt_chunk_tile)[itm.y];
#pragma unroll
            for (int c = D - 1; c >= 0; --c) {
                tc[c] = rem % J.ntile[c];
                rem /= J.ntile[c];
            }
        }
        const MOT_GLOBAL float *grid = gp(J.grid);
        float Bv[NB];
        if constexpr (D == 2) {
            const int64_t base = (int64_t)(tc[0] * T + li) * J.L[1] + tc[1] * T + 4 * lk;
#pragma unroll
            for (int s = 0; s < 4; ++s) Bv[s] = grid[base + s];
        } else {
#pragma unroll
            for (int a = 0; a < 16; ++a) Bv[a] = grid[tc[0] * T + a];
        }
        const int e = source_exponent(J);
        const int64_t p0 = gp(J.tgt_chunk_start)[itm.y], p1 = gp(J.tgt_chunk_start)[itm.y + 1];
        MOT_GLOBAL double *out = gp(J.out);
        if constexpr (D == 1) {
            const MOT_GLOBAL f32x4 *rows = reinterpret_cast<const MOT_GLOBAL f32x4 *>(gp(J.tgt_win));
            for (int64_t p = p0 + threadIdx.x; p < p1; p += 64 * kInterpWaves) {
                float s = 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 w = rows[p * 4 + q];
                    s += w[0] * Bv[4 * q] + w[1] * Bv[4 * q + 1] + w[2] * Bv[4 * q + 2] + w[3] * Bv[4 * q + 3];
                }
                out[p] = ldexp((double)s, e);
            }
        } else {
            const int nstages = (int)((p1 - p0 + kStage - 1) / kStage);
            St stg;
            stg.load(J.tgt_win, nullptr, nullptr, p0, p1);
            stg.store(smem, 0);
            __syncthreads();
            for (int k = 0; k < nstages; ++k) {
                const bool more = k + 1 < nstages;
                if (more) stg.load(J.tgt_win, nullptr, nullptr, p0 + (int64_t)(k + 1) * kStage, p1);
                const float *rl = reinterpret_cast<const float *>(smem + (k & 1) * St::kBytes);
                // this wave's group: stage points 16 wave .. 16 wave + 15
                const float *grow = rl + (16 * wave) * (D * kPatch);
                const float *row = grow + li * (D * kPatch);  // point l % 16
                // grid values as the A operand, window values as B: acc[r] = Z[a = 4 lk + r][p]
                // for the lane's point p = l % 16
                f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                const f32x4 wb = reinterpret_cast<const f32x4 *>(row + kPatch)[lk];
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[0], wb[0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[1], wb[1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[2], wb[2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[3], wb[3], acc, 0, 0, 0);
                // beta_p = sum_a w_0,p[a] Z[a][p]: the lane's four a, then the four lane groups
                const f32x4 wx = reinterpret_cast<const f32x4 *>(row)[lk];
                float z = (acc[0] * wx[0] + acc[1] * wx[1]) + (acc[2] * wx[2] + acc[3] * wx[3]);
                z += lane_xor(z, 16);
                z += lane_xor(z, 32);
                const int64_t p = p0 + (int64_t)k * kStage + 16 * wave + li;
                if (lk == 0 && p < p1) out[p] = ldexp((double)z, e);
                if (more) stg.store(smem + ((k + 1) & 1) * St::kBytes, 0);
                __syncthreads();
            }
        }
    }
}

// 3-D interpolation with the 16 b values of the contraction split over the block's waves.
// Wave w holds B only for b = w, w + 4, w + 8, w + 12 (16 registers rather than 64; a
// twelve-wide window covers three of each wave's four b, so the waves skip alike) and takes
// all four 16-point groups of a stage.  The grid values are the MFMA's A operand and the
// window products its B operand, so for group g lane l's accumulators give
// Z_w[a = 4 (l / 16) + r][p = 16 g + l % 16], the part of Z from the wave's b values, with
// the point along the lanes.  Each lane weights its four a by the point's w_0,p[a] and the
// four lane groups are added by two lane exchanges; the four waves' partial sums of a
// point are added in wave order through LDS after the stage's barrier, and wave 0 stores
// out = 2^e beta.  (A bound of 5 blocks per CU measured 4 % slower than 6.)
__global__ __launch_bounds__(64 * kInterpWaves, 6) void interp3_kernel(const ProdJob *__restrict__ jobs,
                                                                   const int2 *__restrict__ items,
                                                                   int n_items)
{
    static_assert(kInterpWaves == 4 && kStage == 64, "four 16-point groups and four b quarters per stage");
    using St = Stage<3, false>;
    __shared__ __align__(16) unsigned char smem[2 * St::kBytes];
    __shared__ float zb[2][kInterpWaves][kStage];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const ProdJob &J = jobs[itm.x];
        const int T = J.T;
        int tc[3] = {0, 0, 0};
        {
            int rem = gp(J.tgt_chunk_tile)[itm.y];
#pragma unroll
            for (int c = 2; c >= 0; --c) {
                tc[c] = rem % J.ntile[c];
                rem /= J.ntile[c];
            }
        }
        // A[a = l % 16][k = (b, c')] = G[a][b][c'] for b = wave + 4 bb, c' = 4 lk + s
        const MOT_GLOBAL float *grid = gp(J.grid);
        float Bv[16];
        {
            const int64_t base =
                ((int64_t)(tc[0] * T + li) * J.L[1] + tc[1] * T + wave) * J.L[2] + tc[2] * T + 4 * lk;
#pragma unroll
            for (int bb = 0; bb < 4; ++bb)
#pragma unroll
                for (int s = 0; s < 4; ++s) Bv[4 * bb + s] = grid[base + (int64_t)(4 * bb) * J.L[2] + s];
        }
        const int e = source_exponent(J);
        const int64_t p0 = gp(J.tgt_chunk_start)[itm.y], p1 = gp(J.tgt_chunk_start)[itm.y + 1];
        MOT_GLOBAL double *out = gp(J.out);
        const int nstages = (int)((p1 - p0 + kStage - 1) / kStage);
        St stg;
        stg.load(J.tgt_win, nullptr, nullptr, p0, p1);
        stg.store(smem, 0);
        __syncthreads();
        for (int k = 0; k < nstages; ++k) {
            const bool more = k + 1 < nstages;
            if (more) stg.load(J.tgt_win, nullptr, nullptr, p0 + (int64_t)(k + 1) * kStage, p1);
            const float *rl = reinterpret_cast<const float *>(smem + (k & 1) * St::kBytes);
#pragma unroll 1
            for (int g = 0; g < 4; ++g) {
                const float *row = rl + (16 * g + li) * (3 * kPatch);  // point 16 g + l % 16
                const f32x4 wy = reinterpret_cast<const f32x4 *>(row + kPatch)[wave];  // transposed row
                const f32x4 wz = reinterpret_cast<const f32x4 *>(row + 2 * kPatch)[lk];
                f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int bb = 0; bb < 4; ++bb) {
                    // B is zero when b is outside the window of all 16 points: the four
                    // products would add exact zeros
                    if (!__any(wy[bb] != 0.0f)) continue;
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[4 * bb], wy[bb] * wz[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[4 * bb + 1], wy[bb] * wz[1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[4 * bb + 2], wy[bb] * wz[2], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Bv[4 * bb + 3], wy[bb] * wz[3], acc, 0, 0, 0);
                }
                // acc[r] = Z_w[a = 4 lk + r][p = 16 g + l % 16]: weight by the point's own
                // w_0,p[4 lk .. 4 lk + 3], then add the four lane groups (lanes l ^ 16, l ^ 32)
                const f32x4 wx = reinterpret_cast<const f32x4 *>(row)[lk];
                float z = (acc[0] * wx[0] + acc[1] * wx[1]) + (acc[2] * wx[2] + acc[3] * wx[3]);
                z += lane_xor(z, 16);
                z += lane_xor(z, 32);
                if (lk == 0) zb[k & 1][wave][16 * g + li] = z;
            }
            if (more) stg.store(smem + ((k + 1) & 1) * St::kBytes, 0);
            __syncthreads();
            if (wave == 0) {
                const int64_t p = p0 + (int64_t)k * kStage + lane;
                const float s = ((zb[k & 1][0][lane] + zb[k & 1][1][lane]) + zb[k & 1][2][lane]) + zb[k & 1][3][lane];
                if (p < p1) out[p] = ldexp((double)s, e);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// 1-D and 2-D jobs in groups that share their points (the rows of a circle's matrix): spreading
// and interpolation as matrix products with the window matrix, whose entries are formed once
// for 16 jobs.
//   spreading      G[cell][job] = sum_p W[cell][p] v_p[job]      (K = points)
//   interpolation  beta[p][job] = sum_cell W[cell][p] G[cell][job]  (K = cells)
// with W[(a, c')][p] = w_0,p[a] w_1,p[c'] in 2-D and w_0,p[c'] in 1-D.  As many MFMAs as job by
// job (one per job and four points, a sixteenth in 1-D), but a chunk's rows are staged once for
// 16 jobs (64 in 1-D) and there is one operand product for 16 jobs' MFMA, where the kernels
// above read 128 bytes of rows per point and job from L2: 4000 jobs of 4000 points in 2-D, 184 us
// to spread and 194 us to interpolate, take 99 and 128 us (the values read and the patches
// written are 78 us of the spreading at the card's copy rate, the MFMAs 52 us of each).
//
// A result is one long FP32 sum here, where the kernels above split it over wavefronts and
// dimensions; it is kept as exact by several chains and an order from small terms to large
// (scalings of a circle of 1500 points after three sweeps: 5.4e-8 with one chain for a quarter of a
// row's cells and rows in order, 3.7e-8 as below, 3.8e-8 job by job).
//
// gids: job indices, kGroupJobs1 (1-D) or kGroupJobs2 per group, -1 for absent ones.  An item
// (first group, groups, chunk) takes several groups one after another: the next group's
// values (grid cells) are loaded while the current one is multiplied, which a block of one
// group spends as long waiting for as multiplying (interpolation 195 us with one group per
// block).  The rows of a chunk of one stage are staged once for all of them.
template <int D>
struct GroupShape {
    static constexpr int J = D == 1 ? kGroupJobs1 : kGroupJobs2;  // jobs of a group
    static constexpr int PV = kStage * J / 256;                    // values per thread and stage
    static constexpr int kPitch = J + 4;                           // a row's values (LDS banks)
};

template <int D>
__global__ __launch_bounds__(256, 4) void spread_group_kernel(const ProdJob *__restrict__ jobs,
                                                              const int32_t *__restrict__ gids,
                                                              const int4 *__restrict__ items, int n_items)
{
    using S = GroupShape<D>;
    using St = Stage<D, false>;
    constexpr int NA = D == 2 ? 4 : 1;  // accumulators: 2-D patch rows a = 4 wave + u
    __shared__ __align__(16) unsigned char rows[2][St::kBytes];
    __shared__ float vals[2][kStage * S::kPitch];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const int32_t *gid = gids + (int64_t)itm.x * S::J;
        const int ng = itm.y, c = itm.z;
        const ProdJob &J0 = jobs[gid[0]];  // the points, shared by the groups
        const int64_t p0 = gp(J0.src_chunk_start)[c], p1 = gp(J0.src_chunk_start)[c + 1];
        const int nst = (int)((p1 - p0 + kStage - 1) / kStage);
        // thread tid stages PV consecutive points of job tid % J of a group; the values of the
        // group being loaded, and the pointer and exponent of the one after it
        const int vp = tid / S::J * S::PV;
        const double *vsrc = nullptr, *vnext = nullptr;
        int e = 0, enext = 0;
        auto job_of = [&](int g) {  // the group's job of this thread, into vnext and enext
            const int j = g < ng ? gid[g * S::J + tid % S::J] : -1;
            vnext = j >= 0 ? jobs[j].v : nullptr;
            enext = j >= 0 ? source_exponent(jobs[j]) : 0;
        };
        const double *wsrc = J0.v_mul;  // the jobs' common factor
        double v[S::PV], w[S::PV];
        auto load_v = [&](int64_t pb) {
#pragma unroll
            for (int q = 0; q < S::PV; ++q) {
                const int64_t p = pb + vp + q;
                v[q] = vsrc && p < p1 ? gp(vsrc)[p] : 0.0;
                w[q] = wsrc && p < p1 ? gp(wsrc)[p] : 1.0;
            }
        };
        auto store_v = [&](float *buf, int ex) {
#pragma unroll
            for (int q = 0; q < S::PV; ++q) buf[(vp + q) * S::kPitch + tid % S::J] = (float)ldexp(v[q] * w[q], -ex);
        };
        f32x4 acc[2][NA];  // two chains for every other four points
#pragma unroll
        for (int u = 0; u < 2 * NA; ++u) acc[u / NA][u % NA] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        St stg;
        job_of(0);
        vsrc = vnext;
        e = enext;
        stg.load(J0.src_win, nullptr, nullptr, p0, p1);
        load_v(p0);
        job_of(1);
        __syncthreads();  // the previous item's reads of LDS are done
        stg.store(rows[0], 0);
        store_v(vals[0], e);
        __syncthreads();
        int buf = 0;
        for (int g = 0; g < ng; ++g)
            for (int k = 0; k < nst; ++k, buf ^= 1) {
                // next: the following stage of this group, or the next group's first
                const bool last = k + 1 == nst, more = !last || g + 1 < ng;
                if (more) {
                    if (last) {
                        vsrc = vnext;
                        e = enext;
                        job_of(g + 2);
                    }
                    const int64_t pn = last ? p0 : p0 + (int64_t)(k + 1) * kStage;
                    load_v(pn);
                    if (nst > 1) stg.load(J0.src_win, nullptr, nullptr, pn, p1);
                }
                const float *rl = reinterpret_cast<const float *>(rows[nst > 1 ? buf : 0]);
                const float *vl = vals[buf];
                // points past the chunk's end have zero rows and values
                const int cnt = (int)min((int64_t)kStage, p1 - p0 - (int64_t)k * kStage);
                for (int j = 0; j < cnt; j += 16) {
                    float x[4][NA], b[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int pi = j + 4 * q + lk;
                        const float *row = rl + pi * (D * kPatch);
                        if constexpr (D == 2) {
                            const float w1 = row[kPatch + li];
                            const f32x4 w0 = reinterpret_cast<const f32x4 *>(row)[wave];
#pragma unroll
                            for (int u = 0; u < 4; ++u) x[q][u] = w0[u] * w1;
                            b[q] = vl[pi * S::kPitch + li];
                        } else {
                            x[q][0] = row[li];
                            b[q] = vl[pi * S::kPitch + 16 * wave + li];
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int u = 0; u < NA; ++u)
                            acc[q & 1][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q][u], b[q], acc[q & 1][u], 0, 0, 0);
                }
                if (more) {
                    store_v(vals[buf ^ 1], e);
                    if (nst > 1) stg.store(rows[buf ^ 1], 0);
                }
                if (last) {
                    // acc[u][r] = G[c' = 4 lk + r] (2-D: patch row a = 4 wave + u) of job li (1-D: 16 wave
                    // + li)
                    const int jo = gid[g * S::J + (D == 2 ? li : 16 * wave + li)];
                    if (jo >= 0) {
                        MOT_GLOBAL f32x4 *out = reinterpret_cast<MOT_GLOBAL f32x4 *>(gp(jobs[jo].patches)) +
                                                (int64_t)c * (D == 2 ? 64 : 4);
#pragma unroll
                        for (int u = 0; u < NA; ++u) out[(D == 2 ? (4 * wave + u) * 4 : 0) + lk] = acc[0][u] + acc[1][u];
                    }
#pragma unroll
                    for (int u = 0; u < 2 * NA; ++u) acc[u / NA][u % NA] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                }
                __syncthreads();
            }
    }
}

template <int D>
__global__ __launch_bounds__(256, 4) void interp_group_kernel(const ProdJob *__restrict__ jobs,
                                                              const int32_t *__restrict__ gids,
                                                              const int4 *__restrict__ items, int n_items)
{
    using S = GroupShape<D>;
    using St = Stage<D, false>;
    constexpr int kGPitch = 17;             // staged grid cells x 16 jobs (2-D)
    constexpr int NG = D == 2 ? 16 : 4;     // grid values loaded per thread and group
    __shared__ __align__(16) unsigned char rows[St::kBytes];
    __shared__ float cells[D == 2 ? 256 * kGPitch : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int4 itm = items[it];
        const int32_t *gid = gids + (int64_t)itm.x * S::J;
        const int ng = itm.y, c = itm.z;
        const ProdJob &J0 = jobs[gid[0]];
        const int64_t p0 = gp(J0.tgt_chunk_start)[c], p1 = gp(J0.tgt_chunk_start)[c + 1];
        const int tile = gp(J0.tgt_chunk_tile)[c], T = J0.T;
        const int nst = (int)((p1 - p0 + kStage - 1) / kStage);
        // 2-D: thread tid loads grid row a = tid / 16 of the tile for job tid % 16; 1-D: the B
        // operand of the wave's 16 jobs
        int64_t base;
        if constexpr (D == 2) {
            const int t0 = tile / J0.ntile[1], t1 = tile - t0 * J0.ntile[1];
            base = (int64_t)(t0 * T + (tid >> 4)) * J0.L[1] + t1 * T;
        } else {
            base = tile * T + lk;
        }
        const int lj = D == 2 ? tid & 15 : 16 * wave + li;  // job the thread loads the grid of
        const int oj = D == 2 ? li : 16 * wave + li;          // job the lane's results belong to
        const float *gnext = nullptr;
        double *onext = nullptr;
        int enext = 0;
        auto job_of = [&](int g) {
            const int jl = g < ng ? gid[g * S::J + lj] : -1, jo = g < ng ? gid[g * S::J + oj] : -1;
            gnext = jl >= 0 ? jobs[jl].grid : nullptr;
            onext = jo >= 0 ? jobs[jo].out : nullptr;
            enext = jo >= 0 ? source_exponent(jobs[jo]) : 0;
        };
        float gv[NG];
        auto load_g = [&]() {
#pragma unroll
            for (int q = 0; q < NG; ++q) gv[q] = gnext ? gp(gnext)[base + (D == 2 ? q : 4 * q)] : 0.0f;
        };
        St stg;
        job_of(0);
        stg.load(J0.tgt_win, nullptr, nullptr, p0, p1);
        load_g();
        __syncthreads();  // the previous item's reads of LDS are done
        stg.store(rows, 0);
        for (int g = 0; g < ng; ++g) {
            double *out = onext;
            const int e = enext;
            float gb[4];
            if constexpr (D == 2) {
                if (g > 0) __syncthreads();  // the previous group's reads of the cells are done
#pragma unroll
                for (int q = 0; q < 16; ++q) cells[((tid >> 4) * 16 + q) * kGPitch + (tid & 15)] = gv[q];
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) gb[s] = gv[s];
            }
            __syncthreads();
            job_of(g + 1);
            load_g();
            for (int k = 0; k < nst; ++k) {
                const int64_t pb = p0 + (int64_t)k * kStage;
                if (nst > 1 && g + k > 0) {
                    stg.load(J0.tgt_win, nullptr, nullptr, pb, p1);
                    __syncthreads();
                    stg.store(rows, 0);
                    __syncthreads();
                }
                const float *rl = reinterpret_cast<const float *>(rows);
                // 16-point groups: in 2-D group `wave` of the stage for the 16 jobs, in 1-D every one for
                // the wave's 16 jobs
#pragma unroll 1
                for (int q = D == 2 ? wave : 0; q < (D == 2 ? wave + 1 : 4); ++q) {
                    if (pb + 16 * q >= p1) break;
                    const float *row = rl + (16 * q + li) * (D * kPatch);
                    f32x4 acc[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) acc[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if constexpr (D == 2) {
                        float w1[4];
#pragma unroll
                        for (int s = 0; s < 4; ++s) w1[s] = row[kPatch + 4 * s + lk];
                        const float *gc = cells + lk * kGPitch + li;
                        // a chain for each quarter s of a row's cells, two for the inner ones, and rows from
                        // the patch's edges inward, where the windows are largest: the chains round at
                        // the size of the small terms until the last rows
                        f32x4 w0[4], mid[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
                        for (int a4 = 0; a4 < 4; ++a4) w0[a4] = reinterpret_cast<const f32x4 *>(row)[a4];
#pragma unroll
                        for (int j = 0; j < 16; ++j) {
                            const int a = j & 1 ? 15 - j / 2 : j / 2;
#pragma unroll
                            for (int s = 0; s < 4; ++s) {
                                f32x4 &c = (s == 1 || s == 2) && (j & 1) ? mid[s - 1] : acc[s];
                                c = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[a / 4][a % 4] * w1[s],
                                                                         gc[(a * 16 + 4 * s) * kGPitch], c, 0, 0, 0);
                            }
                        }
                        acc[1] += mid[0];
                        acc[2] += mid[1];
                    } else {
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(row[4 * s + lk], gb[s], acc[s], 0, 0, 0);
                    }
                    const f32x4 z = D == 2 ? (acc[0] + acc[3]) + (acc[1] + acc[2]) : (acc[0] + acc[1]) + (acc[2] + acc[3]);
                    // z[r]: point 16 q + 4 lk + r of the stage, the lane's job
                    if (out)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int64_t p = pb + 16 * q + 4 * lk + r;
                            if (p < p1) gp(out)[p] = ldexp((double)z[r], e);
                        }
                }
            }
        }
    }
}

static int nfft_grid(int n_items)
{
    return n_items < 65535 ? n_items : 65535;
}

hipError_t launch_spread3(int group, const ProdJob *jobs, const int4 *items, int n_items, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(64 * kSpreadWaves);
    if (group == 3)
        hipLaunchKernelGGL(spread3_kernel<3>, grid, block, 0, s, jobs, items, n_items);
    else if (group == 2)
        hipLaunchKernelGGL(spread3_kernel<2>, grid, block, 0, s, jobs, items, n_items);
    else if (group == 1)
        hipLaunchKernelGGL(spread3_kernel<1>, grid, block, 0, s, jobs, items, n_items);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_spread(int d, const ProdJob *jobs, const int2 *items, int n_items,
                         int /*max_patch_elems*/, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(64 * kSpreadWaves);
    if (d == 3)
        return hipErrorInvalidValue;  // 3-D items are grouped: launch_spread3
    else if (d == 2)
        hipLaunchKernelGGL(spread_kernel<2>, grid, block, 0, s, jobs, items, n_items);
    else
        hipLaunchKernelGGL(spread_kernel<1>, grid, block, 0, s, jobs, items, n_items);
    return hipGetLastError();
}

hipError_t launch_spread_group(int d, const ProdJob *jobs, const int32_t *gids, const int4 *items, int n_items,
                               hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(256);
    if (d == 2)
        hipLaunchKernelGGL(spread_group_kernel<2>, grid, block, 0, s, jobs, gids, items, n_items);
    else
        hipLaunchKernelGGL(spread_group_kernel<1>, grid, block, 0, s, jobs, gids, items, n_items);
    return hipGetLastError();
}

hipError_t launch_interp_group(int d, const ProdJob *jobs, const int32_t *gids, const int4 *items, int n_items,
                               hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(256);
    if (d == 2)
        hipLaunchKernelGGL(interp_group_kernel<2>, grid, block, 0, s, jobs, gids, items, n_items);
    else
        hipLaunchKernelGGL(interp_group_kernel<1>, grid, block, 0, s, jobs, gids, items, n_items);
    return hipGetLastError();
}

hipError_t launch_fold(int d, const ProdJob *jobs, const int2 *items, int n_items, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(kFoldCellsPerItem);
    if (d == 0)
        hipLaunchKernelGGL((fold_kernel<0, 1>), grid, block, 0, s, jobs, items, n_items);
    else if (d == 3 && n_items <= kFoldSplitItems)
        hipLaunchKernelGGL((fold_kernel<3, 2>), grid, dim3(2 * kFoldCellsPerItem), 0, s, jobs, items, n_items);
    else if (d == 3)
        hipLaunchKernelGGL((fold_kernel<3, 1>), grid, block, 0, s, jobs, items, n_items);
    else if (d == 2)
        hipLaunchKernelGGL((fold_kernel<2, 1>), grid, block, 0, s, jobs, items, n_items);
    else
        hipLaunchKernelGGL((fold_kernel<1, 1>), grid, block, 0, s, jobs, items, n_items);
    return hipGetLastError();
}

hipError_t launch_interp(int d, const ProdJob *jobs, const int2 *items, int n_items,
                         int /*max_patch_elems*/, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const dim3 grid(nfft_grid(n_items)), block(64 * kInterpWaves);
    if (d == 3)
        hipLaunchKernelGGL(interp3_kernel, grid, block, 0, s, jobs, items, n_items);
    else if (d == 2)
        hipLaunchKernelGGL(interp_kernel<2>, grid, block, 0, s, jobs, items, n_items);
    else
        hipLaunchKernelGGL(interp_kernel<1>, grid, block, 0, s, jobs, items, n_items);
    return hipGetLastError();
}

}  // namespace mot
