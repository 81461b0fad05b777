// The sum of the patches that cover a grid cell, shared by the fold and the one-launch
// transforms.
#pragma once

#include <type_traits>

#include "mot_internal.h"

namespace mot {

constexpr int kFoldTab = 2048;  // tile -> chunk table entries staged in LDS

// a / T for 0 <= a < 2^20 and rT = 1 / T (T < 2^10): a + 1/2 keeps the rounded quotient off the
// integers.
__device__ __forceinline__ int div_small(int a, float rT) { return (int)(((float)a + 0.5f) * rT); }

// Sum of the patches covering cell (gu0, gu1, g) (leading coordinates unused below 3-D and
// 2-D) when at most COV tiles cover it per dimension, tch the job's tile -> chunk table (in
// LDS when it fits).  The chunk ranges of all (u, k) pairs of the last two dimensions (in 3-D
// of one leading tile) are looked up together, and the r-th chunks of all pairs are loaded
// together and then added, so a round of loads waits once.  Absent tiles and chunks read entry
// 0 and add zero: predicated loads cost a branch each, which bound small folds (30 x 30 cells
// in 2-D: 8.8 us per launch with branches).  3-D launches that fill the chip (PARTS = 1) are bound
// by the loads themselves, a third of them of absent tiles when tiles have 5 cells, and predicate
// them, with the lookups where the table is in global memory: nine jobs on a 46^3 box 29.3 us
// without and 26.1 with, nine on a 111^3 box, whose table does not fit in LDS, 519 and 389.  In 3-D
// every second leading tile goes to a sum of its own, so that the two threads of a cell (part = 0 and
// 1 of PARTS = 2) give the same bits as one.
template <int D, int COV, int PARTS, class Tab>
__device__ __forceinline__ float fold_cover(const ProdJob &J, const int (&gu)[2], int g, Tab tch, int part)
{
    constexpr int W = 16, NU = D >= 2 ? COV : 1, pe = D == 3 ? 4096 : (D == 2 ? 256 : 16);
    // chunks of a tile loaded together; in 3-D two only where two threads share a cell: launches that
    // fill the chip lose more to the absent second chunks than the loads in flight give (ten sweeps
    // of nine jobs on a 46^3 box: 4.92 ms with one, 5.02 with two)
    constexpr int NR = D == 1 ? 4 : (PARTS == 2 ? 2 : 1);
    constexpr int lead = D == 3 ? 1 : 0;  // index of the u dimension among the leading ones
    constexpr bool kPickPatch = D == 3 && PARTS == 1;                        // predicated loads
    constexpr bool kPickTab = std::is_same<Tab, const MOT_GLOBAL int32_t *>::value;  // and lookups
    const int T = J.T, ntl = J.ntile[D - 1];
    const float rT = 1.0f / (float)T;
    const MOT_GLOBAL float *pat = gp(J.patches);
    // tiles covering c: from ceil((c - W + 1) / T) to c / T
    const int ka = div_small(max(0, g - W + T), rT), kb = min(ntl - 1, div_small(g, rT));
    const int ua = D >= 2 ? div_small(max(0, gu[lead] - W + T), rT) : 0;
    const int ub = D >= 2 ? min(J.ntile[lead] - 1, div_small(gu[lead], rT)) : 0;
    const int t0a = D == 3 ? div_small(max(0, gu[0] - W + T), rT) : 0;
    const int t0b = D == 3 ? min(J.ntile[0] - 1, div_small(gu[0], rT)) : 0;
    // parts of the tile index and patch offset of candidate (u, k) that do not depend on the
    // leading tile t0 of 3-D:
    //   tile = t0 nt1 ntl + tl_b + u ntl + k,  loc = (gu0 - t0 T) W^2 + loc_b - u T W - k T
    const int tl_b = ua * ntl + ka;
    const int loc_b = (D >= 2 ? (gu[lead] - ua * T) * W : 0) + (g - ka * T);
    float acc = 0.0f, other = 0.0f;  // of every second leading tile
    for (int t0 = t0a + part; t0 <= t0b; t0 += PARTS) {
        const int tl0 = (D == 3 ? t0 * J.ntile[1] * ntl : 0) + tl_b;
        const int loc0 = (D == 3 ? (gu[0] - t0 * T) * W * W : 0) + loc_b;
        uint32_t at[NU][COV];
        int nc[NU][COV], most = 0;  // chunks of each candidate tile and of the fullest
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int k = 0; k < COV; ++k) {
                const bool ok = ua + u <= ub && ka + k <= kb;
                const int tl = ok ? tl0 + u * ntl + k : 0;
                int c0 = 0, c1 = 0;
                if (!kPickTab || ok) {
                    c0 = tch[tl];
                    c1 = tch[tl + 1];
                }
                nc[u][k] = ok ? c1 - c0 : 0;
                at[u][k] = (uint32_t)c0 * pe + (uint32_t)(loc0 - u * T * W - k * T);
                most = max(most, nc[u][k]);
            }
        for (int r0 = 0; r0 < most; r0 += NR) {
            float val[NR][NU][COV];
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int k = 0; k < COV; ++k) {
                        const bool there = nc[u][k] > r0 + r;
                        val[r][u][k] = 0.0f;
                        if (!kPickPatch || there) val[r][u][k] = pat[(uint64_t)(there ? at[u][k] : 0u)];
                        at[u][k] += pe;
                    }
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int k = 0; k < COV; ++k) acc += nc[u][k] > r0 + r ? val[r][u][k] : 0.0f;
        }
        if (D == 3 && PARTS == 1) {
            const float t = acc;
            acc = other;
            other = t;
        }
    }
    return acc + other;
}

// The same for any cover (narrow tiles) and any count of chunks.
template <int D, int PARTS, class Tab>
__device__ __forceinline__ float fold_any(const ProdJob &J, const int (&gu)[2], int g, Tab tch, int part)
{
    const int W = J.W, T = J.T, ntl = J.ntile[D - 1];
    int tlo[2] = {0, 0}, thi[2] = {0, 0};
    for (int c = 0; c < D - 1; ++c) {
        tlo[c] = max(0, gu[c] - W + T) / T;  // ceil((g - W + 1) / T)
        thi[c] = min(J.ntile[c] - 1, gu[c] / T);
    }
    const int pe = D == 3 ? W * W * W : (D == 2 ? W * W : W);
    const MOT_GLOBAL float *pat = gp(J.patches);
    const int t2lo = max(0, g - W + T) / T, t2hi = min(ntl - 1, g / T);
    float acc = 0.0f, other = 0.0f;
    for (int t0 = tlo[0] + part; t0 <= thi[0]; t0 += PARTS) {
        for (int t1 = tlo[1]; t1 <= thi[1]; ++t1) {
            int lead_tile = 0, lead_loc = 0;
            if constexpr (D == 3) {
                lead_tile = t0 * J.ntile[1] + t1;
                lead_loc = (gu[0] - t0 * T) * W + (gu[1] - t1 * T);
            } else if constexpr (D == 2) {
                lead_tile = t0;
                lead_loc = gu[0] - t0 * T;
            }
            for (int t2 = t2lo; t2 <= t2hi; ++t2) {
                const int tl = lead_tile * ntl + t2;
                const int lc = lead_loc * W + (g - t2 * T);
                const int ca = tch[tl], cb = tch[tl + 1];
                for (int ch = ca; ch < cb; ++ch) acc += pat[(int64_t)ch * pe + lc];
            }
        }
        if (D == 3 && PARTS == 1) {
            const float t = acc;
            acc = other;
            other = t;
        }
    }
    return acc + other;
}

template <int D, int PARTS = 1, class Tab>
__device__ __forceinline__ float fold_cell(const ProdJob &J, const int (&gu)[2], int g, Tab tch, int part = 0)
{
    // patch entries are addressed in 32 bits by fold_cover
    if (J.T >= 8) {
        if (J.src_nchunks < (1 << 20)) return fold_cover<D, 2, PARTS>(J, gu, g, tch, part);
    } else if (J.T >= 6) {
        if (J.src_nchunks < (1 << 20)) return fold_cover<D, 3, PARTS>(J, gu, g, tch, part);
    } else if (J.T >= 4) {
        if (J.src_nchunks < (1 << 20)) return fold_cover<D, 4, PARTS>(J, gu, g, tch, part);
    }
    return fold_any<D, PARTS>(J, gu, g, tch, part);
}

}  // namespace mot
