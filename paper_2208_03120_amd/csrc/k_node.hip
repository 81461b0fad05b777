// FP64 node updates of the tree sweep (a8, a10) and small utility kernels.
//
// Algorithm 2 in terms of per-node elementwise work (cp = prod_{t in C_k} beta_t, the
// children's messages multiplied in ascending child order starting from 1):
//   update:    phi^k <- mu^k / (gamma_k * cp)            (gamma_root = 1)
//              S terms: sum mu^k log phi^k_old, and for the root
//              sum (mu / phi_new) phi_old (the last term of S^(r))
//   down src:  u_c = (phi^k * gamma_k) * prod_{t in C_k, t != c} beta_t   for every child c
//              (the vector whose transposed kernel product gives gamma_c, eq. gamma_tree)
//   up src:    v_k = phi^k * cp                             (beta_k = K^{(p,k)} v_k)
//   marginal:  P_k = (phi^k * gamma_k) * cp               (Theorem 4.1), and |P_k - mu^k|
//   free node (generalised barycenter, Sec. 6.2): phi^k = 1 instead of the update, no S
//              term and no marginal error (mu^k is not given)
// Every product vector also records max_i exponent(value) in the job's slot so the
// product kernels can scale it into FP32 range without loss.
// Per-item partial sums go to distinct slots (no floating-point atomics): reductions
// are deterministic.
#include "mot_internal.h"

namespace mot {

constexpr int kNodeElems = kNodeItemElems;   // elements per node item
constexpr int kNodeEPT = kNodeElems / 256;     // elements per thread (256 threads)
constexpr int kRegChildren = 16;  // children held in registers (more: read from memory)
constexpr int kFewChildren = 4;   // the same, for launches of nodes with at most 4 children

__device__ __forceinline__ int exp_of(double v)
{
    return (v > 0.0 && v < INFINITY) ? ilogb(v) : INT32_MIN;
}

// Sum over the four wavefronts of a 256-thread group whose wavefronts wrote their sums to red.
__device__ __forceinline__ double group_sum(const double *red)
{
    return ((red[0] + red[1]) + red[2]) + red[3];
}

__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    return group_sum(red);
}

// One node item: up to kNodeItemElems elements of one node.  The messages of up to RC
// children are held in registers (loaded before any output is written); a node with more
// children reads them from memory for every product and records the exponent maxima of its
// down sources with one atomic per element.  Launches of small trees are bound by the chain
// of dependent loads, the FP64 logarithm and division and the block's reductions: the child
// pointers of up to kInlineChildren children are in the job itself, the logarithm is taken
// while the messages load, and all reductions meet at one barrier (500 points: 4.9 -> 3.5 us).
template <int RC>
__global__ __launch_bounds__(256) void node_kernel(const NodeJob *__restrict__ jobs,
                                                   const int2 *__restrict__ items, int n_items)
{
    __shared__ double red[2][4];
    __shared__ int emx[4][RC + 1];
    constexpr bool INL = RC <= kInlineChildren;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const NodeJob &J = jobs[itm.x];
        const int op = J.op;
        const bool upd = op & 1, dsrc = op & 2, usrc = op & 4, root = op & 8, marg = op & 16;
        const bool freen = op & 32;
        const int nch = J.nchild;
        const bool regs = nch <= RC;
        auto beta_of = [&](int t) { return INL ? J.beta_in[t] : (const double *)gp(J.beta)[t]; };
        auto down_of = [&](int t) { return INL ? J.down_in[t] : (double *)gp(J.down_src)[t]; };
        double s1 = 0.0, s2 = 0.0;
        int em_up = INT32_MIN;
        int em[RC];
#pragma unroll
        for (int c = 0; c < RC; ++c) em[c] = INT32_MIN;
        bool bad = false;
        // the inputs of all of this thread's elements (children's messages too, when they
        // fit in registers) are loaded before any output is written, so that the loads
        // are in flight together
        double mu_k[kNodeEPT], ph_k[kNodeEPT], g_k[kNodeEPT];
        double b[RC][kNodeEPT];
#pragma unroll
        for (int k = 0; k < kNodeEPT; ++k) {
            const int64_t i = (int64_t)itm.y + tid + 256 * k;
            mu_k[k] = ph_k[k] = g_k[k] = 1.0;
#pragma unroll
            for (int t = 0; t < RC; ++t) b[t][k] = 1.0;
            if (i < J.n) {
                mu_k[k] = gp(J.mu)[i];
                ph_k[k] = gp(J.phi)[i];
                if (!root) g_k[k] = gp(J.gamma)[i];
                if (regs)
#pragma unroll
                    for (int t = 0; t < RC; ++t)
                        if (t < nch) b[t][k] = gp(beta_of(t))[i];
            }
        }
        if (upd && !freen)
#pragma unroll
            for (int k = 0; k < kNodeEPT; ++k)
                if ((int64_t)itm.y + tid + 256 * k < J.n && mu_k[k] > 0.0) s1 += mu_k[k] * log(ph_k[k]);
#pragma unroll
        for (int k = 0; k < kNodeEPT; ++k) {
            const int64_t i = (int64_t)itm.y + tid + 256 * k;
            if (i >= J.n) break;
            double cp = 1.0;
            if (regs) {
#pragma unroll
                for (int t = 0; t < RC; ++t)
                    if (t < nch) cp *= b[t][k];
            } else {
                for (int t = 0; t < nch; ++t) cp *= gp(gp(J.beta)[t])[i];
            }
            const double g = g_k[k];
            const double mu = mu_k[k];
            double ph = ph_k[k];
            if (upd && freen) {
                gp(J.phi)[i] = 1.0;  // no marginal constraint: phi^k = 1 in every sweep
                ph = 1.0;
            } else if (upd) {
                const double nv = mu / (g * cp);
                if (root && mu > 0.0) s2 += (mu / nv) * ph;
                if (!isfinite(nv)) bad = true;
                gp(J.phi)[i] = nv;
                ph = nv;
            }
            if (marg) {
                const double P = (ph * g) * cp;
                gp(J.marg_out)[i] = P;
                if (!freen) s1 += fabs(P - mu);
            }
            if (usrc) {
                const double v = ph * cp;
                gp(J.up_src)[i] = v;
                em_up = max(em_up, exp_of(v));
            }
            if (dsrc) {
                const double pg = ph * g;
                if (regs) {
#pragma unroll
                    for (int c = 0; c < RC; ++c) {
                        if (c >= nch) break;
                        double w = 1.0;
#pragma unroll
                        for (int t = 0; t < RC; ++t)
                            if (t < nch && t != c) w *= b[t][k];
                        const double u = pg * w;
                        gp(down_of(c))[i] = u;
                        em[c] = max(em[c], exp_of(u));
                    }
                } else {
                    for (int c = 0; c < nch; ++c) {
                        double w = 1.0;
                        for (int t = 0; t < nch; ++t)
                            if (t != c) w *= gp(gp(J.beta)[t])[i];
                        const double u = pg * w;
                        gp(gp(J.down_src)[c])[i] = u;
                        atomicMax(J.down_exp[c], exp_of(u));
                    }
                }
            }
        }
        if (bad) atomicOr(J.flag, 1);
        // wavefront sums and exponent maxima, then over the block: one partial sum pair per
        // item and one atomic per vector
        if (it != (int)blockIdx.x) __syncthreads();  // the previous item's reads of LDS are done
        if (upd || marg) {
            const double t1 = wave_sum(s1);
            const double t2 = root ? wave_sum(s2) : 0.0;
            if (lane == 0) {
                red[0][wave] = t1;
                red[1][wave] = t2;
            }
        }
        if (usrc) {
            const int m = wave_max_int(em_up);
            if (lane == 0) emx[wave][RC] = m;
        }
        if (dsrc && regs) {
#pragma unroll
            for (int c = 0; c < RC; ++c) {
                if (c < nch) {  // nch is uniform over the block
                    const int m = wave_max_int(em[c]);
                    if (lane == 0) emx[wave][c] = m;
                }
            }
        }
        __syncthreads();
        if (tid <= RC) {
            const bool is_up = tid == RC;
            if ((is_up && usrc) || (!is_up && dsrc && regs && tid < nch)) {
                const int m = max(max(emx[0][tid], emx[1][tid]), max(emx[2][tid], emx[3][tid]));
                if (m != INT32_MIN) atomicMax(is_up ? J.up_exp : (INL ? J.dexp_in[tid] : J.down_exp[tid]), m);
            }
        }
        if ((upd || marg) && tid >= 64 && tid < 66) {  // the second wavefront, beside the atomics
            const int slot = J.block0 + (int)(itm.y / kNodeElems);
            gp(J.partial)[2 * slot + tid - 64] = group_sum(red[tid - 64]);
        }
    }
}

hipError_t launch_node(const NodeJob *jobs_dev, const int2 *items, int n_items, int max_children, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    const int grid = n_items < 8192 ? n_items : 8192;
    // the register copies of the children's messages set the kernel's register count, and
    // with it how many blocks run at once: launches whose nodes have at most one or at most
    // kFewChildren children take the smaller forms
    if (max_children <= 1)  // leaves and the nodes of a path
        hipLaunchKernelGGL(node_kernel<1>, dim3(grid), dim3(256), 0, s, jobs_dev, items, n_items);
    else if (max_children <= kFewChildren)
        hipLaunchKernelGGL(node_kernel<kFewChildren>, dim3(grid), dim3(256), 0, s, jobs_dev, items, n_items);
    else
        hipLaunchKernelGGL(node_kernel<kRegChildren>, dim3(grid), dim3(256), 0, s, jobs_dev, items, n_items);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Sweep finalisation, two launches.
//   finalize_l1_kernel, item = (job, first root element): the root marginal
//     P_0 = phi^0 * prod_{t in C_0} beta_t after the upward pass and the L1 error of the
//     item's elements, one partial per item;
//   finalize_reduce_kernel, one block per job: the partial sums in a fixed order,
//     S^(r) = eta * (sum mu log phi_old - sum (mu / phi_new) phi_old)
//     and the error recorded at the plan's sweep counter, the exponent slots re-armed for
//     the next sweep.
// The kernel boundary orders the partials before their reduction, so no block waits on
// another and no device-scope fence is needed.
// L1 error of the elements first + tid, first + tid + 256, .. of an item.
__device__ __forceinline__ double finalize_l1(const FinalJob &J, int64_t first, int tid)
{
    // child products of all of this thread's elements, children in ascending order
    double cp[kNodeEPT], l1 = 0.0;
    bool ok[kNodeEPT];
#pragma unroll
    for (int k = 0; k < kNodeEPT; ++k) {
        cp[k] = 1.0;
        ok[k] = first + tid + 256 * k < J.n0;
    }
    if (J.nchild <= kRegChildren) {
        // all children's messages loaded before the products, so the loads are in
        // flight together; multiplied in ascending child order
        double b[kRegChildren][kNodeEPT];
#pragma unroll
        for (int t = 0; t < kRegChildren; ++t)
#pragma unroll
            for (int k = 0; k < kNodeEPT; ++k)
                b[t][k] = (t < J.nchild && ok[k]) ? gp(gp(J.root_beta)[t])[first + tid + 256 * k] : 1.0;
#pragma unroll
        for (int t = 0; t < kRegChildren; ++t)
#pragma unroll
            for (int k = 0; k < kNodeEPT; ++k)
                if (t < J.nchild) cp[k] *= b[t][k];
    } else {
        for (int t = 0; t < J.nchild; ++t) {
            const MOT_GLOBAL double *bt = gp(gp(J.root_beta)[t]);
#pragma unroll
            for (int k = 0; k < kNodeEPT; ++k)
                if (ok[k]) cp[k] *= bt[first + tid + 256 * k];
        }
    }
#pragma unroll
    for (int k = 0; k < kNodeEPT; ++k) {
        const int64_t i = first + tid + 256 * k;
        if (ok[k]) l1 += fabs(gp(J.phi0)[i] * cp[k] - gp(J.mu0)[i]);
    }
    return l1;
}

// Thread tid's share (of 256) of the node updates' partial sums: a fixed strided subset.  Eight
// strided partials are loaded before they are added (in the same order), so the loads of a
// thread are in flight together.
__device__ __forceinline__ void finalize_partials(const FinalJob &J, int tid, double &s1, double &s2)
{
    constexpr int U = 8;
    s1 = s2 = 0.0;
    for (int p0 = tid; p0 < J.n_partials; p0 += U * 256) {
        double a[U], b[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int p = p0 + q * 256;
            a[q] = p < J.n_partials ? J.s_partial[2 * p] : 0.0;
            b[q] = p < J.n_partials ? J.s_partial[2 * p + 1] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (p0 + q * 256 < J.n_partials) {
                s1 += a[q];
                s2 += b[q];
            }
    }
}

__device__ __forceinline__ void finalize_record(const FinalJob &J, double s1, double s2, double e1)
{
    const int r = *J.sweep_ctr;
    const int slot = r % J.hist_cap;
    J.S_hist[slot] = J.eta * (s1 - s2);
    J.err_hist[slot] = e1;
    J.flag_hist[slot] = *J.flag;
    *J.sweep_ctr = r + 1;
}

__global__ __launch_bounds__(256) void finalize_l1_kernel(const FinalJob *__restrict__ jobs,
                                                          const int2 *__restrict__ items, int n_items)
{
    __shared__ double red[4];
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 itm = items[it];
        const FinalJob &J = jobs[itm.x];
        const double tot = block_sum(finalize_l1(J, itm.y, threadIdx.x), red);
        if (threadIdx.x == 0) J.l1_partial[itm.y / kNodeElems] = tot;
    }
}

__global__ __launch_bounds__(256) void finalize_reduce_kernel(const FinalJob *__restrict__ jobs, int n_jobs)
{
    __shared__ double red[4];
    const int tid = threadIdx.x;
    for (int j = blockIdx.x; j < n_jobs; j += gridDim.x) {
        const FinalJob &J = jobs[j];
        double s1, s2, e1 = 0.0;
        finalize_partials(J, tid, s1, s2);
        for (int p = tid; p < J.n_items; p += blockDim.x) e1 += J.l1_partial[p];
        s1 = block_sum(s1, red);
        s2 = block_sum(s2, red);
        e1 = block_sum(e1, red);
        if (tid == 0) finalize_record(J, s1, s2, e1);
        for (int s = tid; s < J.n_exp_slots; s += blockDim.x) J.exp_slots[s] = INT32_MIN;
        __syncthreads();  // red is reused by the next job
    }
}

// Both steps in one block per job, for roots of at most kFinalSmall elements (a second launch
// costs more than the block's rounds: 500 points, 2.9 and 3.6 us in two launches, 3.8 us in one): four groups of 256 threads take an item each, then the
// first group reduces.  Sums are formed exactly as by the two kernels.
constexpr int kFinalGroups = 4, kFinalSmall = 4096;
static_assert(kFinalSmall % kNodeElems == 0, "whole items");
__global__ __launch_bounds__(256 * kFinalGroups) void finalize_small_kernel(const FinalJob *__restrict__ jobs, int n_jobs)
{
    __shared__ double red[kFinalGroups][4], l1p[kFinalSmall / kNodeElems], red3[3][4];
    const int grp = threadIdx.x >> 8, tid = threadIdx.x & 255, wave = tid >> 6, lane = tid & 63;
    for (int j = blockIdx.x; j < n_jobs; j += gridDim.x) {
        const FinalJob &J = jobs[j];
        for (int q0 = 0; q0 < J.n_items; q0 += kFinalGroups) {
            const int q = q0 + grp;
            double l1 = 0.0;
            if (q < J.n_items) l1 = finalize_l1(J, (int64_t)q * kNodeElems, tid);
            l1 = wave_sum(l1);
            if (lane == 0) red[grp][wave] = l1;
            __syncthreads();
            if (tid == 0 && q < J.n_items) l1p[q] = group_sum(red[grp]);
            __syncthreads();
        }
        if (grp == 0) {
            double s1, s2, e1 = 0.0;
            finalize_partials(J, tid, s1, s2);
            for (int p = tid; p < J.n_items; p += 256) e1 += l1p[p];
            s1 = wave_sum(s1);
            s2 = wave_sum(s2);
            e1 = wave_sum(e1);
            if (lane == 0) {
                red3[0][wave] = s1;
                red3[1][wave] = s2;
                red3[2][wave] = e1;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) finalize_record(J, group_sum(red3[0]), group_sum(red3[1]), group_sum(red3[2]));
        for (int s = threadIdx.x; s < J.n_exp_slots; s += blockDim.x) J.exp_slots[s] = INT32_MIN;
        __syncthreads();
    }
}

hipError_t launch_finalize(const FinalJob *jobs, const int2 *items, int n_items, int n_jobs, bool small, hipStream_t s)
{
    if (n_items == 0 || n_jobs == 0) return hipSuccess;
    if (small) {
        hipLaunchKernelGGL(finalize_small_kernel, dim3(n_jobs < 8192 ? n_jobs : 8192), dim3(256 * kFinalGroups), 0, s,
                           jobs, n_jobs);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(finalize_l1_kernel, dim3(n_items < 8192 ? n_items : 8192), dim3(256), 0, s, jobs, items,
                       n_items);
    hipLaunchKernelGGL(finalize_reduce_kernel, dim3(n_jobs < 8192 ? n_jobs : 8192), dim3(256), 0, s, jobs, n_jobs);
    return hipGetLastError();
}

bool finalize_small(int64_t n0) { return n0 <= kFinalSmall; }

// ---------------------------------------------------------------------------------------
// Utilities

__global__ void fill_int_kernel(int32_t *p, int32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void fill_double_kernel(double *p, double v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
hipError_t launch_fill_int(int32_t *p, int32_t value, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_int_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p,
                       value, count);
    return hipGetLastError();
}
hipError_t launch_fill_double(double *p, double value, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_double_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s,
                       p, value, count);
    return hipGetLastError();
}

// dst[i] = src[perm[i]] for rows of d doubles (original -> binned order)
__global__ void gather_rows_kernel(const double *__restrict__ src, const int32_t *__restrict__ perm,
                                   int64_t n, int d, double *__restrict__ dst)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t j = perm[i];
    for (int c = 0; c < d; ++c) dst[i * d + c] = src[j * d + c];
}
// dst[perm[i]] = src[i] (binned -> original order)
__global__ void scatter_vec_kernel(const double *__restrict__ src, const int32_t *__restrict__ perm,
                                   int64_t n, double *__restrict__ dst)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[perm[i]] = src[i];
}
hipError_t launch_gather_rows(const double *src, const int32_t *perm, int64_t n, int d, double *dst,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src,
                       perm, n, d, dst);
    return hipGetLastError();
}
hipError_t launch_scatter_vec(const double *src, const int32_t *perm, int64_t n, double *dst,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(scatter_vec_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src,
                       perm, n, dst);
    return hipGetLastError();
}

// Pair marginal of a tree edge (Theorem 4.1 applied to two adjacent marginals): one
// row i of the parent per block, columns across the threads; written in original order.
__global__ void tree_pair_kernel(const double *__restrict__ u, const double *__restrict__ xa,
                                 const int32_t *__restrict__ perm_a, const double *__restrict__ w,
                                 const double *__restrict__ xb, const int32_t *__restrict__ perm_b,
                                 int64_t na, int64_t nb, int d, double inv_eta, double *__restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nb) return;
    for (int64_t i = blockIdx.y; i < na; i += gridDim.y) {
        double d2 = 0.0;
        for (int c = 0; c < d; ++c) {
            const double df = xa[i * d + c] - xb[j * d + c];
            d2 += df * df;
        }
        out[(int64_t)perm_a[i] * nb + perm_b[j]] = (u[i] * exp(-d2 * inv_eta)) * w[j];
    }
}

hipError_t launch_tree_pair(const double *u, const double *xa, const int32_t *perm_a, int64_t na,
                            const double *w, const double *xb, const int32_t *perm_b, int64_t nb, int d,
                            double eta, double *out, hipStream_t s)
{
    if (na <= 0 || nb <= 0) return hipSuccess;
    const unsigned gy = (unsigned)(na < 32768 ? na : 32768);
    hipLaunchKernelGGL(tree_pair_kernel, dim3((unsigned)((nb + 255) / 256), gy), dim3(256), 0, s, u, xa, perm_a,
                       w, xb, perm_b, na, nb, d, 1.0 / eta, out);
    return hipGetLastError();
}

// What a caller of sweeps is told after them, gathered for one copy: the last two values of S, the
// last error, the sweeps of the plan so far and the flag (a copy of a few bytes to pageable memory
// costs the host about 12 us; five of them were read one by one).
__global__ void sweep_status_kernel(const int32_t *ctr, const int32_t *flag, int hist_cap, const double *S_hist,
                                    const double *err_hist, SweepStatus *out)
{
    const int r = *ctr, idx = (r - 1 + hist_cap) % hist_cap, idxp = (r - 2 + hist_cap) % hist_cap;
    *out = {S_hist[idxp], S_hist[idx], err_hist[idx], r, *flag};
}

hipError_t launch_sweep_status(const int32_t *ctr, const int32_t *flag, int hist_cap, const double *S_hist,
                               const double *err_hist, SweepStatus *out, hipStream_t s)
{
    hipLaunchKernelGGL(sweep_status_kernel, dim3(1), dim3(1), 0, s, ctr, flag, hist_cap, S_hist, err_hist, out);
    return hipGetLastError();
}

// max exponent of a vector into a slot (for products requested outside a sweep)
__global__ void vec_exp_kernel(const double *__restrict__ v, int64_t n, int32_t *slot)
{
    int m = INT32_MIN;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        m = max(m, exp_of(v[i]));
    m = wave_max_int(m);
    if ((threadIdx.x & 63) == 0 && m != INT32_MIN) atomicMax(slot, m);
}
hipError_t launch_vec_exp(const double *v, int64_t n, int32_t *slot, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(vec_exp_kernel, dim3(blocks), dim3(256), 0, s, v, n, slot);
    return hipGetLastError();
}

}  // namespace mot
