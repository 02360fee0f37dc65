// Ridge (Tikhonov) estimator of Sec. 9: conjugate gradients on the normal
// equations (A^T A + lambda I) x = A^T y.  For a handle with G geometries the
// normal equations are block diagonal, so every (right-hand side, geometry)
// pair runs its own CG with its own step lengths: the same iterates as G
// separate solves.  Every iteration is one block application of A and of A^T
// (all pairs at once) plus FP64 dot products per pair; step lengths live in
// device memory.  The blocking mode looks at the residuals every few
// iterations from the host; the stream-ordered mode runs a fixed number of
// iterations with no host synchronisation (pairs that have converged stop
// changing) so that a whole solve can be captured into a graph.
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "dense.h"

namespace rtt {

// The vector work of an iteration in three kernels (nine before: 20 iterations at 256^2, one right-hand
// side, 1.44 -> 1.00 ms, 0.81 with A^T in one launch; the launches of 4 to 5 us each being the cost).  Grid: (slices of a geometry's
// column block, right-hand sides, geometries); a block takes one slice of one pair and leaves the FP64
// partial of the pair's dot product, and the next kernel's blocks each add the pair's partials in the same
// fixed order.  The residual norms and flags alternate between two buffers: every block of an iteration
// reads one, the first block of a pair writes the other.
constexpr int CG_T = 256;        // threads per block
constexpr int CG_SLICES = 256;   // most slices of a pair (one partial per thread)

// scalar index of (right-hand side v, geometry g): v * G + g
struct CgPair {
    int64_t pair, off;      // scalar index; first element in the block of vectors
    int64_t l0, l1;         // the block's slice of the pair's elements
};
__device__ __forceinline__ CgPair cg_pair(const int64_t* __restrict__ seg, int64_t n)
{
    const int v = blockIdx.y, g = blockIdx.z;
    const int64_t len = seg[2 * g + 1], slice = (len + gridDim.x - 1) / gridDim.x;
    CgPair c;
    c.pair = (int64_t)v * gridDim.z + g;
    c.off = (int64_t)v * n + seg[2 * g];
    c.l0 = (int64_t)blockIdx.x * slice;
    c.l1 = min(len, c.l0 + slice);
    return c;
}
// sum over the block, the same for every thread: lanes by halving distances, then the waves in order
__device__ __forceinline__ double cg_block_sum(double v)
{
    __shared__ double red[CG_T / 64];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    __syncthreads();   // the last sum's readers
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < CG_T / 64; ++w) t += red[w];
    return t;
}
__device__ __forceinline__ double cg_partials(const double* __restrict__ part, int64_t pair)
{
    const int nsl = gridDim.x;
    return cg_block_sum((int)threadIdx.x < nsl ? part[pair * nsl + threadIdx.x] : 0.0);
}

// start: r = p = src (src may be r), x = 0, partials of <r, r>
__global__ __launch_bounds__(CG_T) void k_cg_start(const float* src, float* r, float* __restrict__ p, float* __restrict__ x,
                                                   const int64_t* __restrict__ seg, int64_t n, double* __restrict__ part)
{
    const CgPair c = cg_pair(seg, n);
    double acc = 0.0;
#pragma unroll 4
    for (int64_t i = c.off + c.l0 + threadIdx.x; i < c.off + c.l1; i += CG_T) {
        const float v = src[i];
        if (src != r) r[i] = v;
        p[i] = v;
        x[i] = 0.f;
        acc += (double)v * (double)v;
    }
    acc = cg_block_sum(acc);
    if (threadIdx.x == 0) part[c.pair * gridDim.x + blockIdx.x] = acc;
}

// rr = bb = |A^T y|^2 per pair; a pair with bb = 0 (y orthogonal to the range) is done.  One block per
// pair, nsl partials each.
__global__ __launch_bounds__(CG_T) void k_cg_init(const double* __restrict__ part, int nsl, double* rr, double* bb, int* done)
{
    const int64_t pair = blockIdx.x;
    const double s = cg_block_sum((int)threadIdx.x < nsl ? part[pair * nsl + threadIdx.x] : 0.0);
    if (threadIdx.x == 0) {
        rr[pair] = bb[pair] = s;
        done[pair] = s > 0.0 ? 0 : 1;
    }
}

// Ap += Ap2 (when given) + lambda p, partials of <p, Ap>
__global__ __launch_bounds__(CG_T) void k_cg_pap(float* __restrict__ Ap, const float* __restrict__ Ap2,
                                                 const float* __restrict__ p, float lam, const int64_t* __restrict__ seg, int64_t n, double* __restrict__ part)
{
    const CgPair c = cg_pair(seg, n);
    double acc = 0.0;
#pragma unroll 4
    for (int64_t i = c.off + c.l0 + threadIdx.x; i < c.off + c.l1; i += CG_T) {
        const float pv = p[i];
        float av = Ap[i];
        if (Ap2) av += Ap2[i];
        if (lam != 0.f) av += lam * pv;
        if (Ap2 || lam != 0.f) Ap[i] = av;
        acc += (double)pv * (double)av;
    }
    acc = cg_block_sum(acc);
    if (threadIdx.x == 0) part[c.pair * gridDim.x + blockIdx.x] = acc;
}

// alpha = <r, r> / <p, Ap> (0 for a pair that is done); x += alpha p, r -= alpha Ap, partials of the new <r, r>
__global__ __launch_bounds__(CG_T) void k_cg_xr(float* __restrict__ x, float* __restrict__ r, const float* __restrict__ p,
                                                const float* __restrict__ Ap, const double* __restrict__ pap_part,
                                                const double* __restrict__ rr, const int* __restrict__ done,
                                                const int64_t* __restrict__ seg, int64_t n, double* __restrict__ pap,
                                                double* __restrict__ part)
{
    const CgPair c = cg_pair(seg, n);
    const double pa = cg_partials(pap_part, c.pair);
    const float a = (done[c.pair] || !(pa > 0.0)) ? 0.f : (float)(rr[c.pair] / pa);
    double acc = 0.0;
#pragma unroll 4
    for (int64_t i = c.off + c.l0 + threadIdx.x; i < c.off + c.l1; i += CG_T) {
        float rv = r[i];
        if (a != 0.f) {
            x[i] += a * p[i];
            rv -= a * Ap[i];
            r[i] = rv;
        }
        acc += (double)rv * (double)rv;
    }
    acc = cg_block_sum(acc);
    if (threadIdx.x == 0) {
        part[c.pair * gridDim.x + blockIdx.x] = acc;
        if (blockIdx.x == 0) pap[c.pair] = pa;
    }
}

// beta = new <r, r> / old; the pair is done when the new residual meets the tolerance (or <p, Ap> was not
// positive), else p = r + beta p.  rr / done: this iteration's, rr_out / done_out: the next one's.
__global__ __launch_bounds__(CG_T) void k_cg_p(float* __restrict__ p, const float* __restrict__ r,
                                               const double* __restrict__ rr_part, const double* __restrict__ rr,
                                               const double* __restrict__ bb, const double* __restrict__ pap,
                                               const int* __restrict__ done, const int64_t* __restrict__ seg, int64_t n,
                                               double tol2, double* __restrict__ rr_out, int* __restrict__ done_out)
{
    const CgPair c = cg_pair(seg, n);
    const double old = rr[c.pair], now = cg_partials(rr_part, c.pair);
    const int was = done[c.pair];
    const int is = was || now <= tol2 * bb[c.pair] || !(pap[c.pair] > 0.0);
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        rr_out[c.pair] = was ? old : now;
        done_out[c.pair] = is;
    }
    if (is) return;
    const float beta = (float)(old > 0.0 ? now / old : 0.0);
#pragma unroll 4
    for (int64_t i = c.off + c.l0 + threadIdx.x; i < c.off + c.l1; i += CG_T) p[i] = r[i] + beta * p[i];
}

__global__ void k_cg_resid(const double* rr, const double* bb, float* out, int npair)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= npair) return;
    out[v] = bb[v] > 0.0 ? (float)sqrt(rr[v] / bb[v]) : 0.f;
}

}  // namespace rtt

using namespace rtt;

extern "C" int ridge_solve(const rtt_geometry* g, const float* y, int32_t nrhs, float lambda,
                           const rtt_cg_opts* opts, float* x, rtt_solve_info* info, void* stream)
{
    if (!valid_handle(g)) return fail(RTT_EINVAL, "invalid geometry handle");
    if (nrhs < 0 || nrhs > 4096) return fail(RTT_EINVAL, "nrhs must be 0..4096");
    if (nrhs > 0 && (!y || !x)) return fail(RTT_EINVAL, "NULL data pointer");
    if (!(lambda >= 0.0f) || !std::isfinite(lambda)) return fail(RTT_EINVAL, "lambda must be finite and >= 0");
    const float tol = opts ? opts->tol : 1e-6f;
    const int maxit = opts ? opts->maxit : 1000;
    const uint32_t mask = opts ? opts->order_mask : 0u;
    const int32_t flags = opts ? opts->flags : 0;
    float* resid_dev = opts ? opts->resid_dev : nullptr;
    const bool async = (flags & RTT_SOLVE_ASYNC) != 0;
    if (!(tol > 0.0f) || maxit < 1) return fail(RTT_EINVAL, "need tol > 0 and maxit >= 1");
    if (flags & ~(RTT_SOLVE_ASYNC | RTT_SOLVE_NORMAL_RHS)) return fail(RTT_EINVAL, "unknown ridge_solve flags");
    const bool normal_rhs = (flags & RTT_SOLVE_NORMAL_RHS) != 0;
    if (info) *info = rtt_solve_info{0, 0, 0.f, 0};
    if (nrhs == 0) return RTT_OK;
    hipStream_t s = (hipStream_t)stream;
    const int G = (int)g->members.size();
    const int npair = nrhs * G;
    const int64_t n = g->n_cols, m = g->n_rows;
    int64_t max_cols = 0;
    for (const Member& mb : g->members) max_cols = std::max(max_cols, mb.n_cols);
    Workspace local;
    if (async && !g->solve_ws) g->solve_ws = new (std::nothrow) Workspace(true);
    Workspace& ws = async ? *g->solve_ws : local;
    if (async && !g->solve_ws) return fail(RTT_ENOMEM, "ridge_solve workspace");
    float* r = (float*)ws.get("cg_r", sizeof(float) * (size_t)nrhs * n);
    float* p = (float*)ws.get("cg_p", sizeof(float) * (size_t)nrhs * n);
    float* Ap = (float*)ws.get("cg_ap", sizeof(float) * (size_t)nrhs * n);
    float* q = (float*)ws.get("cg_q", sizeof(float) * (size_t)nrhs * m);
    const int nsl = (int)std::min<int64_t>(std::max<int64_t>(1, max_cols / 1024), CG_SLICES);
    double* sc = (double*)ws.get("cg_scal", sizeof(double) * 4 * npair);
    double* parts = (double*)ws.get("cg_part", sizeof(double) * 2 * (size_t)nsl * npair);
    int* flags_dev = (int*)ws.get("cg_done", sizeof(int) * 2 * npair);
    if (!r || !p || !Ap || !q || !sc || !parts || !flags_dev) return fail(RTT_ENOMEM, "ridge_solve workspace");
    double *rr = sc, *rr_next = sc + npair, *bb = sc + 2 * npair, *pap = sc + 3 * npair;
    double *pap_part = parts, *rr_part = parts + (size_t)nsl * npair;
    int *done = flags_dev, *done_next = flags_dev + npair;
    const int64_t* seg = g->d_seg;   // column blocks
    int rc;
    const dim3 grid((unsigned)nsl, (unsigned)nrhs, (unsigned)G), blk(CG_T);
    const dim3 sgrid((unsigned)((npair + 127) / 128));
    // x = 0, r = A^T y (or the given normal-equation right-hand side), p = r
    if (!normal_rhs && (rc = apply_op(g, -1, true, y, r, nrhs, mask, s))) return rc;
    hipLaunchKernelGGL(k_cg_start, grid, blk, 0, s, normal_rhs ? y : r, r, p, x, seg, n, rr_part);
    hipLaunchKernelGGL(k_cg_init, dim3((unsigned)npair), blk, 0, s, rr_part, nsl, rr, bb, done);
    RTT_HIP(hipGetLastError());
    const double tol2 = (double)tol * (double)tol;
    std::vector<double> h_rr(npair), h_bb(npair);
    std::vector<int> h_done(npair);
    int it = 0;
    if (!async) {
        RTT_HIP(hipMemcpyAsync(h_done.data(), done, sizeof(int) * npair, hipMemcpyDeviceToHost, s));
        RTT_HIP(hipStreamSynchronize(s));
        if (std::all_of(h_done.begin(), h_done.end(), [](int d) { return d != 0; })) {
            if (info) *info = rtt_solve_info{0, npair, 0.f, 0};
            return RTT_OK;
        }
    }
    const int check_every = 8;
    // Where A^T goes by base cells its two launches, the second of which adds to the first, become one that
    // leaves two shares, and the kernel that follows adds them (256^2, one right-hand side: 24.4 -> 15.1 us a
    // product, 20 iterations 1002 -> 814 us).
    // (The buffer depends on the geometry, not on the variant of the moment: a captured solve finds it whatever is pinned.)
    float* Ap2 = nullptr;
    if (G == 1 && adjoint_by_cells(g->members[0])) Ap2 = (float*)ws.get("cg_ap2", sizeof(float) * (size_t)nrhs * n);
    bool parts2 = Ap2 != nullptr;
    if (parts2 && (rc = fill(Ap2, (int64_t)nrhs * n, 0.f, s))) return rc;
    while (it < maxit) {
        if ((rc = apply_op(g, -1, false, p, q, nrhs, mask, s))) return rc;
        rc = RTT_OK;
        parts2 = parts2 && adjoint_parts(g, q, Ap, Ap2, nrhs, mask, s, &rc);
        if (rc || (!parts2 && (rc = apply_op(g, -1, true, q, Ap, nrhs, mask, s)))) return rc;
        hipLaunchKernelGGL(k_cg_pap, grid, blk, 0, s, Ap, parts2 ? Ap2 : nullptr, p, lambda, seg, n, pap_part);
        hipLaunchKernelGGL(k_cg_xr, grid, blk, 0, s, x, r, p, Ap, pap_part, rr, done, seg, n, pap, rr_part);
        hipLaunchKernelGGL(k_cg_p, grid, blk, 0, s, p, r, rr_part, rr, bb, pap, done, seg, n, tol2, rr_next, done_next);
        std::swap(rr, rr_next);
        std::swap(done, done_next);
        RTT_HIP(hipGetLastError());
        ++it;
        if (!async && (it % check_every == 0 || it == maxit)) {
            RTT_HIP(hipMemcpyAsync(h_done.data(), done, sizeof(int) * npair, hipMemcpyDeviceToHost, s));
            RTT_HIP(hipStreamSynchronize(s));
            if (std::all_of(h_done.begin(), h_done.end(), [](int d) { return d != 0; })) break;
        }
    }
    if (resid_dev) hipLaunchKernelGGL(k_cg_resid, sgrid, dim3(128), 0, s, rr, bb, resid_dev, npair);
    RTT_HIP(hipGetLastError());
    if (async) {
        if (info) *info = rtt_solve_info{it, -1, -1.f, 0};
        return RTT_OK;
    }
    RTT_HIP(hipMemcpyAsync(h_rr.data(), rr, sizeof(double) * npair, hipMemcpyDeviceToHost, s));
    RTT_HIP(hipMemcpyAsync(h_bb.data(), bb, sizeof(double) * npair, hipMemcpyDeviceToHost, s));
    RTT_HIP(hipMemcpyAsync(h_done.data(), done, sizeof(int) * npair, hipMemcpyDeviceToHost, s));
    RTT_HIP(hipStreamSynchronize(s));
    double worst = 0.0;
    int ndone = 0;
    for (int v = 0; v < npair; ++v) {
        if (h_bb[v] > 0.0) worst = std::max(worst, std::sqrt(h_rr[v] / h_bb[v]));
        ndone += h_done[v] ? 1 : 0;
    }
    if (info) *info = rtt_solve_info{it, ndone, (float)worst, 0};
    if (ndone < npair) return fail(RTT_ENOCONV, "ridge_solve: CG did not reach tol within maxit");
    return RTT_OK;
}

extern "C" int noise_add(float* y, int64_t n, uint64_t seed, float sigma, void* stream)
{
    if (n < 0) return fail(RTT_EINVAL, "n must be >= 0");
    if (n > 0 && !y) return fail(RTT_EINVAL, "NULL data pointer");
    if (!std::isfinite(sigma)) return fail(RTT_EINVAL, "sigma must be finite");
    return normal_add(y, n, seed, sigma, (hipStream_t)stream);
}
