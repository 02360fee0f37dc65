// A^T, base-cell form (dt_obs/dt_src = 1/Q, Q = 1 or 2): the form for geometries with many rays per
// cell.  A ray feeds the four corners of its base cell only, so the rays of one base cell reduce to
// four sums per hat.  A wave (or S waves, each a share of the cell's rays) walks the rays of one base
// cell over a chunk of hats: it reads NB ray records with scalar loads, forms the transposed hat sum of
// every ray's data row (lanes run over hats; the earlier taps are the previous lane's, taken by a wave
// shift) and adds it into the four corner sums with one 4x4x1 matrix instruction per 64 hats (16
// independent blocks: A = the ray's four corner weights, B = four hats' sums).
//
// A workgroup takes G consecutive base cells of one row; the first one only completes the workgroup's
// first column, the others' left and right sums meet in LDS and leave as G - 1 finished columns of the
// rows ci and ci + 1.  Two base rows share a target row when they are neighbours, so the even base rows
// run first and store, then the odd ones add, in two launches: no atomics, no scratch, bitwise
// reproducible, and the result does not depend on V, NB or NVW.
//
#include <algorithm>

#include "rtt_internal.h"

namespace rtt {
namespace {

constexpr int WAVE = 64;
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i4v __attribute__((ext_vector_type(4)));

struct CellArgs {
    const FwdRec* rec;        // sorted by base cell
    const int32_t* cstart;    // CSR over base cells
    int n_r, n_phi, K, F;
    int pr;                   // row parity of the launch
    int cgroups;              // workgroups along a row of cells
    int kchunks;              // hat chunks per cell (cells_chunk hats each)
    int nvec;
    const float* y;
    float* x;
    float* x2;                // both parities in one launch: the odd rows' share (as x), or NULL
    int64_t y_stride, x_stride;
    uint32_t mask;
};

// Hats per wave: 64 V, less Q when the first Q lanes of the chunk are halo lanes, which load the frames of
// the hats before the chunk and only feed their neighbours (otherwise lane 0 loads those frames too).
template <int Q, int V, bool HALO>
constexpr int cells_chunk() { return WAVE * V - (HALO ? Q : 0); }

// past every row's range, and still past it after the uniform part of an offset is added
constexpr int LANE_OUT = 0x40000000;

// the previous lane's value; lane 0 takes `first`
__device__ __forceinline__ float shr1(float first, float src)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, first), __builtin_bit_cast(int, src),
                                                                 0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}
// the previous lane's value; lane 0 takes lane 63's
__device__ __forceinline__ float ror1(float src)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, src), 0x13C /* wave_ror:1 */, 0xf, 0xf, false));
}

template <int Q, int V, int NB, int NVW, int W, int S, bool HALO>
__global__ __launch_bounds__(W * WAVE, 4) void k_adjoint_cells(CellArgs a)
{
    static_assert(Q == 1 || Q == 2, "frame steps of a whole or half hat");
    static_assert(W % S == 0 && W / S >= 2, "whole cells per workgroup, one of them for the left neighbour");
    static_assert(NB <= FWD_PAD + 1, "a batch reads up to NB - 1 records past its cell");
    constexpr int G = W / S;
    typedef const __attribute__((address_space(4))) int32_t* ci32p;
    typedef const __attribute__((address_space(4))) i4v* ci4p;
    constexpr int H = HALO ? Q : 0;
    constexpr int C = cells_chunk<Q, V, HALO>();
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // consecutive blocks of an XCD take consecutive cells (the hardware deals blocks round robin)
    const unsigned nblk = gridDim.x, bx = blockIdx.x & 7u, bi = blockIdx.x >> 3, per = nblk >> 3, rem = nblk & 7u;
    const int lin = (int)(bx * per + min(bx, rem) + bi);
    const int kch = lin % a.kchunks;
    const int tb = lin / a.kchunks;
    const int pr = a.x2 ? (int)blockIdx.z : a.pr;
    const int ci = pr + 2 * (tb / a.cgroups);
    const int jb = (tb % a.cgroups) * (G - 1);       // first column of the workgroup
    const int grp = wave / S, part = wave % S;
    const int jo = jb + grp - 1;                     // this wave's base column
    const int cj = jo < 0 ? a.n_phi - 1 : jo;
    int w0 = 0, w1 = 0;
    if (ci < a.n_r - 1 && jo < a.n_phi) {            // no ray has its base cell in the last row
        w0 = ((ci32p)a.cstart)[ci * a.n_phi + cj];
        w1 = ((ci32p)a.cstart)[ci * a.n_phi + cj + 1];
    }
    if (S > 1) {
        const int n = w1 - w0, b = w0;
        w0 = b + n * part / S;
        w1 = b + n * (part + 1) / S;
    }
    const int v0 = blockIdx.y * NVW;
    const int nv = min(NVW, a.nvec - v0);
    const int kc = kch * C;
    // hats of this lane: kc - H + lane + 64 v; byte offset of its frame relative to the ray's first hat
    int lane_off[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int kk = lane + WAVE * v;
        lane_off[v] = kc - H + kk < a.K ? Q * kk * 4 : LANE_OUT;
    }
    const int first_off = lane == 0 ? -Q * 4 : LANE_OUT;   // without halo lanes: the frames before lane 0's,
    const int first_off2 = lane == 0 ? -2 * Q * 4 : LANE_OUT;   // and (Q = 2) the pair before those
    const unsigned rowbytes = (unsigned)a.F * 4u;
    const char* ybase[NVW];
#pragma unroll
    for (int u = 0; u < NVW; ++u) ybase[u] = (const char*)(a.y + (int64_t)(v0 + (u < nv ? u : 0)) * a.y_stride);

    f4 acc[NVW][V];
#pragma unroll
    for (int u = 0; u < NVW; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[u][v] = (f4){0.f, 0.f, 0.f, 0.f};

    for (int e = w0; e < w1; e += NB) {
        // the batch's records; those past the end of the range are read (they exist: the next cell's, or
        // the padding of the record array) and switched off below
        const FwdRec* __restrict__ rb = a.rec + e;
        i4v rec[NB];
        float th[NB], bw[NB];
        int org[NB];
        bool half[NB];
        unsigned roff[NB], range[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            rec[j] = *(ci4p)((const char*)rb + j * sizeof(FwdRec) + offsetof(FwdRec, k0));   // k0, th0, row, order
            bw[j] = (&rb[j].b00)[lane & 3];   // lane l: corner weight l mod 4 (matrix operand A)
        }
        __builtin_amdgcn_sched_barrier(0);    // every scalar load is issued before the first is used
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const i4v q = rec[j];
            const int thb = q.y;
            org[j] = q.x;
            if constexpr (Q == 1) {
                th[j] = __builtin_bit_cast(float, thb);
            } else {
                // half steps: hat k takes the frames 2 (k - k0) - s + {-2, -1, 0, 1} with the weights
                // r, 1/2 + r, 1 - r, 1/2 - r, where th0 = s / 2 + r (th0 in [0, 1]: its bits compare)
                half[j] = (unsigned)thb >= 0x3F000000u;
                th[j] = __builtin_bit_cast(float, thb) - (half[j] ? 0.5f : 0.f);
            }
            roff[j] = (unsigned)q.z * rowbytes;
            // a switched-off ray reads zeros, without touching memory
            const int in = ((e - w1) + j) >> 31, sel = (int)(a.mask << (31 - (unsigned)q.w)) >> 31;
            range[j] = rowbytes & (unsigned)(in & sel);
        }
        f2 yv[NB][NVW][V], fv[NB][NVW], gv[NB][NVW];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int ub = Q * (kc - H - org[j]) * 4;
#pragma unroll
            for (int u = 0; u < NVW; ++u) {
                const __amdgpu_buffer_rsrc_t ry =
                    __builtin_amdgcn_make_buffer_rsrc((void*)(ybase[u] + roff[j]), (short)0, (int)range[j], 0x00020000);
                // the frame (Q = 1) or the frame pair (Q = 2, even rows: inside the row or outside)
                // of a hat; frames outside [0, F) read 0 (an earlier frame's offset wraps past the range)
                auto ld = [&](int off) -> f2 {
                    if constexpr (Q == 1)
                        return (f2){__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ry, off, 0, 0)), 0.f};
                    else
                        return __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(ry, off, 0, 0));
                };
#pragma unroll
                for (int v = 0; v < V; ++v) yv[j][u][v] = ld(lane_off[v] + ub);
                if constexpr (!HALO) {
                    fv[j][u] = ld(first_off + ub);
                    if constexpr (Q == 2) gv[j][u] = ld(first_off2 + ub);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if constexpr (Q == 2) {
                if (half[j]) {   // (uniform) odd first frame: pairs move by one frame
#pragma unroll
                    for (int u = 0; u < NVW; ++u) {
                        float prev = 0.f;
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            const f2 y = yv[j][u][v];
                            const float sh = v > 0 ? shr1(ror1(prev), y[1]) : HALO ? ror1(y[1]) : shr1(fv[j][u][1], y[1]);
                            prev = y[1];
                            yv[j][u][v] = (f2){sh, y[0]};
                        }
                        if constexpr (!HALO) fv[j][u] = (f2){gv[j][u][1], fv[j][u][0]};
                    }
                }
            }
            // weights of the earlier (e) and the later (l) taps
            const float r = th[j];
            const float we0 = r, we1 = 0.5f + r, wl0 = 1.0f - r, wl1 = 0.5f - r;
#pragma unroll
            for (int u = 0; u < NVW; ++u) {
                float prev = 0.f;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    // later taps of this hat, earlier taps of the next one (which the next lane adds)
                    const f2 y = yv[j][u][v];
                    float l = wl0 * y[0], en = we0 * y[0];
                    if constexpr (Q == 2) {
                        l += wl1 * y[1];
                        en += we1 * y[1];
                    }
                    float sh;
                    if (v > 0) {
                        sh = shr1(ror1(prev), en);
                    } else if constexpr (HALO) {
                        sh = ror1(en);
                    } else {
                        float f = we0 * fv[j][u][0];
                        if constexpr (Q == 2) f += we1 * fv[j][u][1];
                        sh = shr1(f, en);
                    }
                    prev = en;
                    acc[u][v] = __builtin_amdgcn_mfma_f32_4x4x1f32(bw[j], l + sh, acc[u][v], 0, 0, 0);
                }
            }
        }
    }

    // register c of acc: the corner in row ci + (c & 1), column cj (c < 2) or the next one.  Every
    // column is the sum of its own cell's left corners and the previous cell's right corners, the
    // parts of a cell added in part order.
    __shared__ float red[W][4][V][WAVE];
#pragma unroll
    for (int u = 0; u < NVW; ++u) {
        if (u > 0) __syncthreads();
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int c = 0; c < 4; ++c) red[wave][c][v][lane] = acc[u][v][c];
        __syncthreads();
        if (u >= nv || grp == 0 || jo >= a.n_phi) continue;
        // the 2 V (row, slot) pieces of the column over the cell's S waves
#pragma unroll
        for (int i = 0; i < 2 * V; ++i) {
            if (i % S != part) continue;
            const int r = i / V, v = i % V;
            float left = red[grp * S][r][v][lane], right = red[(grp - 1) * S][2 + r][v][lane];
#pragma unroll
            for (int q = 1; q < S; ++q) {
                left += red[grp * S + q][r][v][lane];
                right += red[(grp - 1) * S + q][2 + r][v][lane];
            }
            const int k = kc - H + lane + WAVE * v;
            if (k < kc || k >= a.K || ci + r >= a.n_r) continue;
            float* __restrict__ p = (pr && a.x2 ? a.x2 : a.x) + (int64_t)(v0 + u) * a.x_stride + ((int64_t)(ci + r) * a.n_phi + jo) * a.K + k;
            *p = pr == 0 || a.x2 ? left + right : *p + (left + right);
        }
    }
}

template <int Q, int V, int NB, int NVW, int W, int S, bool HALO>
void cells_launch(CellArgs a, hipStream_t s)
{
    // the halo lane when it costs no extra chunk
    if constexpr (HALO) {
        if ((a.K + cells_chunk<Q, V, true>() - 1) / cells_chunk<Q, V, true>() > (a.K + WAVE * V - 1) / (WAVE * V)) {
            cells_launch<Q, V, NB, NVW, W, S, false>(a, s);
            return;
        }
    }
    constexpr int C = cells_chunk<Q, V, HALO>(), G = W / S;
    a.kchunks = (a.K + C - 1) / C;
    a.cgroups = (a.n_phi + G - 2) / (G - 1);
    if (a.x2) {
        hipLaunchKernelGGL((k_adjoint_cells<Q, V, NB, NVW, W, S, HALO>),
                           dim3((unsigned)((a.n_r + 1) / 2) * (unsigned)a.cgroups * (unsigned)a.kchunks,
                                (unsigned)((a.nvec + NVW - 1) / NVW), 2),
                           dim3(W * WAVE), 0, s, a);
        return;
    }
    for (a.pr = 0; a.pr < 2; ++a.pr) {
        // the even rows take the last row too (it has no rays of its own but may have to be cleared)
        const int rows = a.pr == 0 ? (a.n_r + 1) / 2 : (a.n_r - 1) / 2;
        if (rows == 0) continue;
        hipLaunchKernelGGL((k_adjoint_cells<Q, V, NB, NVW, W, S, HALO>),
                           dim3((unsigned)rows * (unsigned)a.cgroups * (unsigned)a.kchunks, (unsigned)((a.nvec + NVW - 1) / NVW)),
                           dim3(W * WAVE), 0, s, a);
    }
}

template <int Q, int V, int NB, int W, int S>
void cells_nvw(const CellArgs& a, hipStream_t s)
{
    if (a.nvec >= 2) cells_launch<Q, V, NB / 2, 2, W, S, true>(a, s);
    else cells_launch<Q, V, NB, 1, W, S, true>(a, s);
}

template <int Q, int W, int S>
void cells_dispatch(const CellArgs& a, hipStream_t s)
{
    // Hat slots per lane: the fewest lanes over all chunks, a visit's set-up counted as 40 lanes (256^2
    // with 200 hats, one vector: 1 slot 25.5 us, 2 slots 21.9, 3 slots 24.4; 200^2 with 130 hats, 8
    // vectors: 45, 45, 43).  Q = 1 stops at 3 slots (4 are slower at 256 hats: 252 against 237 us), Q = 2
    // has 1, 2 or 4 (512^2 with 256 hats: 154, 143, 134 us).
    int best = 0, cost = 0;
    for (int v : {1, 2, 3, 4}) {
        if (v == (Q == 1 ? 4 : 3)) continue;
        const int c = WAVE * v;   // (halo lanes are given up where they would add a chunk)
        const int cst = ((a.K + c - 1) / c) * (c + 40);
        if (best == 0 || cst < cost) {
            best = v;
            cost = cst;
        }
    }
    switch (best) {
    case 1: cells_nvw<Q, 1, 8, W, S>(a, s); break;
    case 2: cells_nvw<Q, 2, 8 / Q, W, S>(a, s); break;
    default: cells_nvw<Q, Q == 1 ? 3 : 4, 4, W, S>(a, s); break;
    }
}

template <int Q>
void cells_split(const CellArgs& a, int64_t rays_per_cell, hipStream_t s)
{
    // Waves per cell, by the geometry alone (the order of additions depends on it): one wave walks up
    // to 20 rays by itself (200^2, 13 rays a cell, 64 vectors: 316 us on one wave, 345 on two); 256^2, 46
    // rays a cell, one vector: 33 us on one wave, 22 on two, 25 on four.
    if (rays_per_cell < 20) cells_dispatch<Q, 8, 1>(a, s);
    else if (rays_per_cell < 80) cells_dispatch<Q, 8, 2>(a, s);
    else cells_dispatch<Q, 16, 4>(a, s);
}

}  // namespace

bool adjoint_cells_ok(const Member& m)
{
    const int64_t lim = (int64_t)1 << 26;   // offsets 4 Q (k - k0) stay far inside 32 bits
    return m.P == 1 && (m.Q == 1 || m.Q == 2) && m.grid.n_frames < lim && m.grid.n_hat < lim &&
           m.n_rows < ((int64_t)1 << 30) && m.k0_min > -lim && m.k0_max < lim && (int64_t)m.grid.n_r * m.grid.n_phi < ((int64_t)1 << 28);
}

int launch_adjoint_cells(const rtt_geometry* g, const Member& m, const float* y, float* x, int nvec, int64_t y_stride,
                         int64_t x_stride, uint32_t mask, hipStream_t s, float* x2)
{
    CellArgs a{};
    a.rec = g->d_fwd + m.ray_begin;
    a.cstart = g->d_cell_start + m.cell_begin;
    a.n_r = m.grid.n_r;
    a.n_phi = m.grid.n_phi;
    a.K = m.grid.n_hat;
    a.F = m.grid.n_frames;
    a.nvec = nvec;
    a.y = y;
    a.x = x;
    a.x2 = x2;
    a.y_stride = y_stride;
    a.x_stride = x_stride;
    a.mask = mask;
    const int64_t per_cell = m.n_rays / std::max<int64_t>(1, (int64_t)(m.grid.n_r - 1) * m.grid.n_phi);
    if (m.Q == 1) cells_split<1>(a, per_cell, s);
    else cells_split<2>(a, per_cell, s);
    RTT_HIP(hipGetLastError());
    return RTT_OK;
}

}  // namespace rtt
