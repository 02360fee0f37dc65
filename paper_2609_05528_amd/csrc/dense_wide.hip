// Gram and combine products of wide blocks (more than 32 vectors) on gfx950.
//
// gram_split: upper tiles of G = Y Y^T on the bf16 matrix cores with FP32 accuracy.  Every FP32 operand x is
// written as x = h + m + l with bf16 parts (round to nearest each time: the three parts hold 24 significand
// bits, so the sum is x), and a product is formed from the six partial products h h, h m, m h, m m, h l, l h,
// each exact in FP32; the three left out are below 2^-26 of the product.  A 32 x 32 x 16 step costs 6 x 32
// cycles instead of the 8 x 64 of the FP32 form.  A workgroup of 8 waves takes one slice of the long dimension
// and all tiles: a 32-column chunk of every row is split once into LDS (rows padded to 80 bytes, which
// spreads a fragment's 16-byte reads over all banks), and each wave owns up to 7 tiles.  Every element is
// read from memory once; the 64 x 64 blocks of the FP32 form read it 4.5 times.  (Parts below 2^-126 vanish,
// so values below about 2^-110 lose relative accuracy; an infinity gives NaN.)
// 288 vectors of 1.55M: 1.85 -> 1.03 ms alone with random rows (0.72 to 0.75 in an rSVD's trace), of which 0.01 the
// FP64 sum of the partials; rms error of the normalised Gram matrix 1.6e-8 -> 3e-9.  The matrix cores are 59% busy
// (rank-256 rSVD), the waves wait for LDS fragments and at the chunk barriers.
//
// combine_wide: Out = beta Out + C^T Y with FP32 matrix instructions.  A wave owns 32 columns and up to 9 row
// blocks of Out; its columns of Y go from memory to registers, 16 rows two steps ahead, and C comes through
// LDS in fragment order.  Y is read once, against three passes with 4 row blocks each.  288 x 288 upper
// triangular over 1.55M columns: 1.81 -> 1.56 ms (0.56 -> 0.45 over 393k; 1.66 and 0.48 with the wait for the
// next C in front of a step's products, which left the rows of Y one step to arrive), bound by the FP32 matrix
// rate (143 GFLOP, 0.93 ms at the rate of a large library product) and the 3.6 GB moved (0.76 ms).  The bf16 split of the Gram form was measured
// here too (1.37 ms) and dropped: its matrix instructions cut the small terms of a step off towards zero where
// one term is much larger (R^-1 of a second pass: 1 beside 1e-4), as if the coefficients were off by up to
// 1.5e-8, and the TSVD estimate at rank 256 lost a digit (1e-5 against 1.5e-6).
#include <algorithm>

#include "dense.h"

namespace rtt {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 b2v __attribute__((ext_vector_type(2)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// the three bf16 parts of two floats, each pair packed (first in the low half)
struct Split2 {
    uint32_t h, m, l;
};
__device__ __forceinline__ uint32_t pack_bf16(f2v x)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, b2v));
}
__device__ __forceinline__ f2v unpack_bf16(uint32_t p)
{
    return (f2v){__builtin_bit_cast(float, p << 16), __builtin_bit_cast(float, p & 0xffff0000u)};
}
__device__ __forceinline__ Split2 split2(float x0, float x1)
{
    Split2 s;
    f2v r = {x0, x1};
    s.h = pack_bf16(r);
    r -= unpack_bf16(s.h);
    s.m = pack_bf16(r);
    r -= unpack_bf16(s.m);
    s.l = pack_bf16(r);
    return s;
}

__device__ __forceinline__ f16v mfma_bf16(u4v a, u4v b, f16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, b), c, 0, 0, 0);
}
// the six partial products, the small ones first
__device__ __forceinline__ f16v mfma_split(const u4v* a, const u4v* b, f16v c)
{
    c = mfma_bf16(a[0], b[2], c);
    c = mfma_bf16(a[2], b[0], c);
    c = mfma_bf16(a[1], b[1], c);
    c = mfma_bf16(a[0], b[1], c);
    c = mfma_bf16(a[1], b[0], c);
    return mfma_bf16(a[0], b[0], c);
}

constexpr int SW = 8;                 // waves per workgroup
constexpr int SCOL = 32;              // columns of a Gram chunk
constexpr int SROW = SCOL + 8;        // bf16 values per padded row in LDS

// M = 32 T rows, 16-byte aligned rows when VL
template <int T, bool VL>
__global__ __launch_bounds__(SW * 64, 2) void k_gram_split(const float* __restrict__ Y, int64_t ld, int64_t L, int64_t slice,
                                                           float* __restrict__ part, const int* __restrict__ run_if)
{
    if (run_if && !*run_if) return;
    constexpr int M = 32 * T, NTILE = T * (T + 1) / 2, NT = (NTILE + SW - 1) / SW;
    constexpr int NQ = M * (SCOL / 4);                      // 16-byte groups of a chunk
    constexpr int NL = (NQ + SW * 64 - 1) / (SW * 64);      // per thread
    __shared__ __attribute__((aligned(16))) uint16_t lds[2][3][M][SROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t l0 = (int64_t)blockIdx.x * slice, l1 = min(L, l0 + slice);
    // this wave's tiles: consecutive in the row-major list of upper tiles (the last wave repeats the last one)
    int bm[NT], bn[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        int t = min(wave * NT + i, NTILE - 1), r = 0;
        while (t >= T - r) {
            t -= T - r;
            ++r;
        }
        bm[i] = r;
        bn[i] = r + t;
    }
    // this thread's groups of a chunk (threads past the last group repeat it)
    int row[NL], col4[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int e = min(tid + q * SW * 64, NQ - 1);
        row[q] = e / (SCOL / 4);
        col4[q] = (e % (SCOL / 4)) * 4;
    }
    f4v raw[NL];
    auto load_full = [&](int64_t lc, int q) {
        const float* __restrict__ p = Y + (int64_t)row[q] * ld + lc + col4[q];
        if (VL) raw[q] = *(const f4v*)p;
        else raw[q] = (f4v){p[0], p[1], p[2], p[3]};
    };
    auto load_edge = [&](int64_t lc) {
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int64_t l = lc + col4[q];
            const float* __restrict__ p = Y + (int64_t)row[q] * ld + l;
#pragma unroll
            for (int t = 0; t < 4; ++t) raw[q][t] = l + t < l1 ? p[t] : 0.f;
        }
    };
    auto load = [&](int64_t lc) {
        if (lc + SCOL <= l1) {
#pragma unroll
            for (int q = 0; q < NL; ++q) load_full(lc, q);
        } else {
            load_edge(lc);
        }
    };
    auto store = [&](int buf, int q) {
        const Split2 a = split2(raw[q][0], raw[q][1]), b = split2(raw[q][2], raw[q][3]);
        *(u2v*)&lds[buf][0][row[q]][col4[q]] = (u2v){a.h, b.h};
        *(u2v*)&lds[buf][1][row[q]][col4[q]] = (u2v){a.m, b.m};
        *(u2v*)&lds[buf][2][row[q]][col4[q]] = (u2v){a.l, b.l};
    };
    f16v acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = (f16v){};
    const int fr = lane & 31, fk = (lane >> 5) * 8;         // fragment row and first k of this lane
    // A chunk's products are summed from zero and then added to the accumulators: the matrix cores round the
    // sum of a long chain down a little each time (288 rows of 1.5M: diagonal off by 1.9e-6 without, 2e-8 with,
    // 3e-7 in the FP32 form).
    auto tile = [&](int buf, int i) {
        f16v t = (f16v){};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u4v a[3], b[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                a[p] = *(const u4v*)&lds[buf][p][bm[i] * 32 + fr][16 * ks + fk];
                b[p] = *(const u4v*)&lds[buf][p][bn[i] * 32 + fr][16 * ks + fk];
            }
            t = mfma_split(a, b, t);
        }
        acc[i] += t;
    };
    load(l0);
#pragma unroll
    for (int q = 0; q < NL; ++q) store(0, q);
    if (l0 + SCOL < l1) load(l0 + SCOL);
    __syncthreads();
    int buf = 0;
    int64_t lc = l0;
    // The next chunk is split into the other buffer and the one after it loaded while this one's tiles are
    // multiplied, a piece per tile, so that the vector and the matrix instructions of a wave overlap.
    for (; lc + 3 * SCOL <= l1; lc += SCOL) {
#pragma unroll
        for (int i = 0; i < (NT > NL ? NT : NL); ++i) {
            if (i < NL) {
                store(buf ^ 1, i);
                load_full(lc + 2 * SCOL, i);
            }
            if (i < NT) tile(buf, i);
        }
        __syncthreads();
        buf ^= 1;
    }
    for (; lc < l1; lc += SCOL) {
        if (lc + SCOL < l1) {
#pragma unroll
            for (int q = 0; q < NL; ++q) store(buf ^ 1, q);
        }
        if (lc + 2 * SCOL < l1) load(lc + 2 * SCOL);
#pragma unroll
        for (int i = 0; i < NT; ++i) tile(buf, i);
        __syncthreads();
        buf ^= 1;
    }
    float* __restrict__ out = part + (int64_t)blockIdx.x * M * M;
    const int col = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        if (wave * NT + i >= NTILE) break;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int ii = bm[i] * 32 + 8 * (r >> 2) + 4 * hi + (r & 3), jj = bn[i] * 32 + col;
            out[(int64_t)ii * M + jj] = acc[i][r];
        }
    }
}

// C (K x M) in fragment order: frag[((step * nb + block) * 2 + part) * 64 + lane] holds the rows
// 16 step + 8 (lane / 32) + 4 part + 0 .. 3 of column 32 block + lane % 32.  The last step moves back to end
// at K: the rows that the step before had already are zero there, and so are columns past M.
__global__ __launch_bounds__(64) void k_coef_frag(const float* __restrict__ C, int K, int M, int nb, f4v* __restrict__ frag,
                                                  const int* __restrict__ run_if)
{
    if (run_if && !*run_if) return;
    const int lane = threadIdx.x, t = blockIdx.x, g = blockIdx.y;
    const int kb = min(16 * t, K - 16) + (lane >> 5) * 8, m = g * 32 + (lane & 31);
    f4v* __restrict__ o = frag + ((int64_t)t * nb + g) * 2 * 64 + lane;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        f4v x;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = kb + 4 * p + i;
            x[i] = (m < M && k >= 16 * t) ? C[(int64_t)k * M + m] : 0.f;
        }
        o[p * 64] = x;
    }
}

// MG 32-row blocks of Out from block g0 on, C in the order of k_coef_frag (nb blocks).  upper: C[k][m] = 0
// for k > m.  A step's eight 32 x 32 x 2 products take the rows j and 8 + j of the step.
template <int MG>
__global__ __launch_bounds__(SW * 64, 2) void k_combine_wide(const f4v* __restrict__ frag, int nb, int K, int M, int g0,
                                                             const float* __restrict__ Y, int64_t ldy,
                                                             float* __restrict__ Out, int64_t ldo, int64_t L, float beta,
                                                             int upper, const int* __restrict__ run_if)
{
    if (run_if && !*run_if) return;
    constexpr int NU = MG * 2 * 64;                          // 16-byte units of a 16-row step of C
    constexpr int NC = (NU + SW * 64 - 1) / (SW * 64);
    __shared__ __attribute__((aligned(16))) f4v cs[2][MG * 2][64];
    const int m0 = g0 * 32;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t l = ((int64_t)blockIdx.x * SW + wave) * 32 + (lane & 31);
    const int half = lane >> 5;
    const int64_t lc = l < L ? l : L - 1;                    // lanes past the end read the last column, store nothing
    // uniform row address plus a 32-bit offset per lane (half 1 takes the rows 8 .. 15 of a step)
    const uint32_t yoff = (uint32_t)(((int64_t)half * 8 * ldy + lc) * 4);
    const int kend = upper ? min(K, m0 + MG * 32) : K;
    const int klast = (kend - 1) & ~15;
    f4v cr[NC];
    auto load_c = [&](int k0) {
        const f4v* __restrict__ p = frag + ((int64_t)(min(k0, klast) >> 4) * nb + g0) * 2 * 64;
#pragma unroll
        for (int q = 0; q < NC; ++q) cr[q] = p[min(tid + q * SW * 64, NU - 1)];
    };
    auto store_c = [&](int buf) {
        f4v* __restrict__ o = &cs[buf][0][0];
#pragma unroll
        for (int q = 0; q < NC; ++q) o[min(tid + q * SW * 64, NU - 1)] = cr[q];
    };
    float ya[8], yb[8];
    auto load_y = [&](int k0, float* y) {
        const char* __restrict__ p = (const char*)(Y + (int64_t)min(min(k0, klast), K - 16) * ldy) + yoff;
#pragma unroll
        for (int t = 0; t < 8; ++t) y[t] = *(const float*)(p + (int64_t)t * ldy * 4);
    };
    f16v acc[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g) acc[g] = (f16v){};
    int buf = 0;
    // One 16-row step: y holds its rows of Y, then receives those two steps ahead.  The next step's C goes to LDS
    // at the end: the wait for it covers the loads that are older, the rows of Y of the next step, and not the
    // ones issued here, which have two steps to arrive.  Loads past the last step repeat it (no branch around
    // a load: the compiler would wait for all of them at the join).
    auto step = [&](int k0, float* y) {
        float b[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) b[t] = y[t];
        load_y(k0 + 32, y);
        // row blocks that end before k0 are exact zeros; a step past the last does nothing
        const int gmin = k0 >= kend ? MG : upper && k0 > m0 ? (k0 - m0) >> 5 : 0;
#pragma unroll
        for (int g = 0; g < MG; ++g)
            if (g >= gmin) {
                const f4v a0 = cs[buf][2 * g][lane], a1 = cs[buf][2 * g + 1][lane];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    acc[g] = __builtin_amdgcn_mfma_f32_32x32x2f32(t < 4 ? a0[t & 3] : a1[t & 3], b[t], acc[g], 0, 0, 0);
            }
        store_c(buf ^ 1);
        load_c(k0 + 32);
        __syncthreads();
        buf ^= 1;
    };
    load_c(0);
    load_y(0, ya);
    load_y(16, yb);
    store_c(0);
    load_c(16);
    __syncthreads();
    for (int k0 = 0; k0 < kend; k0 += 32) {
        step(k0, ya);
        step(k0 + 16, yb);
    }
    if (l >= L) return;
#pragma unroll
    for (int g = 0; g < MG; ++g) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + g * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            if (m < M) {
                float* o = Out + (int64_t)m * ldo + l;
                if (beta == 0.f) __builtin_nontemporal_store(acc[g][r], o);
                else *o = beta * (*o) + acc[g][r];
            }
        }
    }
}

template <int T>
void gram_t(const float* Y, int64_t ld, int64_t L, int64_t slice, int nsplit, bool vl, float* part, const int* run_if,
            hipStream_t s)
{
    if (vl) hipLaunchKernelGGL((k_gram_split<T, true>), dim3((unsigned)nsplit), dim3(SW * 64), 0, s, Y, ld, L, slice, part, run_if);
    else hipLaunchKernelGGL((k_gram_split<T, false>), dim3((unsigned)nsplit), dim3(SW * 64), 0, s, Y, ld, L, slice, part, run_if);
}

template <int MG>
void combine_t(const f4v* frag, int nb, int K, int M, int g0, const float* Y, int64_t ldy, float* Out, int64_t ldo, int64_t L,
               float beta, int upper, hipStream_t s, const int* run_if)
{
    hipLaunchKernelGGL((k_combine_wide<MG>), dim3((unsigned)((L + SW * 32 - 1) / (SW * 32))), dim3(SW * 64), 0, s, frag,
                       nb, K, M, g0, Y, ldy, Out, ldo, L, beta, upper, run_if);
}

}  // namespace

int gram_split_slices(int64_t L, int64_t* slice)
{
    // one workgroup per CU (its LDS allows no second one at 288 rows; 512 slices were slower, 1.13 against 1.05
    // ms, for their partials); whole chunks
    int n = (int)std::min<int64_t>(std::max<int64_t>(1, L / 1024), 256);
    *slice = ((L + n - 1) / n + SCOL - 1) / SCOL * SCOL;
    return (int)((L + *slice - 1) / *slice);
}

void gram_split(const float* Y, int64_t ld, int M, int64_t L, int64_t slice, int nsplit, float* part, hipStream_t s,
                const int* run_if)
{
    const bool vl = (((uintptr_t)Y) & 15) == 0 && (ld % 4) == 0;
    switch (M / 32) {
    case 2: gram_t<2>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 3: gram_t<3>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 4: gram_t<4>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 5: gram_t<5>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 6: gram_t<6>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 7: gram_t<7>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 8: gram_t<8>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    case 9: gram_t<9>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    default: gram_t<10>(Y, ld, L, slice, nsplit, vl, part, run_if, s); break;
    }
}

size_t combine_wide_bytes(int K, int M) { return (size_t)((K + 15) / 16) * ((M + 31) / 32) * 2 * 64 * sizeof(f4v); }

void combine_wide(void* scratch, const float* C, int K, int M, const float* Y, int64_t ldy, float* Out, int64_t ldo, int64_t L,
                  float beta, int upper, hipStream_t s, const int* run_if)
{
    const int nb = (M + 31) / 32;
    f4v* p = (f4v*)scratch;
    hipLaunchKernelGGL(k_coef_frag, dim3((unsigned)((K + 15) / 16), (unsigned)nb), dim3(64), 0, s, C, K, M, nb, p, run_if);
    // the fewest launches of at most 9 row blocks (144 accumulators, two waves per SIMD), of equal size
    const int nl = (nb + 8) / 9, per = (nb + nl - 1) / nl;
    for (int b = 0; b < nb; b += per) {
        switch (std::min(per, nb - b)) {
#define RTT_CW(MG_) combine_t<MG_>(p, nb, K, M, b, Y, ldy, Out, ldo, L, beta, upper, s, run_if)
        case 1: RTT_CW(1); break;
        case 2: RTT_CW(2); break;
        case 3: RTT_CW(3); break;
        case 4: RTT_CW(4); break;
        case 5: RTT_CW(5); break;
        case 6: RTT_CW(6); break;
        case 7: RTT_CW(7); break;
        case 8: RTT_CW(8); break;
        default: RTT_CW(9); break;
#undef RTT_CW
        }
    }
}

}  // namespace rtt
