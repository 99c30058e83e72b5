// Full-4PCF contraction on the matrix cores for any Lambda = (la, lb, lc) with l <= 10 and up to
// 10 bins (float32): the ones without a compile-time kernel of quad_mfma.h.  The sums are those of
// that file,
//   L_mc[b1 b2](x) = sum_ma C(ma, mb, mc) a^b1_{la,ma}(x) a^b2_{lb,mb}(x),  mb = -ma - mc
//   Z[b1 b2][b3]  += sum_x Re( L_mc[b1 b2](x) w(x) a^b3_{lc,mc}(x) )      (Im for odd Lambda),
// with the coupling on the vector ALUs and the sum over the cells as 16x16x4 float32 MFMAs
// (M = 16 pairs, N = b3 padded to 16, K = the cells of the four lane groups).
//
// The orders are known at run time only, so the coefficients are read from the staged tile in LDS
// and the 3j terms from a table by uniform (scalar) loads.  What bounds such a loop is the LDS
// read per product, so a lane computes a T x T block of pairs per term: lane row i of every M tile
// is (i1, i2) = (i / 4, i % 4) and tile (t1, t2) holds the pairs b1 = i1 + 4 t1, b2 = i2 + 4 t2, which
// takes 2 T reads for T^2 products (T = 3 for 9 or 10 bins: 6 reads of 512 B a wave, 24 LDS cycles,
// for 36 FMAs, 72 cycles of one of the four SIMDs).  la = lb computes only the tiles t1 <= t2
// (Z[b2][b1] = +-Z[b1][b2]).  The next term's values are in flight during the current one, and the
// table comes kGRun terms to a scalar load, a run ahead (read one by one, each term waited for its
// scalar load: 2.8 ms against 2.3).
// Measured on 64^3 cells, 10 bins, lmax 5, odd parity (14 canonical Lambda): 2.3 ms, where the vector
// kernel (quad_kernel), with its two LDS reads for every product, takes 13.8.  No unit is
// full (at 3.5 waves a SIMD the vector ALUs are busy 42 % of the cycles, at two an instruction, the LDS 37 %,
// the matrix cores 23 %): staging 16 cells at a time leaves nothing to overlap with, and 30 % of the
// coupling is spent on the bins that pad 10 to 12.
//
// LDS: one row of ncol x 4 T float2 per cell padded to an odd length; lane group g reads cells 4 apart,
// so the 16 values of a read (4 cells, 4 bins) and the 16 cells of a store fall on distinct banks.
#include <algorithm>

#include "sb_kgen.h"

namespace sb {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) QuadGTerm *TermPtr;   // scalar loads
typedef const __attribute__((address_space(4))) int *IntPtr;

constexpr int kLdsBudget = 37 * 1024;   // with the row table, four workgroups a CU
constexpr int kMaxTile = 64;
constexpr int kBatch = 10;              // rows in flight per thread while staging

__host__ __device__ constexpr int row_pitch(int ncol, int t) { return ncol * 4 * t + 1; }
// cells staged at once: a multiple of 16 (every wave takes four at a time)
__host__ __device__ constexpr int tile_cells(int ncol, int t) {
    const int k = kLdsBudget / (16 * row_pitch(ncol, t) * (int)sizeof(float2));
    return 16 * (k < 1 ? 1 : k > kMaxTile / 16 ? kMaxTile / 16 : k);
}

// The tile's contribution of one wave to acc: the wave's cells in steps of four.
template <int T, bool ODD, bool SYM>
__device__ __forceinline__ void contract_tile_cells(const float2 *tile, const float *wt, int tc, int S, int offc, TermPtr terms,
                                                    int t0, int t1, int wave, int i, int g,
                                                    f4v (&acc)[SYM ? T * (T + 1) / 2 : T * T]) {
    constexpr int NT = SYM ? T * (T + 1) / 2 : T * T;
    const int i1 = i >> 2, i2 = i & 3;
    const int ib = i < 4 * T ? i : 0;
    for (int s = 0; s < tc; s += 16) {
        const int cell = s + 4 * g + wave;
        const float2 *row = tile + cell * S;
        const float2 *r1 = row + i1, *r2 = row + i2, *rc = row + offc + ib;
        const float wv = i < 4 * T ? wt[cell] : 0.f;
        float2 L[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) L[k] = make_float2(0.f, 0.f);
        float2 n1[T], n2[T];
        auto fetch = [&](const QuadGTerm &q) {
#pragma unroll
            for (int k = 0; k < T; ++k) n1[k] = r1[(q.off & 0xffffu) + 4 * k];
#pragma unroll
            for (int k = 0; k < T; ++k) n2[k] = r2[(q.off >> 16) + 4 * k];
        };
        QuadGTerm cur[kGRun], nxt[kGRun];
        auto run_at = [&](int t, QuadGTerm *q) {
#pragma unroll
            for (int j = 0; j < kGRun; ++j) {
                q[j].off = terms[t + j].off; q[j].c = terms[t + j].c; q[j].flags = terms[t + j].flags;
            }
        };
        run_at(t0, nxt);
        fetch(nxt[0]);
        for (int tr = t0; tr < t1; tr += kGRun) {
#pragma unroll
            for (int j = 0; j < kGRun; ++j) cur[j] = nxt[j];
            run_at(min(tr + kGRun, t1 - kGRun), nxt);   // past the end: the last run again
#pragma unroll
            for (int j = 0; j < kGRun; ++j) {
            float2 x1[T], u[T];
            const uint32_t flags = cur[j].flags;
            const float c = cur[j].c, c2 = __uint_as_float(__float_as_uint(c) ^ (flags & kGConj2));
            const float s1 = __uint_as_float(0x3f800000u | (flags << 1 & kGConj2));
#pragma unroll
            for (int k = 0; k < T; ++k) {
                x1[k] = n1[k];
                u[k] = make_float2(c * n2[k].x, c2 * n2[k].y);
            }
            fetch(j + 1 < kGRun ? cur[j + 1] : nxt[0]);
            if (flags & kGPaired) {
                // mc = 0: the terms +-ma together, real (even Lambda) or imaginary (odd)
                int k = 0;
#pragma unroll
                for (int a = 0; a < T; ++a)
#pragma unroll
                    for (int b = SYM ? a : 0; b < T; ++b, ++k) {
                        if (!ODD) {
                            L[k].x = __builtin_fmaf(x1[a].x, u[b].x, L[k].x);
                            L[k].x = __builtin_fmaf(x1[a].y, u[b].y, L[k].x);
                        } else {
                            L[k].y = __builtin_fmaf(x1[a].y, u[b].x, L[k].y);
                            L[k].y = __builtin_fmaf(-x1[a].x, u[b].y, L[k].y);
                        }
                    }
            } else {
                int k = 0;
#pragma unroll
                for (int a = 0; a < T; ++a) {
                    const float y1 = s1 * x1[a].y;
#pragma unroll
                    for (int b = SYM ? a : 0; b < T; ++b, ++k) {
                        L[k].x = __builtin_fmaf(x1[a].x, u[b].x, L[k].x);
                        L[k].x = __builtin_fmaf(-y1, u[b].y, L[k].x);
                        L[k].y = __builtin_fmaf(x1[a].x, u[b].y, L[k].y);
                        L[k].y = __builtin_fmaf(y1, u[b].x, L[k].y);
                    }
                }
            }
            if (flags & kGLast) {   // this mc is complete: contract over the four cells
                const float2 v = rc[(flags >> 8 & 255u) * 4 * T];
                const float bx = wv * v.x, by = wv * v.y;
                // even: Re(L a) = L.x a.x - L.y a.y; odd: Im(L a) = L.y a.x + L.x a.y; a_{l0} is real
#pragma unroll
                for (int k = 0; k < NT; ++k)
                    acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(ODD ? L[k].y : L[k].x, bx, acc[k], 0, 0, 0);
                if ((flags & kGPaired) == 0)
#pragma unroll
                    for (int k = 0; k < NT; ++k)
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(ODD ? L[k].x : L[k].y, ODD ? by : -by, acc[k], 0, 0, 0);
#pragma unroll
                for (int k = 0; k < NT; ++k) L[k] = make_float2(0.f, 0.f);
            }
            }
        }
    }
}

template <int T, bool ODD, bool SYM>
__device__ __forceinline__ void quad_gen_body(const QuadArgs &a, const float2 *coef, const float *w, double *partial, int lam,
                                              int blk, float2 *tile, uint32_t *rows) {
    constexpr int NT = SYM ? T * (T + 1) / 2 : T * T;
    constexpr int NBP = 4 * T;
    const int nb = a.nbins, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const IntPtr st = (IntPtr)(uintptr_t)(a.stage + (int64_t)kStageStride * lam);
    const IntPtr tp = (IntPtr)(uintptr_t)a.gptr;
    const TermPtr terms = (TermPtr)(uintptr_t)a.gterms;
    const int ncol = st[3], offc = st[2] * NBP;
    const int S = row_pitch(ncol, T), TC = tile_cells(ncol, T);
    const int t0 = tp[lam], t1 = tp[lam + 1];
    float *wt = reinterpret_cast<float *>(tile + TC * S);
    f4v acc[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[k] = f4v{0.f, 0.f, 0.f, 0.f};
    // bins beyond nbins hold zeros throughout
    for (int f = tid; f < TC * ncol * (NBP - nb); f += 256) {
        const int c = f % TC, kb = f / TC;
        tile[c * S + (kb / (NBP - nb)) * NBP + nb + kb % (NBP - nb)] = make_float2(0.f, 0.f);
    }
    const int64_t c0 = (int64_t)blk * a.cells_per_block;
    const int64_t c1 = min(c0 + a.cells_per_block, a.ng);
    // staging: a quarter wave takes 16 consecutive cells of one row (column, bin), kBatch rows in
    // flight.  Row table: array * nbins + bin, LDS offset, part of a packed m = 0 array
    for (int f = tid; f < ncol * nb; f += 256) {
        const int k = f / nb, b = f % nb, lm = a.stage[(int64_t)kStageStride * lam + 4 + k];
        const int arr = a.lm_src ? a.lm_src[2 * lm] : lm, part = a.lm_src ? a.lm_src[2 * lm + 1] : 0;
        rows[f] = (uint32_t)(arr * nb + b) | (uint32_t)(k * NBP + b) << 10 | (uint32_t)part << 20;
    }
    const int c16 = tid & 15, q16 = tid >> 4, nrow = ncol * nb;
    for (int64_t tc = c0; tc < c1; tc += TC) {
        __syncthreads();
        for (int cb = 0; cb < TC; cb += 16) {
            const bool in = tc + cb + c16 < c1;
            const float2 *src = coef + tc + cb + c16;
            float2 *dst = tile + (cb + c16) * S;
            for (int f0 = q16; f0 < nrow; f0 += 16 * kBatch) {
                float2 v[kBatch];
                uint32_t e[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    e[j] = f0 + 16 * j < nrow ? rows[f0 + 16 * j] : 0u;
                    v[j] = in && f0 + 16 * j < nrow ? src[(int64_t)(e[j] & 1023u) * a.ng] : make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (f0 + 16 * j < nrow) {
                        const uint32_t part = e[j] >> 20;
                        if (part == 1) v[j].y = 0.f;                          // packed m = 0 column: one real part
                        else if (part == 2) v[j] = make_float2(v[j].y, 0.f);
                        dst[(e[j] >> 10) & 1023u] = v[j];
                    }
            }
        }
        if (tid < TC) wt[tid] = tc + tid < c1 ? w[tc + tid] : 0.f;
        __syncthreads();
        if (t0 < t1) contract_tile_cells<T, ODD, SYM>(tile, wt, TC, S, offc, terms, t0, t1, wave, i, g, acc);
    }
    // accumulator tile (t1, t2): lane (i, g) holds pair (g + 4 t1, r + 4 t2), bin b3 = i in element r
    __syncthreads();
    float *red = reinterpret_cast<float *>(tile);
    const int nv = nb * nb * nb;
    int k = 0;
#pragma unroll
    for (int ta = 0; ta < T; ++ta)
#pragma unroll
        for (int tb = SYM ? ta : 0; tb < T; ++tb, ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int p1 = g + 4 * ta, p2 = r + 4 * tb;
                if (p1 < nb && p2 < nb && i < nb) red[wave * nv + (p1 * nb + p2) * nb + i] = acc[k][r];
            }
    __syncthreads();
    for (int v = tid; v < nv; v += 256) {
        int vs = v;
        double sg = 1.0;
        if (SYM) {   // tiles t1 > t2: the mirrored pair (sign -1 for odd Lambda)
            const int p1 = v / (nb * nb), p2 = (v / nb) % nb;
            if ((p1 >> 2) > (p2 >> 2)) {
                vs = (p2 * nb + p1) * nb + v % nb;
                sg = ODD ? -1.0 : 1.0;
            }
        }
        const double s = ((double)red[vs] + (double)red[nv + vs]) + ((double)red[2 * nv + vs] + (double)red[3 * nv + vs]);
        partial[((int64_t)lam * nv + v) * a.nblocks + blk] = sg * s;
    }
}

// 1D grid over (cell block, Lambda) items, eight shares of consecutive items: the workgroups of an
// XCD (dealt to them in turn) run the Lambda of a cell block one after the other, while its
// coefficients are in that XCD's cache.
template <int T, bool ODD>
__global__ __launch_bounds__(256, 4) void quad_gen_kernel(QuadArgs a) {
    extern __shared__ float2 tile[];
    __shared__ uint32_t rows[3 * (kMaxL + 1) * 4 * T];
    const int n = a.nblocks * a.nglam, share = (n + 7) / 8;
    const int item = (int)(blockIdx.x % 8) * share + (int)(blockIdx.x / 8);
    if ((int)(blockIdx.x / 8) >= share || item >= n) return;
    const int blk = item / a.nglam;
    const int lam = ((IntPtr)(uintptr_t)a.glam)[item % a.nglam];
    const float2 *coef = a.coef + (int64_t)blockIdx.y * a.coef_fs;   // field of the launch
    const float *w = a.w + (int64_t)blockIdx.y * a.w_fs;
    double *partial = a.partial + (int64_t)blockIdx.y * a.part_fs;
    const IntPtr l = (IntPtr)(uintptr_t)(a.lam_l + 3 * lam);
    if (l[0] == l[1]) quad_gen_body<T, ODD, true>(a, coef, w, partial, lam, blk, tile, rows);
    else quad_gen_body<T, ODD, false>(a, coef, w, partial, lam, blk, tile, rows);
}

template <int T>
hipError_t launch_t(const QuadArgs &a, hipStream_t s) {
    // the largest tile of any column count of the plan, and the reduction's 4 nbins^3 floats
    size_t shm = (size_t)4 * a.nbins * a.nbins * a.nbins * sizeof(float);
    for (int c = 1; c <= a.max_cols; ++c)
        shm = std::max(shm, (size_t)tile_cells(c, T) * (row_pitch(c, T) * sizeof(float2) + sizeof(float)));
    const int64_t n = (int64_t)a.nblocks * a.nglam;
    dim3 grid((unsigned)((n + 7) / 8 * 8), (unsigned)(a.fields > 1 ? a.fields : 1));
    if (a.odd) hipLaunchKernelGGL((quad_gen_kernel<T, true>), grid, dim3(256), shm, s, a);
    else hipLaunchKernelGGL((quad_gen_kernel<T, false>), grid, dim3(256), shm, s, a);
    return hipGetLastError();
}

}  // namespace

int quad_gen_side(int nbins) { return nbins <= 4 ? 1 : nbins <= 8 ? 2 : 3; }

hipError_t launch_quad_gen(const QuadArgs &a, hipStream_t s) {
    if (a.nbins < 1 || a.nbins > 10 || a.nglam < 1 || a.max_cols > 3 * (kMaxL + 1)) return hipErrorInvalidValue;
    switch (quad_gen_side(a.nbins)) {
        case 1: return launch_t<1>(a, s);
        case 2: return launch_t<2>(a, s);
        default: return launch_t<3>(a, s);
    }
}

}  // namespace sb
