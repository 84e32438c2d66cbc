// ff_matvec.hip -- float-float matrix-vector product y = A x, its backward
// pass (dA = g x^T, dx = A^T g) and the backward pass of the float-float dot.
//
// A is M x N, row-major, hi and lo planes with leading dimension lda.  The
// forward pass reads A once (8 bytes per element) and performs Mul22 + Add22
// (~26 VALU) per element; the fused backward reads A once and writes dA once
// (16 bytes per element) with Mul22 (dA) + Mul22 + Add22 (dx) (~38 VALU).
// Both are HBM-bound on gfx950 (ridge ~9.8 binary32 operations per byte).
//
// Fast forward: a group of 16 to 512 threads per row or pair of rows; lane t
// takes the float4 groups t, t + threads, ... of its rows, each load of x
// serving both, keeps four Add22 accumulators per row (one per float4
// component), then a butterfly over the group's lanes and, for several
// wavefronts, an in-order LDS combine give y_i.  x is re-read from L2.
// Fast backward: the workgroup grid is (column tiles) x (row bands); a
// thread owns four adjacent columns, walks the row pairs of its band, writes
// dA_ij = Mul22(g_i, x_j) and accumulates Mul22(g_i, A_ij) per column; the
// per-band partial column sums go to the workspace and a second launch adds
// them in band order.
#include <type_traits>

#include "ff_device.h"
#include "ff_host.h"

namespace ffk {

// Four consecutive words at any 4-byte alignment: gfx950's 16-byte global
// accesses need no more, so rows of any length and any plane take them.
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));

// Backward band kernel: workgroups of 128 threads of four columns each, as many
// across the columns as these need (16 to 128) and the rest over further
// bands.  A band is so many rows that the matrix makes about 2^17 threads
// (two wavefronts per SIMD), at most 128 rows: 128-row bands left 1024 x 1024
// with sixteen workgroups (70 us, 8.6 now).  At most 1024 bands, so that
// combining their partial sums stays short.
constexpr int kColBlock = 128;
constexpr int64_t kBandRows = 128;

inline int64_t band_rows_of(int64_t M, int64_t N)
{
    if (N < 64)
        return kBandRows;
    int64_t rows = ffh::cdiv(M * N, int64_t(1) << 19);
    rows = rows < 4 ? 4 : rows;
    rows = rows < ffh::cdiv(M, 1024) ? ffh::cdiv(M, 1024) : rows;
    rows = (rows + 1) & ~int64_t(1);
    return rows < kBandRows ? rows : kBandRows;
}

// Fast forward: RT consecutive threads per group of R rows.  The rows share
// each load of x, and each lane issues the loads of kRowUnroll float4 groups
// (all rows' planes and x) before any arithmetic.
//
// SHORT, for rows of few rounds: the words after the last whole group are loaded
// first, and the last round's second group, where it lies past the end, is the
// last one loaded again and not added.  Loaded as they come they made a short
// row wait for memory up to three times (64 x 1023: 4.5 us, 3.3 now; 1600 x 1030:
// 7.2, 5.6); with many rounds, or two rows, the other loop has fewer operations
// and registers (1536 x 2049 with two rows 6.8 us, 7.5 with the loads first).
constexpr int kRowUnroll = 2;

template <int BLOCK, int RT, int R, bool SHORT>
__global__ __launch_bounds__(BLOCK) void matvec_rows(int64_t M, int64_t N,
                                                     const float *__restrict__ Ah,
                                                     const float *__restrict__ Al, int64_t lda,
                                                     const float *__restrict__ xh,
                                                     const float *__restrict__ xl,
                                                     float *__restrict__ yh, float *__restrict__ yl)
{
    constexpr int kGroups = BLOCK / RT, kWaves = RT > 64 ? RT / 64 : 1, U = kRowUnroll;
    const int t = threadIdx.x % RT;
    const int64_t r0 = (static_cast<int64_t>(blockIdx.x) * kGroups + threadIdx.x / RT) * R;
    // rows r0 .. r0 + R - 1; a row beyond M repeats the last one (not stored)
    const float *rh[R], *rl[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int64_t r = r0 + q < M ? r0 + q : M - 1;
        rh[q] = Ah + r * lda;
        rl[q] = Al + r * lda;
    }
    float2 acc[R][4];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            acc[q][k] = make_float2(0.0f, 0.0f);
    auto add_term = [&](int q, int k, float ah, float al, float bh, float bl) {
        float ph, pl;
        ffd::mul22<false>(ah, al, bh, bl, ph, pl);
        ffd::add22(acc[q][k].x, acc[q][k].y, ph, pl, acc[q][k].x, acc[q][k].y);
    };
    const int64_t ng = N >> 2;
    const f32x4 *xh4 = reinterpret_cast<const f32x4 *>(xh);
    const f32x4 *xl4 = reinterpret_cast<const f32x4 *>(xl);
    const int64_t j_last = 4 * ng + t;
    if constexpr (SHORT) {
        static_assert(R == 1, "one row");
        float word_bh, word_bl, word_ah, word_al;
        if (j_last < N) {
            word_bh = xh[j_last];
            word_bl = xl[j_last];
            word_ah = rh[0][j_last];
            word_al = rl[0][j_last];
        }
        for (int64_t g = t; g < ng; g += U * RT) {
            f32x4 bh[U], bl[U], ah[U], al[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t at = g + u * RT < ng ? g + u * RT : ng - 1;
                bh[u] = xh4[at];
                bl[u] = xl4[at];
                ah[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(rh[0]) + at);
                al[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(rl[0]) + at);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u == 0 || g + u * RT < ng)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        add_term(0, k, ah[u][k], al[u][k], bh[u][k], bl[u][k]);
        }
        if (j_last < N)
            add_term(0, 0, word_ah, word_al, word_bh, word_bl);
    } else {
        int64_t g = t;
        for (; g + (U - 1) * RT < ng; g += U * RT) {
            f32x4 bh[U], bl[U], ah[R][U], al[R][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                bh[u] = xh4[g + u * RT];
                bl[u] = xl4[g + u * RT];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    ah[q][u] = __builtin_nontemporal_load(
                        reinterpret_cast<const f32x4 *>(rh[q]) + g + u * RT);
                    al[q][u] = __builtin_nontemporal_load(
                        reinterpret_cast<const f32x4 *>(rl[q]) + g + u * RT);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < R; ++q)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        add_term(q, k, ah[q][u][k], al[q][u][k], bh[u][k], bl[u][k]);
        }
        for (; g < ng; g += RT) {
            const f32x4 bh = xh4[g], bl = xl4[g];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const f32x4 ah =
                    __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(rh[q]) + g);
                const f32x4 al =
                    __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(rl[q]) + g);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    add_term(q, k, ah[k], al[k], bh[k], bl[k]);
            }
        }
        if (j_last < N)
#pragma unroll
            for (int q = 0; q < R; ++q)
                add_term(q, 0, rh[q][j_last], rl[q][j_last], xh[j_last], xl[j_last]);
    }
    float h[R], l[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        float h2 = acc[q][2].x, l2 = acc[q][2].y;
        h[q] = acc[q][0].x;
        l[q] = acc[q][0].y;
        ffd::add22(h[q], l[q], acc[q][1].x, acc[q][1].y, h[q], l[q]);
        ffd::add22(h2, l2, acc[q][3].x, acc[q][3].y, h2, l2);
        ffd::add22(h[q], l[q], h2, l2, h[q], l[q]);
#pragma unroll
        for (int m = (RT < 64 ? RT : 64) / 2; m >= 1; m >>= 1) {
            const float oh = __shfl_xor(h[q], m, 64), ol = __shfl_xor(l[q], m, 64);
            ffd::add22(h[q], l[q], oh, ol, h[q], l[q]);
        }
    }
    if constexpr (kWaves > 1) {
        static_assert(RT == BLOCK, "one group of several wavefronts");
        __shared__ float2 part[R][kWaves];
        if ((t & 63) == 0)
#pragma unroll
            for (int q = 0; q < R; ++q)
                part[q][t >> 6] = make_float2(h[q], l[q]);
        __syncthreads();
        if (t == 0)
#pragma unroll
            for (int q = 0; q < R; ++q)
#pragma unroll
                for (int k = 1; k < kWaves; ++k)
                    ffd::add22(h[q], l[q], part[q][k].x, part[q][k].y, h[q], l[q]);
    }
    if (t == 0)
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (r0 + q < M) {
                yh[r0 + q] = h[q];
                yl[r0 + q] = l[q];
            }
}

// Plain forward: one thread per row, terms added in column order.
__global__ __launch_bounds__(256) void matvec_plain(int64_t M, int64_t N,
                                                    const float *__restrict__ Ah,
                                                    const float *__restrict__ Al, int64_t lda,
                                                    const float *__restrict__ xh,
                                                    const float *__restrict__ xl,
                                                    float *__restrict__ yh, float *__restrict__ yl)
{
    const int64_t r = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (r >= M)
        return;
    float h = 0.0f, l = 0.0f;
    for (int64_t j = 0; j < N; ++j) {
        float ph, pl;
        ffd::mul22<false>(Ah[r * lda + j], Al[r * lda + j], xh[j], xl[j], ph, pl);
        ffd::add22(h, l, ph, pl, h, l);
    }
    yh[r] = h;
    yl[r] = l;
}

// Fused backward over row bands: thread owns COLS adjacent columns of one
// band, both rows' loads of a pair issued before any arithmetic; 2^col_shift
// threads of the workgroup span the columns.  Band b of n takes the row pairs
// b, b + n, b + 2 n, ..., so that the workgroups in flight sweep the four
// planes together: with adjacent rows per band every band kept pages of its
// own open (14271 x 4110: 263 us, 234 now; 14336 x 4096: 218, 171; 4096 x 4096:
// 57, 51; 8191 x 8191: 235, 220; 8192 x 8192: 172, 169, 6.3 TB/s; of 30 shapes
// the two that lost, 4096 x 16384 and 2048 x 32768, follow the planes' placement:
// 170-198 us against 172-182, and 184-212 against 190-193, over four).  Loading two
// pairs ahead of the stores, or four rows at once, gave nothing.
template <int BLOCK, int COLS, bool WANT_DA, bool WANT_DX>
__global__ __launch_bounds__(BLOCK) void matvec_bwd_band(
    int64_t M, int64_t N, const float *__restrict__ Ah, const float *__restrict__ Al, int64_t lda,
    const float *__restrict__ xh, const float *__restrict__ xl, const float *__restrict__ gh,
    const float *__restrict__ gl, float *__restrict__ dAh, float *__restrict__ dAl, int64_t ldda,
    float2 *__restrict__ part, int nbands, int col_shift)
{
    const int across = 1 << col_shift;
    int64_t c0 = ((static_cast<int64_t>(blockIdx.x) << col_shift) + (threadIdx.x & (across - 1))) *
                 COLS;
    const int64_t band = (static_cast<int64_t>(blockIdx.y) * BLOCK + threadIdx.x) >> col_shift;
    if (c0 >= N || band >= nbands)
        return;
    // the last thread's columns end with the row: those it shares with the
    // thread before are computed twice, to the same bits
    if (c0 + COLS > N)
        c0 = N - COLS;
    float x_h[COLS], x_l[COLS];
    float2 acc[COLS];
#pragma unroll
    for (int k = 0; k < COLS; ++k) {
        acc[k] = make_float2(0.0f, 0.0f);
        if (WANT_DA) {
            x_h[k] = xh[c0 + k];
            x_l[k] = xl[c0 + k];
        }
    }
    auto row = [&](int64_t i, const float (&a_h)[COLS], const float (&a_l)[COLS]) {
        const float g_h = gh[i], g_l = gl[i];
        if (WANT_DA) {
            float d_h[COLS], d_l[COLS];
#pragma unroll
            for (int k = 0; k < COLS; ++k)
                ffd::mul22<false>(g_h, g_l, x_h[k], x_l[k], d_h[k], d_l[k]);
            if constexpr (COLS == 4) {
                const f32x4 vh = {d_h[0], d_h[1], d_h[2], d_h[3]};
                const f32x4 vl = {d_l[0], d_l[1], d_l[2], d_l[3]};
                __builtin_nontemporal_store(vh, reinterpret_cast<f32x4 *>(dAh + i * ldda + c0));
                __builtin_nontemporal_store(vl, reinterpret_cast<f32x4 *>(dAl + i * ldda + c0));
            } else {
                dAh[i * ldda + c0] = d_h[0];
                dAl[i * ldda + c0] = d_l[0];
            }
        }
        if (WANT_DX) {
#pragma unroll
            for (int k = 0; k < COLS; ++k) {
                float ph, pl;
                ffd::mul22<false>(g_h, g_l, a_h[k], a_l[k], ph, pl);
                ffd::add22(acc[k].x, acc[k].y, ph, pl, acc[k].x, acc[k].y);
            }
        }
    };
    auto load_row = [&](int64_t i, float (&a_h)[COLS], float (&a_l)[COLS]) {
        if (WANT_DX) {
            if constexpr (COLS == 4) {
                const f32x4 vh = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Ah + i * lda + c0));
                const f32x4 vl = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Al + i * lda + c0));
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    a_h[k] = vh[k];
                    a_l[k] = vl[k];
                }
            } else {
                a_h[0] = Ah[i * lda + c0];
                a_l[0] = Al[i * lda + c0];
            }
        }
    };
    const int64_t step = 2 * static_cast<int64_t>(nbands);
    int64_t i = 2 * band;
    for (; i + 2 <= M; i += step) {
        float a_h[2][COLS], a_l[2][COLS];
#pragma unroll
        for (int p = 0; p < 2; ++p)
            load_row(i + p, a_h[p], a_l[p]);
#pragma unroll
        for (int p = 0; p < 2; ++p)
            row(i + p, a_h[p], a_l[p]);
    }
    if (i < M) {   // the last row of an odd number
        float a_h[COLS], a_l[COLS];
        load_row(i, a_h, a_l);
        row(i, a_h, a_l);
    }
    if (WANT_DX) {
#pragma unroll
        for (int k = 0; k < COLS; ++k)
            part[band * N + c0 + k] = acc[k];
    }
}

// dx_j = sum over bands of the per-band partials, for COLS columns per
// workgroup: GROUPS groups of threads take bands g, g + GROUPS, ... (rows of
// partials of COLS columns, several loads in flight per thread), then the
// group sums are added in a fixed tree through LDS.  64 columns by 8 groups
// for wide matrices; 16 by 64 where there are few columns and more bands.
template <int COLS, int GROUPS>
__global__ __launch_bounds__(COLS * GROUPS) void matvec_bwd_combine(
    int64_t N, int64_t nbands, const float2 *__restrict__ part, float *__restrict__ dxh,
    float *__restrict__ dxl, int64_t first)
{
    __shared__ float2 sums[GROUPS][COLS];
    const int col = threadIdx.x % COLS, grp = threadIdx.x / COLS;
    const int64_t j = (first + blockIdx.x) * COLS + col;
    float h = 0.0f, l = 0.0f;
    if (j < N) {
        int64_t b = grp;
        for (; b + 3 * GROUPS < nbands; b += 4 * GROUPS) {
            float2 p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                p[u] = part[(b + u * GROUPS) * N + j];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                ffd::add22(h, l, p[u].x, p[u].y, h, l);
        }
        for (; b < nbands; b += GROUPS) {
            const float2 p = part[b * N + j];
            ffd::add22(h, l, p.x, p.y, h, l);
        }
    }
    sums[grp][col] = make_float2(h, l);
    __syncthreads();
#pragma unroll
    for (int w = GROUPS / 2; w >= 1; w >>= 1) {
        if (grp < w) {
            const float2 a = sums[grp][col], c = sums[grp + w][col];
            float rh, rl;
            ffd::add22(a.x, a.y, c.x, c.y, rh, rl);
            sums[grp][col] = make_float2(rh, rl);
        }
        __syncthreads();
    }
    if (grp == 0 && j < N) {
        dxh[j] = sums[0][col].x;
        dxl[j] = sums[0][col].y;
    }
}

// Plain backward, dx: one thread per column, rows in order.
__global__ __launch_bounds__(256) void matvec_bwd_plain_dx(
    int64_t M, int64_t N, const float *__restrict__ Ah, const float *__restrict__ Al, int64_t lda,
    const float *__restrict__ gh, const float *__restrict__ gl, float *__restrict__ dxh,
    float *__restrict__ dxl)
{
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (j >= N)
        return;
    float h = 0.0f, l = 0.0f;
    for (int64_t i = 0; i < M; ++i) {
        float ph, pl;
        ffd::mul22<false>(gh[i], gl[i], Ah[i * lda + j], Al[i * lda + j], ph, pl);
        ffd::add22(h, l, ph, pl, h, l);
    }
    dxh[j] = h;
    dxl[j] = l;
}

// Plain backward, dA: one thread per element.
__global__ __launch_bounds__(256) void matvec_bwd_plain_da(
    int64_t M, int64_t N, const float *__restrict__ xh, const float *__restrict__ xl,
    const float *__restrict__ gh, const float *__restrict__ gl, float *__restrict__ dAh,
    float *__restrict__ dAl, int64_t ldda)
{
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j >= N || i >= M)
        return;
    float h, l;
    ffd::mul22<false>(gh[i], gl[i], xh[j], xl[j], h, l);
    dAh[i * ldda + j] = h;
    dAl[i * ldda + j] = l;
}

// Backward pass of the single float-float dot s = sum x_i y_i for one
// upstream gradient g: dx_i = Mul22(g, y_i), dy_i = Mul22(g, x_i).  One
// workgroup of kDotBwdThreads per block of kDotBwdThreads * kDotBwdPer
// consecutive elements, in launch order; a thread loads all its
// lane-contiguous elements first, then computes and stores.  Small
// workgroups stream this pattern (four planes in, four out) fastest: 128
// threads by one element moved 6.2 TB/s at N = 2^28, against 6.0 for 128 by
// 2 and 5.35 for 1024 by 2; no block pays a per-block set-up here.
constexpr int kDotBwdThreads = 128;
constexpr int kDotBwdPer = 1;

__global__ __launch_bounds__(kDotBwdThreads) void dot_backward(const float *__restrict__ g_hi,
                                                    const float *__restrict__ g_lo,
                                                    const float *__restrict__ xh,
                                                    const float *__restrict__ xl,
                                                    const float *__restrict__ yh,
                                                    const float *__restrict__ yl,
                                                    float *__restrict__ dxh,
                                                    float *__restrict__ dxl,
                                                    float *__restrict__ dyh,
                                                    float *__restrict__ dyl, int64_t n)
{
    constexpr int kPer = kDotBwdPer;
    const float gh = g_hi[0], gl = g_lo[0];
    const int64_t b0 = static_cast<int64_t>(blockIdx.x) * (kDotBwdThreads * kPer) + threadIdx.x;
    const bool want_dx = dxh != nullptr, want_dy = dyh != nullptr;
    float ox[kPer], oxl[kPer], oy[kPer], oyl[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = b0 + static_cast<int64_t>(kDotBwdThreads) * k;
        const bool in = i < n;
        ox[k] = (want_dy && in) ? xh[i] : 0.0f;
        oxl[k] = (want_dy && in) ? xl[i] : 0.0f;
        oy[k] = (want_dx && in) ? yh[i] : 0.0f;
        oyl[k] = (want_dx && in) ? yl[i] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = b0 + static_cast<int64_t>(kDotBwdThreads) * k;
        if (i >= n)
            break;
        float h, l;
        if (want_dx) {
            ffd::mul22<false>(gh, gl, oy[k], oyl[k], h, l);
            dxh[i] = h;
            dxl[i] = l;
        }
        if (want_dy) {
            ffd::mul22<false>(gh, gl, ox[k], oxl[k], h, l);
            dyh[i] = h;
            dyl[i] = l;
        }
    }
}

// Backward pass of the batched dot s_v = sum over vector v of x_i y_i:
// every element i of vector v gets dx_i = Mul22(g_v, y_i) and
// dy_i = Mul22(g_v, x_i); elements of no vector get zeros.  Two launches:
//   records   one thread per block of kBwdBlock consecutive elements: a
//             binary search over the clamped offsets for the vector owning
//             the block's first element, stored with that vector's gradient
//             and the next vector's start as one 16-byte record
//   gradients one workgroup per block, launched in order, so that the
//             resident workgroups sweep memory together: thread t takes
//             elements b0 + t + kBwdThreads k (each wavefront access is 256
//             contiguous bytes of a plane) and issues all its loads first,
//             then the block's record (one scalar load, on a counter of its
//             own); the vector starts inside a wavefront's range (usually
//             none) are walked, up to kBwdWalk of them, and past that (vectors
//             of a few elements) each lane searches its remaining elements'
//             owners
// Small blocks stream this pattern (two planes in, four out) fastest: a
// pass-through kernel moved 6.5 TB/s at 256 threads by one element, 6.25 at
// 128 by 1, 5.6 at 512 by 2 and 5.5 at 512 by 8 (438.9 M elements on
// MI355X).  A search per block at that size -- even one shared by the
// workgroup's wavefronts -- cost more than the access pattern gained (its
// dependent loads wait behind the streaming traffic), hence the records.
// 24 to 32 bytes per element and two Mul22: HBM-bound.
constexpr int kBwdThreads = 256;
constexpr int kBwdPer = 1;
constexpr int64_t kBwdBlock = static_cast<int64_t>(kBwdThreads) * kBwdPer;
constexpr int kBwdWalk = 8;
constexpr int kBwdRecordThreads = 256;

__device__ __forceinline__ int64_t clamped_offset(const int64_t *__restrict__ offsets, int64_t v,
                                                  int64_t total)
{
    const int64_t o = offsets[v];
    return o < 0 ? 0 : (o > total ? total : o);
}

// Number of vector starts at or before position p, minus one: the vector
// owning element p, in [-1, nvec] (-1: before the first vector, nvec: after
// the last).  With offsets out of order the result is still in that range.
__device__ __forceinline__ int64_t owner_of(const int64_t *__restrict__ offsets, int32_t nvec,
                                            int64_t total, int64_t p)
{
    int64_t lo = 0, hi = static_cast<int64_t>(nvec) + 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (clamped_offset(offsets, mid, total) <= p)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo - 1;
}

// Record of block b: x = the vector owning element b * kBwdBlock (-1 .. nvec),
// y, z = the bits of its gradient (zero when it is no vector), w = the start
// of the next vector relative to the block's first element, clipped to
// [0, INT32_MAX] (INT32_MAX: none within reach).
__global__ __launch_bounds__(kBwdRecordThreads) void dot_bwd_records(
    const float *__restrict__ g_hi, const float *__restrict__ g_lo,
    const int64_t *__restrict__ offsets, int32_t nvec, int64_t total, int64_t nblocks,
    int4 *__restrict__ records)
{
    const int64_t b = static_cast<int64_t>(blockIdx.x) * kBwdRecordThreads + threadIdx.x;
    if (b >= nblocks)
        return;
    const int64_t b0 = b * kBwdBlock;
    const int64_t v = owner_of(offsets, nvec, total, b0);
    const bool ok = v >= 0 && v < nvec;
    const float gh = ok ? g_hi[v] : 0.0f, gl = ok ? g_lo[v] : 0.0f;
    int64_t rel = INT32_MAX;
    if (v < nvec) {
        const int64_t o = clamped_offset(offsets, v + 1, total) - b0;
        rel = o < 0 ? 0 : (o < INT32_MAX ? o : INT32_MAX);
    }
    records[b] = make_int4(static_cast<int32_t>(v), __float_as_int(gh), __float_as_int(gl),
                           static_cast<int32_t>(rel));
}

template <bool XLO, bool YLO, bool DX, bool DY>
__global__ __launch_bounds__(kBwdThreads) void dot_batched_bwd(
    const float *__restrict__ g_hi, const float *__restrict__ g_lo,
    const int64_t *__restrict__ offsets, int32_t nvec, int64_t total,
    const int4 *__restrict__ records, int64_t first,
    const float *__restrict__ xh, const float *__restrict__ xl, const float *__restrict__ yh,
    const float *__restrict__ yl, float *__restrict__ dxh, float *__restrict__ dxl,
    float *__restrict__ dyh, float *__restrict__ dyl)
{
    const int t = threadIdx.x;
    const int64_t block = first + blockIdx.x, b0 = block * kBwdBlock;
    // all of this thread's operands first
    int64_t idx[kBwdPer];
    float ox[kBwdPer], oxl[kBwdPer], oy[kBwdPer], oyl[kBwdPer];
#pragma unroll
    for (int k = 0; k < kBwdPer; ++k) {
        const int64_t i = b0 + t + static_cast<int64_t>(kBwdThreads) * k;
        idx[k] = i;
        const bool in = i < total;
        ox[k] = (DY && in) ? xh[i] : 0.0f;
        oxl[k] = (DY && XLO && in) ? xl[i] : 0.0f;
        oy[k] = (DX && in) ? yh[i] : 0.0f;
        oyl[k] = (DX && YLO && in) ? yl[i] : 0.0f;
    }
    const int4 r = records[block];
    // the wavefront's first and last element, the same on every lane
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t w0 = b0 + 64 * wave;
    if (w0 >= total)
        return;
    const int64_t w_end = w0 + 63 + static_cast<int64_t>(kBwdThreads) * (kBwdPer - 1);
    const int64_t w_last = w_end < total ? w_end : total - 1;
    int64_t v = r.x;
    int64_t nxt = r.w == INT32_MAX ? INT64_MAX : b0 + r.w;
    bool has[kBwdPer];
    float gkh[kBwdPer], gkl[kBwdPer];
    {
        const bool ok = v >= 0 && v < nvec;
        const float gh = __int_as_float(r.y), gl = __int_as_float(r.z);
#pragma unroll
        for (int k = 0; k < kBwdPer; ++k) {
            has[k] = ok;
            gkh[k] = gh;
            gkl[k] = gl;
        }
    }
    // elements at or after the start nxt of vector v + 1 belong to it (or to
    // a later vector, found when its own start is reached)
    for (int step = 0; step < kBwdWalk && nxt <= w_last; ++step) {
        ++v;
        const bool ok = v < nvec;
        const float gh = ok ? g_hi[v] : 0.0f, gl = ok ? g_lo[v] : 0.0f;
#pragma unroll
        for (int k = 0; k < kBwdPer; ++k) {
            if (idx[k] >= nxt) {
                has[k] = ok;
                gkh[k] = gh;
                gkl[k] = gl;
            }
        }
        nxt = ok ? clamped_offset(offsets, v + 1, total) : INT64_MAX;
    }
    if (nxt <= w_last) {
        // more vector starts in this range than the walk takes
#pragma unroll
        for (int k = 0; k < kBwdPer; ++k) {
            if (idx[k] >= nxt && idx[k] < total) {
                const int64_t u = owner_of(offsets, nvec, total, idx[k]);
                has[k] = u >= 0 && u < nvec;
                gkh[k] = has[k] ? g_hi[u] : 0.0f;
                gkl[k] = has[k] ? g_lo[u] : 0.0f;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kBwdPer; ++k) {
        const int64_t i = idx[k];
        if (i >= total)
            break;
        float a = 0.0f, b = 0.0f, c = 0.0f, d = 0.0f;
        if (has[k]) {
            if (DX)
                ffd::mul22<false>(gkh[k], gkl[k], oy[k], oyl[k], a, b);
            if (DY)
                ffd::mul22<false>(gkh[k], gkl[k], ox[k], oxl[k], c, d);
        }
        if (DX) {
            dxh[i] = a;
            dxl[i] = b;
        }
        if (DY) {
            dyh[i] = c;
            dyl[i] = d;
        }
    }
}

// A plane-by-plane gradient as a float-float value: one launch for what takes
// six of elementwise tensor operations (33 us of a small training step).
constexpr int kGradientThreads = 256;

__global__ __launch_bounds__(kGradientThreads) void gradient_value(
    const float *__restrict__ gh, const float *__restrict__ gl, float *__restrict__ vh,
    float *__restrict__ vl, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kGradientThreads + threadIdx.x;
    if (i >= n)
        return;
    const float h = gh[i], l = gl[i];
    vh[i] = h;
    vl[i] = h == l ? 0.0f : l;
}

bool all_aligned(std::initializer_list<const void *> ptrs, uintptr_t bytes)
{
    for (const void *p : ptrs)
        if (p && !ffh::aligned(p, bytes))
            return false;
    return true;
}

// Partial sums of dx: one row of N per band.
size_t band_bytes(int64_t M, int64_t N, int64_t band_rows)
{
    return static_cast<size_t>(ffh::cdiv(M, band_rows)) * static_cast<size_t>(N) * sizeof(float2);
}

// Enough for the bands of this matrix and of every smaller one, so that a
// workspace for a caller's largest matrix serves the others (the bands of 8192 x
// 8000 take 4.22 MB, those of 8192 x 8192 4.19): shorter than 128 rows, there are
// fewer than 1 more than 2^19 / N, M / 4 and 1024 of them.
size_t queried_bytes(int64_t M, int64_t N)
{
    int64_t sums = int64_t(1) << 19;
    sums = sums < ffh::cdiv(M * N, 4) ? sums : ffh::cdiv(M * N, 4);
    sums = sums < 1024 * N ? sums : 1024 * N;
    const size_t bytes = N < 64 ? 0 : static_cast<size_t>(sums + N) * sizeof(float2);
    const size_t longest = band_bytes(M, N, kBandRows);
    return bytes > longest ? bytes : longest;
}

} // namespace ffk

using namespace ffk;

extern "C" {

ff_status ff_matvec(int64_t M, int64_t N, const float *A_hi, const float *A_lo, int64_t lda,
                    const float *x_hi, const float *x_lo, float *y_hi, float *y_lo, int32_t algo,
                    void *stream)
{
    if (M < 0 || N < 0 || lda < N)
        return FF_ERR_SIZE;
    if (algo != FF_MATVEC_FAST && algo != FF_MATVEC_PLAIN)
        return FF_ERR_ARG;
    if (M == 0)
        return FF_OK;
    if (!y_hi || !y_lo || (N > 0 && (!A_hi || !A_lo || !x_hi || !x_lo)))
        return FF_ERR_NULL;
    if (!all_aligned({A_hi, A_lo, x_hi, x_lo, y_hi, y_lo}, 4))
        return FF_ERR_ALIGN;
    if (M > INT32_MAX)
        return FF_ERR_SIZE;
    hipStream_t st = ffh::as_stream(stream);
    if (algo == FF_MATVEC_PLAIN) {
        ffh::in_parts(M, ffh::kMostThreads, [&](int64_t at, int64_t count) {
            hipLaunchKernelGGL(matvec_plain, dim3(static_cast<unsigned>(ffh::cdiv(count, 256))),
                               dim3(256), 0, st, count, N, A_hi + at * lda, A_lo + at * lda, lda,
                               x_hi, x_lo, y_hi + at, y_lo + at);
        });
    } else {
        auto launch = [&](auto kernel, int block, int rows) {
            ffh::in_parts(M, ffh::kMostThreads / block * rows, [&](int64_t at, int64_t count) {
                hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(ffh::cdiv(count, rows))),
                                   dim3(block), 0, st, count, N, A_hi + at * lda, A_lo + at * lda,
                                   lda, x_hi, x_lo, y_hi + at, y_lo + at);
            });
        };
        // As many threads per row as it feeds with a few float4 groups each, one
        // row per group of threads, two where there are rows enough for 512
        // workgroups.  From 2048 rows on, us against 256 threads by two rows: 16384
        // x 64 3.4 / 18.0, 16384 x 512 11.9 / 21.8 (16 threads); 16384 x 1000 24.1 /
        // 27.8 (64); and for two rows against one 1000 x 16384 23.9 / 27.3, 8192 x
        // 8192 81 / 90.  Below, us with the matrix cached (from HBM) against the next
        // best: 64 x 63 2.7, the other loop 2.8, and 64 x 64 2.5, this one 2.7; 64 x 127 2.8
        // (2.5), 64 threads 3.0 (2.8); 500 x 257 3.2 (3.3), 128
        // threads 3.3 (3.4); 500 x 511 3.4 (3.6), 256 threads 3.5 (3.7); 1600 x 3001
        // 9.2 (9.5), 256 threads 10.7 (10.3); 768 x 1023 4.2 (4.3), 128 threads 4.4
        // (4.5); 1000 x 8191 13.6 (14.3), 128 threads 15.6 (16.7); 64 x 16384 7.4
        // with 512 threads, 13.5 with 256.
        if (M < 2048 && N <= 64)
            launch(N % 4 ? matvec_rows<256, 16, 1, true> : matvec_rows<256, 16, 1, false>, 256, 16);
        else if (M < 2048 && N <= 128)
            launch(matvec_rows<256, 32, 1, true>, 256, 8);
        else if (M < 2048 && N <= 288)
            launch(matvec_rows<256, 64, 1, true>, 256, 4);
        else if (M < 1280 ? N <= 512 : M < 2048 && N > 512 && N <= 8192)
            launch(matvec_rows<128, 128, 1, true>, 128, 1);
        else if (M < 1280 && (N <= 1024 || (M >= 768 && N <= 8192)))
            launch(matvec_rows<256, 256, 1, true>, 256, 1);
        else if (M < 768)
            launch(matvec_rows<512, 512, 1, false>, 512, 1);
        else if (M >= 2048 && (N <= 128 || (N <= 512 && M >= 4096)))
            launch(matvec_rows<256, 16, 1, false>, 256, 16);
        else if (N <= 512 || (M >= 2048 && N <= 2048))
            launch(matvec_rows<256, 64, 1, false>, 256, 4);
        else
            launch(matvec_rows<256, 256, 2, false>, 256, 2);
    }
    return ffh::launch_status();
}

size_t ff_matvec_backward_workspace_size(int64_t M, int64_t N, int32_t algo)
{
    if (M < 0 || N < 0 || algo != FF_MATVEC_FAST)
        return 0;
    return queried_bytes(M, N);
}

ff_status ff_matvec_backward(int64_t M, int64_t N, const float *A_hi, const float *A_lo,
                             int64_t lda, const float *x_hi, const float *x_lo, const float *g_hi,
                             const float *g_lo, float *dA_hi, float *dA_lo, int64_t ldda,
                             float *dx_hi, float *dx_lo, int32_t algo, void *ws, size_t ws_bytes,
                             void *stream)
{
    if (M < 0 || N < 0 || lda < N)
        return FF_ERR_SIZE;
    if (algo != FF_MATVEC_FAST && algo != FF_MATVEC_PLAIN)
        return FF_ERR_ARG;
    const bool want_da = dA_hi || dA_lo;
    const bool want_dx = dx_hi || dx_lo;
    if ((want_da && (!dA_hi || !dA_lo)) || (want_dx && (!dx_hi || !dx_lo)))
        return FF_ERR_NULL;
    if (want_da && ldda < N)
        return FF_ERR_SIZE;
    if (N == 0 || (!want_da && !want_dx))
        return FF_OK;
    if ((M > 0 && (!g_hi || !g_lo)) || (want_da && (!x_hi || !x_lo)) ||
        (want_dx && M > 0 && (!A_hi || !A_lo)))
        return FF_ERR_NULL;
    if (!all_aligned({A_hi, A_lo, x_hi, x_lo, g_hi, g_lo, dA_hi, dA_lo, dx_hi, dx_lo}, 4))
        return FF_ERR_ALIGN;
    if (M > 65535 * kBandRows || M > INT32_MAX)
        return FF_ERR_SIZE;
    hipStream_t st = ffh::as_stream(stream);
    if (algo == FF_MATVEC_PLAIN) {
        if (want_da && M > 65535)
            return FF_ERR_SIZE;
        if (want_da && M > 0)
            hipLaunchKernelGGL(matvec_bwd_plain_da,
                               dim3(static_cast<unsigned>(ffh::cdiv(N, 256)), static_cast<unsigned>(M)),
                               dim3(256), 0, st, M, N, x_hi, x_lo, g_hi, g_lo, dA_hi, dA_lo, ldda);
        if (want_dx)
            hipLaunchKernelGGL(matvec_bwd_plain_dx, dim3(static_cast<unsigned>(ffh::cdiv(N, 256))),
                               dim3(256), 0, st, M, N, A_hi, A_lo, lda, g_hi, g_lo, dx_hi, dx_lo);
        return ffh::launch_status();
    }
    int64_t band_rows = band_rows_of(M, N);
    if (want_dx && M > 0) {
        if (!ws)
            return FF_ERR_NULL;
        // a workspace that only holds longer bands' sums gets longer bands
        while (band_rows < kBandRows && ws_bytes < band_bytes(M, N, band_rows))
            band_rows = 2 * band_rows < kBandRows ? 2 * band_rows : kBandRows;
        if (ws_bytes < band_bytes(M, N, band_rows))
            return FF_ERR_WORKSPACE;
        if (!ffh::aligned(ws, 16))
            return FF_ERR_ALIGN;
    }
    const int64_t nbands = ffh::cdiv(M, band_rows);
    float2 *part = static_cast<float2 *>(ws);
    if (M > 0) {
        // One column per thread for dA alone off 16-byte alignment, 36 to 352 MiB
        // of it (mostly held by the Infinity Cache), whole 256-byte stores there:
        // us with one and four columns, 2500 x 2501 11.7 / 12.7, 4095 x 4095 27.5 /
        // 36.4, 1000 x 32765 50 / 73, 6000 x 6001 55 / 84, 6700 x 6701 101 / 106; but
        // 2000 x 2001 9.2 / 8.7, 7001 x 7001 126 / 116, 8191 x 8191 198 / 150.
        const bool split = !want_dx && M * N > (int64_t(9) << 19) && M * N < (int64_t(11) << 22) &&
                           !(all_aligned({dA_hi, dA_lo}, 16) && ldda % 4 == 0);
        const int cols = N >= 4 && !split ? 4 : 1;
        int col_shift = 4;
        while ((1 << col_shift) < kColBlock && (int64_t(cols) << col_shift) < N)
            ++col_shift;
        const int64_t across = int64_t(cols) << col_shift, stacked = kColBlock >> col_shift;
        const dim3 grid(static_cast<unsigned>(ffh::cdiv(N, across)),
                        static_cast<unsigned>(ffh::cdiv(nbands, stacked)));
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(kColBlock), 0, st, M, N, A_hi, A_lo, lda, x_hi,
                               x_lo, g_hi, g_lo, dA_hi, dA_lo, ldda, part,
                               static_cast<int>(nbands), col_shift);
        };
        if (cols == 4) {
            if (want_da && want_dx)
                launch(matvec_bwd_band<kColBlock, 4, true, true>);
            else if (want_da)
                launch(matvec_bwd_band<kColBlock, 4, true, false>);
            else
                launch(matvec_bwd_band<kColBlock, 4, false, true>);
        } else {
            if (want_da && want_dx)
                launch(matvec_bwd_band<kColBlock, 1, true, true>);
            else if (want_da)
                launch(matvec_bwd_band<kColBlock, 1, true, false>);
            else
                launch(matvec_bwd_band<kColBlock, 1, false, true>);
        }
    }
    if (want_dx && N >= 4096)
        ffh::in_parts(ffh::cdiv(N, 64), ffh::kMostThreads / 512, [&](int64_t first, int64_t count) {
            hipLaunchKernelGGL((matvec_bwd_combine<64, 8>), dim3(static_cast<unsigned>(count)),
                               dim3(64 * 8), 0, st, N, nbands, part, dx_hi, dx_lo, first);
        });
    else if (want_dx)
        hipLaunchKernelGGL((matvec_bwd_combine<16, 64>),
                           dim3(static_cast<unsigned>(ffh::cdiv(N, 16))), dim3(16 * 64), 0, st, N,
                           nbands, part, dx_hi, dx_lo, int64_t(0));
    return ffh::launch_status();
}

ff_status ff_dot_backward(const float *g_hi, const float *g_lo, const float *x_hi,
                          const float *x_lo, const float *y_hi, const float *y_lo, float *dx_hi,
                          float *dx_lo, float *dy_hi, float *dy_lo, int64_t n, void *stream)
{
    if (n < 0)
        return FF_ERR_SIZE;
    const bool want_dx = dx_hi || dx_lo, want_dy = dy_hi || dy_lo;
    if ((want_dx && (!dx_hi || !dx_lo)) || (want_dy && (!dy_hi || !dy_lo)))
        return FF_ERR_NULL;
    if (n == 0 || (!want_dx && !want_dy))
        return FF_OK;
    if (!g_hi || !g_lo || (want_dx && (!y_hi || !y_lo)) || (want_dy && (!x_hi || !x_lo)))
        return FF_ERR_NULL;
    if (!all_aligned({g_hi, g_lo, x_hi, x_lo, y_hi, y_lo, dx_hi, dx_lo, dy_hi, dy_lo}, 4))
        return FF_ERR_ALIGN;
    if (ffh::cdiv(n, int64_t(kDotBwdThreads) * kDotBwdPer) > INT32_MAX)
        return FF_ERR_SIZE;
    // (planes that may be null are only moved along where they are read or written)
    ffh::in_parts(n, ffh::kMostThreads, [&](int64_t at, int64_t count) {
        const int64_t blocks = ffh::cdiv(count, int64_t(kDotBwdThreads) * kDotBwdPer);
        auto from = [&](auto *plane, bool used) { return used ? plane + at : nullptr; };
        hipLaunchKernelGGL(dot_backward, dim3(static_cast<unsigned>(blocks)), dim3(kDotBwdThreads),
                           0, ffh::as_stream(stream), g_hi, g_lo, from(x_hi, want_dy),
                           from(x_lo, want_dy), from(y_hi, want_dx), from(y_lo, want_dx),
                           from(dx_hi, want_dx), from(dx_lo, want_dx), from(dy_hi, want_dy),
                           from(dy_lo, want_dy), count);
    });
    return ffh::launch_status();
}

ff_status ff_gradient_value(const float *g_hi, const float *g_lo, float *v_hi, float *v_lo,
                            int64_t n, void *stream)
{
    if (n < 0)
        return FF_ERR_SIZE;
    if (n == 0)
        return FF_OK;
    if (!g_hi || !g_lo || !v_hi || !v_lo)
        return FF_ERR_NULL;
    if (!all_aligned({g_hi, g_lo, v_hi, v_lo}, 4))
        return FF_ERR_ALIGN;
    if (ffh::cdiv(n, int64_t(kGradientThreads)) > INT32_MAX)
        return FF_ERR_SIZE;
    ffh::in_parts(n, ffh::kMostThreads, [&](int64_t at, int64_t count) {
        const int64_t blocks = ffh::cdiv(count, int64_t(kGradientThreads));
        hipLaunchKernelGGL(gradient_value, dim3(static_cast<unsigned>(blocks)),
                           dim3(kGradientThreads), 0, ffh::as_stream(stream), g_hi + at, g_lo + at,
                           v_hi + at, v_lo + at, count);
    });
    return ffh::launch_status();
}

size_t ff_dot_batched_backward_workspace_size(int64_t total_len)
{
    if (total_len <= 0)
        return 0;
    return static_cast<size_t>(ffh::cdiv(total_len, kBwdBlock)) * sizeof(int4);
}

ff_status ff_dot_batched_backward(const float *g_hi, const float *g_lo, const int64_t *offsets,
                                  int32_t nvec, int64_t total_len, const float *x_hi,
                                  const float *x_lo, const float *y_hi, const float *y_lo,
                                  float *dx_hi, float *dx_lo, float *dy_hi, float *dy_lo,
                                  void *ws, size_t ws_bytes, void *stream)
{
    if (nvec < 0 || total_len < 0)
        return FF_ERR_SIZE;
    const bool want_dx = dx_hi || dx_lo, want_dy = dy_hi || dy_lo;
    if ((want_dx && (!dx_hi || !dx_lo)) || (want_dy && (!dy_hi || !dy_lo)))
        return FF_ERR_NULL;
    if (total_len == 0 || (!want_dx && !want_dy))
        return FF_OK;
    if (!offsets || (nvec > 0 && (!g_hi || !g_lo)) || (want_dx && !y_hi) || (want_dy && !x_hi))
        return FF_ERR_NULL;
    if (!ffh::aligned(offsets, 8) ||
        !all_aligned({g_hi, g_lo, x_hi, x_lo, y_hi, y_lo, dx_hi, dx_lo, dy_hi, dy_lo}, 4))
        return FF_ERR_ALIGN;
    const int64_t blocks = ffh::cdiv(total_len, kBwdBlock);
    if (blocks > INT32_MAX)
        return FF_ERR_SIZE;
    if (!ws || ws_bytes < ff_dot_batched_backward_workspace_size(total_len))
        return FF_ERR_WORKSPACE;
    if (!ffh::aligned(ws, 16))
        return FF_ERR_ALIGN;
    int4 *records = static_cast<int4 *>(ws);
    hipLaunchKernelGGL(dot_bwd_records,
                       dim3(static_cast<unsigned>(ffh::cdiv(blocks, int64_t(kBwdRecordThreads)))),
                       dim3(kBwdRecordThreads), 0, ffh::as_stream(stream), g_hi, g_lo, offsets,
                       nvec, total_len, blocks, records);
    const bool xlo = want_dy && x_lo, ylo = want_dx && y_lo;
    auto launch = [&](auto kernel) {
        ffh::in_parts(blocks, ffh::kMostThreads / kBwdThreads, [&](int64_t first, int64_t count) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(count)), dim3(kBwdThreads), 0,
                               ffh::as_stream(stream), g_hi, g_lo, offsets, nvec, total_len,
                               static_cast<const int4 *>(records), first, x_hi, x_lo, y_hi, y_lo,
                               dx_hi, dx_lo, dy_hi, dy_lo);
        });
    };
    // one instantiation per (low words present, outputs wanted)
    if (want_dx && want_dy) {
        if (xlo && ylo)
            launch(dot_batched_bwd<true, true, true, true>);
        else if (xlo)
            launch(dot_batched_bwd<true, false, true, true>);
        else if (ylo)
            launch(dot_batched_bwd<false, true, true, true>);
        else
            launch(dot_batched_bwd<false, false, true, true>);
    } else if (want_dx) {
        if (ylo)
            launch(dot_batched_bwd<false, true, true, false>);
        else
            launch(dot_batched_bwd<false, false, true, false>);
    } else {
        if (xlo)
            launch(dot_batched_bwd<true, false, false, true>);
        else
            launch(dot_batched_bwd<false, false, false, true>);
    }
    return ffh::launch_status();
}

} // extern "C"
