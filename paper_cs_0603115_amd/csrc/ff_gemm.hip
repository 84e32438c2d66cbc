// ff_gemm.hip -- float-float matrix product C = A B (row-major planes).
//
// Two algorithms.
//
// FMA loop (the plain float-float GEMM): C_ij = Add22 accumulation, k
// ascending, of Mul22(A_ik, B_kj) -- section 4.1's operators applied term by
// term.  LDS-tiled (1, 4 or 16 outputs per thread), VALU bound: ~26 binary32
// operations per multiply-add, no contraction.  Bit for bit the sequential
// definition.
//
// Sliced (the fast path; the paper has no GEMM): every entry of A and B is
// turned into a signed fixed-point integer relative to a power of two of its
// row (A) or column (B):
//     X_ik = round(A_ik 2^(54 - e_i)),  2^e_i > max_k |A_ik|,
// and the integer product X Y is formed exactly in a residue number system:
// modulo sixteen pairwise coprime integers m up to 256 (ff_gemm_residue.h),
// whose product P = 2^125.37 exceeds twice the largest sum of 16384 products.
// Each modulus is one plain integer GEMM on matrix cores,
//   * int8 residues, v_mfma_i32_32x32x32_i8, int32 accumulation;
//   * BF16 residues (integers |r| <= 128 are exact in BF16),
//     v_mfma_f32_32x32x16_bf16, FP32 accumulation reduced mod m every 640 k,
//     before any partial sum can exceed 2^24,
// its sums are reduced mod m to one byte per output and modulus, and a last
// pass puts the sixteen bytes of an output together to the 128-bit integer
// T = sum_k X_ik Y_kj and rounds it once to float-float:
//     C_ij ~ T 2^(e_i + f_j - 108).
// K beyond 16384 is split into chunks summed with Add22.  No binary64
// arithmetic is used anywhere.  Error sources: rounding of X (at most one
// unit of 2^(e_i - 54) per entry) and the final rounding (2^-48 |C_ij|).
//
// Why residues: sixteen products instead of the 28 digit-pair products that
// seven 8-bit digits per operand need for the same 54 bits (and those drop
// the 21 pairs below 2^-56).  The matrix products are bound by the power that
// the matrix cores draw (the chip clocks down to 1.7-1.8 GHz under either
// form), so fewer products is what counts: at 4096^3 the product kernel takes
// 0.91 ms against 1.55 ms for the digit pairs, and the other passes over the
// planes 0.36 against 0.20 ms.
//
// Four launches: partial maxima, and per chunk of K and panel of C residue planes,
// products and reconstruction.

#include <type_traits>

#include "ff_device.h"
#include "ff_gemm_residue.h"
#include "ff_host.h"

namespace ffk {

// ----------------------------------------------------------------- plain

// Workgroup = 16 R x 16 R outputs, R x R per thread, K in stages of KS entries
// through LDS; the next stage is loaded while one is multiplied.  An output is a
// serial chain of ~26 operations per k, so a small product is bound by the
// chains that a wavefront carries: four by four per thread took 240 us at
// 200 x 300 x 257 on twenty workgroups, one per thread takes 23; with
// workgroups enough the vector unit is the bound (1024^3: 1010 us with four by
// four, 516 now, 2 x 2).
template <int R, int KS>
__global__ __launch_bounds__(256) void gemm_fma_loop(int64_t M, int64_t N, int64_t K,
                                                     const float *__restrict__ Ah,
                                                     const float *__restrict__ Al, int64_t lda,
                                                     const float *__restrict__ Bh,
                                                     const float *__restrict__ Bl, int64_t ldb,
                                                     float *__restrict__ Ch,
                                                     float *__restrict__ Cl, int64_t ldc)
{
    constexpr int kTile = 16 * R, kPer = kTile * KS / 256;
    __shared__ float sAh[KS][kTile + 1], sAl[KS][kTile + 1];
    __shared__ float sBh[KS][kTile], sBl[KS][kTile];
    const int t = threadIdx.x, tx = t % 16, ty = t / 16;
    const int64_t i0 = static_cast<int64_t>(blockIdx.y) * kTile;
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kTile;
    float ch[R][R], cl[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c)
            ch[r][c] = cl[r][c] = 0.0f;
    float fah[kPer], fal[kPer], fbh[kPer], fbl[kPer];
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            const int e = n * 256 + t;
            const int64_t ai = i0 + e / KS, ak = k0 + e % KS;
            const bool in_a = ai < M && ak < K;
            fah[n] = in_a ? Ah[ai * lda + ak] : 0.0f;
            fal[n] = in_a ? Al[ai * lda + ak] : 0.0f;
            const int64_t bk = k0 + e / kTile, bj = j0 + e % kTile;
            const bool in_b = bk < K && bj < N;
            fbh[n] = in_b ? Bh[bk * ldb + bj] : 0.0f;
            fbl[n] = in_b ? Bl[bk * ldb + bj] : 0.0f;
        }
    };
    auto term = [&](int kk) {
        float ah[R], al[R], bh[R], bl[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ah[r] = sAh[kk][ty + 16 * r];
            al[r] = sAl[kk][ty + 16 * r];
            bh[r] = sBh[kk][tx + 16 * r];
            bl[r] = sBl[kk][tx + 16 * r];
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < R; ++c) {
                float ph, pl;
                ffd::mul22<false>(ah[r], al[r], bh[c], bl[c], ph, pl);
                ffd::add22(ch[r][c], cl[r][c], ph, pl, ch[r][c], cl[r][c]);
            }
    };
    fetch(0);
    for (int64_t k0 = 0; k0 < K; k0 += KS) {
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            const int e = n * 256 + t;
            sAh[e % KS][e / KS] = fah[n];
            sAl[e % KS][e / KS] = fal[n];
            sBh[e / kTile][e % kTile] = fbh[n];
            sBl[e / kTile][e % kTile] = fbl[n];
        }
        __syncthreads();
        fetch(k0 + KS);   // beyond K: zeros, not used
        if (K - k0 >= KS) {
#pragma unroll 4
            for (int kk = 0; kk < KS; ++kk)
                term(kk);
        } else {
            for (int kk = 0; kk < static_cast<int>(K - k0); ++kk)
                term(kk);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int64_t gi = i0 + ty + 16 * r, gj = j0 + tx + 16 * c;
            if (gi < M && gj < N) {
                Ch[gi * ldc + gj] = ch[r][c];
                Cl[gi * ldc + gj] = cl[r][c];
            }
        }
}

// ---------------------------------------------------------------- sliced

constexpr int kP = 54;                // fixed-point bits: |X| <= 2^kP
constexpr int64_t kMaxKChunk = 16384; // sums of this many products stay below P / 2
constexpr int kBlk = 32;              // rows (or columns) of one matrix-core operand
constexpr int kFragBytes = 1024;      // one operand: 32 rows by 32 bytes of K
constexpr int kXcds = 8;              // accelerator dies, one L2 each; workgroup b runs on die b % 8
constexpr int kStageFrags = 2;        // operands per block of rows and stage

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16 bytes of memory at any 4-byte alignment: the hardware loads and stores
// them in one instruction.  Every row of the operands is read this way; word
// by word, rows of odd lengths took 6.2 us (maxima) and 28.6 us (residues) at
// 1000 x 1531 x 2047, now 6.3 and 23.2.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct ResiduesI8 {
    using Acc = i32x16;
    static constexpr int kEsize = 1;
    static constexpr int kFragK = 32;      // K of one operand
    static constexpr int kFoldStages = 0;  // int32 sums: |S| <= 2^14 K <= 2^28
};
struct ResiduesBF16 {
    using Acc = f32x16;
    static constexpr int kEsize = 2;
    static constexpr int kFragK = 16;
    static constexpr int kFoldStages = 20; // FP32 sums reduced every 640 k: |S - 2^14 m| < 640 2^14
};

// Smallest e with |x| < 2^e for every x with |x| <= the value of bits ub.
__device__ __forceinline__ int exponent_bound(uint32_t ub)
{
    if (ub == 0)
        return 0;
    const int be = static_cast<int>(ub >> 23);
    return be == 0 ? -126 : be - 126;
}

// Partial maxima of |hi| (as bits): workgroups [0, row_groups) take four rows
// of A each by a 4096-k segment, one wavefront per row; the others take 64
// columns of B by a band of kColBand rows.  Partial maxima instead of atomics
// need no launch that clears them; the next launch reduces them per block.
constexpr int kRowSegment = 4096;
constexpr int kColBand = 128;

__global__ __launch_bounds__(256) void absmax_partials(
    int64_t M, int64_t N, int64_t K, const float *__restrict__ Ah, int64_t lda,
    const float *__restrict__ Bh, int64_t ldb, int64_t row_groups, int64_t col_groups,
    uint32_t *__restrict__ rowpart, uint32_t *__restrict__ colpart)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t rgrid = row_groups * ((K + kRowSegment - 1) / kRowSegment);
    int64_t b = blockIdx.x;
    if (b < rgrid) {
        const int64_t seg = b / row_groups;
        const int64_t row = (b % row_groups) * 4 + wave;
        if (row >= M)
            return;
        const int64_t k0 = seg * kRowSegment;
        const int64_t k1 = (k0 + kRowSegment < K) ? k0 + kRowSegment : K;
        const float *a = Ah + row * lda;
        uint32_t m = 0;
        if (k1 - k0 >= 4) {
            // entries past the end repeat the last four, so that eight loads
            // are in flight whatever the length
            for (int64_t k = k0 + 4 * lane; k - 4 * lane < k1; k += 8 * 256) {
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int64_t at = k + 256 * s < k1 - 4 ? k + 256 * s : k1 - 4;
                    const f32x4 v = *reinterpret_cast<const f32x4u *>(a + at);
                    m = max(m, max(max(__float_as_uint(v[0]) & 0x7fffffffu,
                                       __float_as_uint(v[1]) & 0x7fffffffu),
                                   max(__float_as_uint(v[2]) & 0x7fffffffu,
                                       __float_as_uint(v[3]) & 0x7fffffffu)));
                }
            }
        } else {
            for (int64_t k = k0; k < k1; ++k)
                m = max(m, __float_as_uint(a[k]) & 0x7fffffffu);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            m = max(m, static_cast<uint32_t>(__shfl_xor(static_cast<int>(m), off, 64)));
        if (lane == 0)
            rowpart[seg * M + row] = m;
        return;
    }
    // rows past K repeat the last one, so that every load is issued at once
    b -= rgrid;
    const int64_t band = b / col_groups, j0 = b % col_groups * 64;
    uint32_t m[4] = {0, 0, 0, 0};
    constexpr int kGroups = 16, kRows = kColBand / kGroups;
    __shared__ uint32_t part[kGroups][64];
    const int group = threadIdx.x / (256 / kGroups);
    const int64_t k0 = band * kColBand + group * kRows;
    const int64_t j = j0 + 4 * (threadIdx.x & 15);
    if (j + 4 <= N) {
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int64_t row = k0 + k < K ? k0 + k : K - 1;
            const f32x4 v = *reinterpret_cast<const f32x4u *>(Bh + row * ldb + j);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                m[u] = max(m[u], __float_as_uint(v[u]) & 0x7fffffffu);
        }
    } else {
        for (int u = 0; u < 4 && j + u < N; ++u)
            for (int k = 0; k < kRows; ++k) {
                const int64_t row = k0 + k < K ? k0 + k : K - 1;
                m[u] = max(m[u], __float_as_uint(Bh[row * ldb + j + u]) & 0x7fffffffu);
            }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        part[group][4 * (threadIdx.x & 15) + u] = m[u];
    __syncthreads();
    if (wave == 0 && j0 + lane < N) {
        uint32_t r = 0;
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
            r = max(r, part[g][lane]);
        colpart[band * N + j0 + lane] = r;
    }
}

// Residue planes.  Plane i of an operand holds its residues mod m_i as the
// matrix cores read them: for each block of 32 rows of A (columns of B) and
// each K-step of 32 bytes one contiguous 1 KiB operand, in which lane l of a
// wavefront finds its 16 bytes at 16 l: row l % 32, the K bytes 16 (l / 32)
// onwards.  Copying an operand into LDS and reading it back are then both
// straight 1 KiB accesses, free of bank conflicts without a swizzle.
// Rows beyond M (columns beyond N) and entries beyond K are zero.
//
// A workgroup writes `spans` times kResidueSpan K-entries of one block in all
// sixteen planes, each span staged through LDS while the loads of the next are
// in flight; a wavefront takes 16 rows by 16 K-entries at a
// time, in four rounds s of 64: lane l holds the seven digits of row l % 16,
// K-entry 4 s + l / 16.  The sums of digits times powers of 256 for all
// sixteen moduli are an int8 matrix product, moduli x digits by digits x
// entries, in four instructions per round: instruction j holds its constants
// in K group j alone and so takes the entries of the lanes l / 16 = j.  Lane l
// of its result has the moduli 4 (l / 16) .. + 3 of row l % 16, K-entry 4 s +
// j, so that after the four rounds a lane owns sixteen neighbouring residues
// of four moduli, and each of its four stores covers 256 consecutive bytes in
// four planes.  Vector work per entry: ~28 operations for the digits and 2.75
// per residue (residue_from_biased, and packing), against 7 per residue with
// dot products on the vector unit.  Both operands of 4096^3 (268 MB read, 537
// MB written): 160 us, 5.0 TB/s, against 175 us with dot products (vector unit
// 81 % busy then).
constexpr int kResidueSpan = 64;   // K-entries staged at a time

// Pitch in words of a staged row of A (K contiguous) and of a staged K row of
// B (columns contiguous): with these the entries of a round fall on distinct
// LDS banks.
constexpr int kPitchA = kResidueSpan + 4, kPitchB = kBlk + 16;
constexpr int kStaged = kResidueSpan * kPitchB > kBlk * kPitchA ? kResidueSpan * kPitchB
                                                               : kBlk * kPitchA;

template <class Dg>
__global__ __launch_bounds__(256, 4) void residue_planes(
    int64_t M, int64_t N, int64_t K, const float *__restrict__ Ah, const float *__restrict__ Al,
    int64_t lda, const float *__restrict__ Bh, const float *__restrict__ Bl, int64_t ldb, int nRB,
    int nCB, int nKB, int spans, const uint32_t *__restrict__ rowpart, int64_t rowpitch,
    const uint32_t *__restrict__ colpart, int64_t colpitch, int nseg, int nband,
    int *__restrict__ rowexp, int *__restrict__ colexp, uint8_t *__restrict__ Ap,
    uint8_t *__restrict__ Bp, int64_t plane_a, int64_t plane_b)
{
    constexpr int kPer = kResidueSpan * kBlk / 256;   // staged entries per thread and plane
    __shared__ alignas(16) float staged[2][kStaged];
    __shared__ uint32_t part[8][kBlk];
    __shared__ int exps[kBlk];
    const int t = threadIdx.x;
    const int k_padded = nKB * Dg::kFragK;
    const int per_group = spans * kResidueSpan;
    const int groups = (k_padded + per_group - 1) / per_group;
    const int64_t b = blockIdx.x;
    const int64_t blk_all = b / groups;
    const int first = static_cast<int>(b % groups) * per_group;
    const int last = first + per_group < k_padded ? first + per_group : k_padded;
    const bool is_a = blk_all < nRB;
    const int64_t blk = is_a ? blk_all : blk_all - nRB;
    const int64_t limit = is_a ? M : N;

    // 32 rows by kResidueSpan K-entries of A, or kResidueSpan K rows by 32
    // columns of B, 16 bytes per load
    const float *const ph = is_a ? Ah : Bh, *const pl = is_a ? Al : Bl;
    const int64_t ld = is_a ? lda : ldb, xn = is_a ? K : N, yn = is_a ? M : K;
    const int across = (is_a ? kResidueSpan : kBlk) / 4, pitch = is_a ? kPitchA : kPitchB;
    f32x4 fh[kPer / 4], fl[kPer / 4];
    auto fetch = [&](int span0) {
        const int64_t x0 = is_a ? span0 : blk * kBlk, y0 = is_a ? blk * kBlk : span0;
#pragma unroll
        for (int n = 0; n < kPer / 4; ++n) {
            const int q = n * 256 + t;
            const int64_t x = x0 + q % across * 4, y = y0 + q / across;
            const float *const h = ph + y * ld + x, *const l = pl + y * ld + x;
            if (y < yn && x + 4 <= xn) {
                fh[n] = *reinterpret_cast<const f32x4u *>(h);
                fl[n] = *reinterpret_cast<const f32x4u *>(l);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = y < yn && x + u < xn;
                    fh[n][u] = in ? h[u] : 0.0f;
                    fl[n][u] = in ? l[u] : 0.0f;
                }
            }
        }
    };
    fetch(first);
    {
        // the block's 32 exponents from the partial maxima
        const int64_t r = blk * kBlk + (t & 31);
        const uint32_t *src = is_a ? rowpart : colpart;
        const int n = is_a ? nseg : nband;
        uint32_t m = 0;
        if (r < limit)
            for (int s = t >> 5; s < n; s += 8)
                m = max(m, src[s * (is_a ? rowpitch : colpitch) + r]);
        part[t >> 5][t & 31] = m;
        __syncthreads();
        if (t < kBlk) {
            for (int s = 1; s < 8; ++s)
                m = max(m, part[s][t]);
            const int e = exponent_bound(m);
            exps[t] = e;
            if (first == 0 && r < limit)
                (is_a ? rowexp : colexp)[r] = e;
        }
        __syncthreads();
    }
    const int lane = t & 63, wave = t >> 6;
    const int row0 = 16 * (wave & 1);
    const int group = lane >> 4, row = row0 + (lane & 15);
    const int e = exps[row];
    const int step_k = is_a ? 1 : kPitchB, step_r = is_a ? kPitchA : 1;
    // constants of modulus lane % 16, in the K group of instruction j only
    int64_t c[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        c[j] = group == j ? static_cast<int64_t>(
                                static_cast<uint64_t>(kResidue.digit_hi[lane & 15]) << 32 |
                                kResidue.digit_lo[lane & 15])
                          : 0;
    // the four moduli of this lane's results
    BiasedModulus bm[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        bm[r] = kBiased.of[4 * group + r];
    const i32x4 bias = {bm[0].bits, bm[1].bits, bm[2].bits, bm[3].bits};
    const int64_t plane = is_a ? plane_a : plane_b;
    uint8_t *const dst =
        (is_a ? Ap : Bp) + 4 * group * plane + blk * nKB * kFragBytes + row * 16;
#pragma unroll 1
    for (int span0 = first; span0 < last; span0 += kResidueSpan) {
#pragma unroll
        for (int n = 0; n < kPer / 4; ++n) {
            const int at = (n * 256 + t) / across * pitch + (n * 256 + t) % across * 4;
            *reinterpret_cast<f32x4 *>(&staged[0][at]) = fh[n];
            *reinterpret_cast<f32x4 *>(&staged[1][at]) = fl[n];
        }
        __syncthreads();
        if (span0 + kResidueSpan < last)
            fetch(span0 + kResidueSpan);
#pragma unroll 1
        for (int in = 16 * (wave >> 1); in < kResidueSpan; in += 32) {
            const int k0 = span0 + in;
            if (k0 >= k_padded)
                break;
            const int at0 = (in + group) * step_k + row * step_r;
            uint32_t w[4][4 * Dg::kEsize];   // modulus, word of the 16 K-entries
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                uint32_t dl, dh;
                entry_digits(staged[0][at0 + 4 * s * step_k], staged[1][at0 + 4 * s * step_k], e, dl,
                             dh);
                const int64_t d = static_cast<int64_t>(static_cast<uint64_t>(dh) << 32 | dl);
                i32x4 v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = __builtin_amdgcn_mfma_i32_16x16x32_i8(c[j], d, bias, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (Dg::kEsize == 1) {
                        w[r][s] = pack_low_bytes(
                            residue_from_biased(v[0][r], bm[r]), residue_from_biased(v[1][r], bm[r]),
                            residue_from_biased(v[2][r], bm[r]), residue_from_biased(v[3][r], bm[r]));
                    } else {
                        // |r| <= 128 has at most 8 significant bits: its BF16
                        // pattern is the upper half of the binary32 one, exactly
                        w[r][2 * s] = __builtin_amdgcn_perm(
                            __float_as_uint(residue_float_from_biased(v[1][r], bm[r])),
                            __float_as_uint(residue_float_from_biased(v[0][r], bm[r])), 0x07060302u);
                        w[r][2 * s + 1] = __builtin_amdgcn_perm(
                            __float_as_uint(residue_float_from_biased(v[3][r], bm[r])),
                            __float_as_uint(residue_float_from_biased(v[2][r], bm[r])), 0x07060302u);
                    }
                }
            }
            // 16 K-entries of one row: half an operand row (int8) or one (BF16)
            uint8_t *const at = dst + static_cast<int64_t>(k0 / Dg::kFragK) * kFragBytes +
                                (Dg::kEsize == 1 ? k0 % Dg::kFragK / 16 * (kFragBytes / 2) : 0);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int h = 0; h < Dg::kEsize; ++h)
                    *reinterpret_cast<uint4 *>(at + r * plane + h * (kFragBytes / 2)) =
                        make_uint4(w[r][4 * h], w[r][4 * h + 1], w[r][4 * h + 2], w[r][4 * h + 3]);
        }
        __syncthreads();   // everyone has read the span before it is overwritten
    }
}

__device__ __forceinline__ i32x16 mma(const uint4 &a, const uint4 &b, const i32x16 &c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const i32x4 *>(&a),
                                                 *reinterpret_cast<const i32x4 *>(&b), c, 0, 0,
                                                 0);
}
__device__ __forceinline__ f32x16 mma(const uint4 &a, const uint4 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(&a),
                                                   *reinterpret_cast<const bf16x8 *>(&b), c, 0,
                                                   0, 0);
}

// One LDS DMA: 16 bytes per lane from `from + lane_off` to LDS bytes `to +
// 16 lane` (global_load_lds_dwordx4).  In assembly, so that the compiler does
// not track the LDS it writes and put waits for every DMA in flight before
// the reads of other stages: the waits are the kernel's own.  It has no
// register result, and a wait the compiler places for a load of its own can
// only become stricter by the operations it does not count.
__device__ __forceinline__ void lds_dma16(const uint8_t *from, uint32_t lane_off, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(to), "v"(lane_off), "s"(from)
                 : "memory");
}

// s_waitcnt immediate that waits until at most n vector-memory operations of
// this wavefront are outstanding (export and LDS counters left at maximum).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// s_waitcnt immediate that waits until at most n LDS operations of this
// wavefront are outstanding.
constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | ((n & 15) << 8); }

// Workgroup barrier without a memory fence: the LDS DMA of the next stages
// keeps flying across it (a __syncthreads fence would wait for it).  The
// "memory" clobber keeps the compiler from moving LDS accesses across.
__device__ __forceinline__ void barrier_no_fence() { asm volatile("s_barrier" ::: "memory"); }

// Modulus i, from bytes (uniform across the workgroup).
__device__ __forceinline__ int modulus_of(int i)
{
    constexpr auto word = [](int w) {
        return static_cast<uint32_t>(kModulus[4 * w] - 1) |
               static_cast<uint32_t>(kModulus[4 * w + 1] - 1) << 8 |
               static_cast<uint32_t>(kModulus[4 * w + 2] - 1) << 16 |
               static_cast<uint32_t>(kModulus[4 * w + 3] - 1) << 24;
    };
    constexpr uint32_t w0 = word(0), w1 = word(1), w2 = word(2), w3 = word(3);
    const uint32_t w = i < 8 ? (i < 4 ? w0 : w1) : (i < 12 ? w2 : w3);
    return static_cast<int>((w >> (8 * (i & 3))) & 255u) + 1;
}

// The products of the residue planes: workgroup = (modulus, 64 TM x 64 TN tile
// of C), four wavefronts of TM x TN matrix-core blocks (32 x 32) each.
//
// 4 x 4 (256 x 256 tiles, one wavefront per SIMD with all 256 accumulation
// registers): an operand read from LDS feeds four MFMAs, 64 LDS bytes per
// cycle and compute unit of the 128 it can deliver.  A wavefront keeps its
// matrix core busy by itself: operands are read one K-step ahead into a
// second register set, four stages of 64 K-bytes ring through LDS, and LDS
// reads and DMA are issued between MFMAs (an MFMA occupies the matrix core
// for 32 cycles and the issue port for 4).  One barrier per stage.  Measured
// at 4096^3 (int8): 0.88 ms, 2.50 POP/s, matrix cores busy 69 % of the
// cycles at 1.68 GHz.  BF16: the FP32 sums have to be reduced every 767 k at
// the latest; one block of sixteen sums per stage, between its MFMAs of the two
// K-steps and one sum per MFMA of the other blocks, is hidden by the matrix
// core: 1.61 ms at 4096^3 (1.37 PFLOP/s), against 2.07 ms reduced between
// stages; 224 against 285 us at 2048^3.
// 4 x 2 (256 x 128 tiles, three stages in the ring, two workgroups per compute
// unit): one works while the other starts or stores, at 96 LDS bytes per cycle
// for operands; the product kernel of 1000 x 1531 x 2047 takes 46 us, 51 with
// 2 x 2 (128 LDS bytes per cycle, all it can deliver).  2 x 2 and 1 x 1 are for
// outputs with too few larger tiles.
//
// Where the tiles of a modulus are few (own_xcd), each die computes two moduli
// alone, so that a plane is fetched into one L2 instead of all eight.
// Otherwise workgroups run modulus by modulus, so that the planes in use are
// one modulus's, and each XCD takes a contiguous run of its tiles.  Either way
// tiles are ordered in strips of four tile rows, so that neighbours share L2.
template <class Dg, int TM, int TN>
__global__ __launch_bounds__(256, TM * TN == 16 ? 1 : 2) void gemm_residues(
    const uint8_t *__restrict__ Ap, const uint8_t *__restrict__ Bp, int64_t plane_a,
    int64_t plane_b, int nKB, int nTI, int nTJ, uint8_t *__restrict__ Cr, int64_t plane_c,
    int exact, int own_xcd)
{
    using Acc = typename Dg::Acc;
    constexpr int kChunk = kStageFrags * kFragBytes;      // a block's bytes per stage
    constexpr int kSlotBytes = 2 * (TM + TN) * kChunk;
    constexpr int kShare = (TM + TN) / 2;                 // chunks each wave sends per stage
    constexpr int kDma = kShare * kStageFrags;            // DMA instructions per wave and stage
    constexpr int kRead = TM + TN;                        // operands per K-step and wave
    constexpr int kBlocks = TM * TN;
    constexpr int kSlots = TM == TN ? 4 : 3;
    __shared__ uint4 ring[kSlots * kSlotBytes / 16];
    uint8_t *const lds = reinterpret_cast<uint8_t *>(ring);
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) uint8_t *)lds));

    const int tiles = nTI * nTJ;
    int mod, ti, tj;
    {
        int j;
        if (own_xcd) {
            const int nth = blockIdx.x / kXcds;
            mod = blockIdx.x % kXcds * (kModuli / kXcds) + nth / tiles;
            j = nth % tiles;
        } else {
            mod = blockIdx.x / tiles;
            j = blockIdx.x % tiles;
            if (tiles % kXcds == 0)               // XCD j % 8 takes a contiguous run
                j = (j % kXcds) * (tiles / kXcds) + j / kXcds;
        }
        const int group = j / (4 * nTJ), rows = nTI - 4 * group < 4 ? nTI - 4 * group : 4;
        const int in = j - group * 4 * nTJ;
        ti = 4 * group + in % rows;
        tj = in / rows;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // this wavefront's DMA share of the 2 TM chunks of A and 2 TN of B
    const uint8_t *src[kShare];
#pragma unroll
    for (int c = 0; c < kShare; ++c) {
        const int n = wave * kShare + c;
        const bool of_a = n < 2 * TM;
        const int64_t blk = of_a ? static_cast<int64_t>(ti) * (2 * TM) + n
                                 : static_cast<int64_t>(tj) * (2 * TN) + n - 2 * TM;
        src[c] = (of_a ? Ap + mod * plane_a : Bp + mod * plane_b) + blk * nKB * kFragBytes;
    }
    const int nst = nKB / kStageFrags;
    // DMA q of stage st; past the end the last stage again, so that every
    // stage sends the same number and the waits below need no cases
    const uint32_t lane16 = lane * 16;
    auto dma = [&](int st, int q) {
        const int c = q / kStageFrags, h = q % kStageFrags;
        lds_dma16(src[c] + static_cast<int64_t>(st < nst ? st : nst - 1) * kChunk +
                      h * kFragBytes,
                  lane16,
                  lds_base + (st % kSlots) * kSlotBytes + (wave * kShare + c) * kChunk + h * kFragBytes);
    };

    const int m = modulus_of(mod);
    const float inv = 1.0f / static_cast<float>(m);
    Acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = Dg::kFoldStages > 0 ? kFoldUnits * m : 0;

    // BF16 residues: one FP32 sum reduced mod m
    auto fold = [&](int block, int r) {
        if constexpr (Dg::kFoldStages > 0) {
            const float c = acc[block / TN][block % TN][r];
            acc[block / TN][block % TN][r] = reduce_float(c, m, inv);
        }
    };

    uint4 f0[kRead], f1[kRead];
    const int oa = wm * TM * kChunk + lane * 16, ob = (2 * TM + wn * TN) * kChunk + lane * 16;
    // operand q (TM of A, then TN of B) of K-step kk in the slot at byte `at`
    auto read = [&](uint4 (&f)[kRead], int at, int kk, int q) {
        f[q] = *reinterpret_cast<const uint4 *>(
            lds + at + (q < TM ? oa + q * kChunk : ob + (q - TM) * kChunk) + kk * kFragBytes);
    };
    // MFMA q of a K-step
    auto mfma = [&](const uint4 (&f)[kRead], int q) {
        const int i = q / TN, j = q % TN;
        acc[i][j] = mma(f[i], f[TM + j], acc[i][j]);
    };
    constexpr int kSteps = kBlocks > kRead ? kBlocks : kRead;

#pragma unroll
    for (int s = 0; s < kSlots; ++s)
#pragma unroll
        for (int q = 0; q < kDma; ++q)
            dma(s, q);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((kSlots - 1) * kDma));
    barrier_no_fence();
    __builtin_amdgcn_sched_barrier(0);
    // Stage st, whose first K-step has been read into f0: multiplies it while
    // the second K-step is read; then, once stage st + 1 has landed everywhere
    // and everyone has read this slot, reads that stage's first K-step and
    // sends stage st + kSlots into this slot under the second K-step's MFMAs.
    // BF16: the sums of block `FOLD` are reduced between its MFMA of the first
    // K-step and that of the second, one sum per MFMA of the other blocks.
    auto stage = [&](int st, auto which, auto ahead) {
        constexpr int FOLD = decltype(which)::value;
        constexpr bool AHEAD = decltype(ahead)::value;
        constexpr bool kFold = FOLD >= 0 && FOLD < kBlocks;
        const int at = (st % kSlots) * kSlotBytes, next = ((st + 1) % kSlots) * kSlotBytes;
#pragma unroll
        for (int q = 0; q < kSteps; ++q) {
            if (q < kRead)
                read(f1, at, 1, q);
            if (q < kBlocks)
                mfma(f0, q);
            if (kFold && kBlocks == 16 && q > FOLD)
                fold(FOLD, q - FOLD - 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (kFold) {
            if constexpr (kBlocks == 16) {
                fold(FOLD, 15);
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    fold(FOLD, r);
            }
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((kSlots - 2) * kDma) & lgkmcnt_imm(0));
        barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kSteps; ++q) {
            if (q < kRead && AHEAD)
                read(f0, next, 0, q);
            if (kFold && kBlocks == 16 && q < FOLD)
                fold(FOLD, 15 - FOLD + q);
            if (q < kBlocks)
                mfma(f1, q);
            if (q < kDma)
                dma(st + kSlots, q);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int st = 0;
    if constexpr (Dg::kFoldStages == 0) {
#pragma unroll
        for (int q = 0; q < kRead; ++q)
            read(f0, 0, 0, q);
#pragma unroll 1
        do
            stage(st, std::integral_constant<int, -1>{}, std::true_type{});
        while (++st < nst);
    } else {
        // rounds of twenty stages; the sixteen blocks are folded in the stages
        // away from the loop's edge, and no operands are read ahead across it:
        // what is live there in ordinary registers was spilled
        static_assert(Dg::kFoldStages == 20, "stages of a round");
#define FF_STAGE(N)                                                                     \
    stage(st, std::integral_constant<int, (N >= 2 && N < 18) ? N - 2 : -1>{},           \
          std::integral_constant<bool, N != 19>{});                                     \
    if (++st == nst)                                                                    \
        break;
#pragma unroll 1
        for (;;) {
#pragma unroll
            for (int q = 0; q < kRead; ++q)
                read(f0, st % kSlots * kSlotBytes, 0, q);
            FF_STAGE(0) FF_STAGE(1) FF_STAGE(2) FF_STAGE(3) FF_STAGE(4)
            FF_STAGE(5) FF_STAGE(6) FF_STAGE(7) FF_STAGE(8) FF_STAGE(9)
            FF_STAGE(10) FF_STAGE(11) FF_STAGE(12) FF_STAGE(13) FF_STAGE(14)
            FF_STAGE(15) FF_STAGE(16) FF_STAGE(17) FF_STAGE(18) FF_STAGE(19)
        }
#undef FF_STAGE
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no DMA outlives the workgroup

    // Residue planes of C: per modulus and 32 x 32 block 1 KiB, word w of
    // lane l (rows 8 w + 4 (l / 32) + 0..3 of column l % 32) at 256 w + 4 l.
    const int64_t nCB = static_cast<int64_t>(nTJ) * (2 * TN);
    uint8_t *const out = Cr + mod * plane_c;
    auto store = [&](auto low_byte) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t rb = static_cast<int64_t>(ti) * (2 * TM) + wm * TM + i;
                const int64_t cb = static_cast<int64_t>(tj) * (2 * TN) + wn * TN + j;
                uint8_t *const dst = out + (rb * nCB + cb) * kFragBytes + lane * 4;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t r[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        r[u] = low_byte(acc[i][j][4 * w + u]);
                    *reinterpret_cast<uint32_t *>(dst + 256 * w) =
                        pack_low_bytes(r[0], r[1], r[2], r[3]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
    };
    // (the empty assembly keeps the compiler from computing the part common to
    // the two reductions for all 256 sums ahead of the branch, which would
    // hold them in as many registers again)
    if constexpr (Dg::kFoldStages > 0) {
        store([&](float c) { return residue_of_float(c, m, inv); });
    } else if (exact || m > 244) {
        store([&](int c) {
            asm volatile("; two steps" : "+v"(c));
            return reduce_low_byte(reduce_once(c, m, inv), m, inv);
        });
    } else {
        store([&](int c) {
            asm volatile("; one step" : "+v"(c));
            return reduce_low_byte(c, m, inv);
        });
    }
}

// Transposes a register of each of four lane groups: on return r[w] of lane
// group g holds what r[g] of lane group w held.
__device__ __forceinline__ void transpose_lane_groups(uint32_t (&r)[4])
{
    auto a = __builtin_amdgcn_permlane32_swap(r[0], r[2], false, false);
    auto b = __builtin_amdgcn_permlane32_swap(r[1], r[3], false, false);
    auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    r[0] = c[0];
    r[1] = c[1];
    r[2] = d[0];
    r[3] = d[1];
}

// C from its residues: workgroup = 32 x 32 block of C, wavefront w its rows
// 8 w + 4 (lane / 32) + 0..3 at column lane % 32, one row (u) at a time, so
// that a lane owns one output and its sixteen residues per round.
//
// The base-256 digits (sixteen, with overlaps) of sum_i r_i R_i - q P are an
// int8 matrix product, constants by residues: instruction triple g holds its
// constants in K group g alone and so takes the outputs of the lanes l / 16 =
// g; lane l of its result has digits 4 (l / 16) .. + 3 of output l % 16 of
// that group.  A transpose between the lane groups brings every lane the
// sixteen digits of its own output.  On the vector unit the same sums were
// 80 dot products and their register moves of 262 operations per output, and
// the kernel was bound by them: 135 us at 4096 x 4096, now 92 us (402 MB).
__global__ __launch_bounds__(256, 4) void combine_residues(
    int64_t M, int64_t N, int64_t nBJ, const uint8_t *__restrict__ Cr, int64_t nCB, int64_t plane,
    const int *__restrict__ rowexp, const int *__restrict__ colexp, float *__restrict__ Ch,
    float *__restrict__ Cl, int64_t ldc, int accumulate)
{
    constexpr ResidueTables tab = kResidue;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t bi = blockIdx.x / nBJ, bj = blockIdx.x % nBJ;
    const uint8_t *src = Cr + (bi * nCB + bj) * kFragBytes + wave * 256 + lane * 4;
    uint32_t v[kModuli];
#pragma unroll
    for (int i = 0; i < kModuli; ++i)
        v[i] = *reinterpret_cast<const uint32_t *>(src + i * plane);
    const int64_t i0 = bi * kBlk + 8 * wave + 4 * (lane >> 5), j = bj * kBlk + (lane & 31);
    const int fj = j < N ? colexp[j] - 2 * kP : 0;
    // constants of digit lane % 16, in the K group of triple g only
    int64_t lo[4], hi[4], mp[4];
    {
        const int d = lane & 15;
        const uint64_t l = static_cast<uint64_t>(kResidue.recon[d][1]) << 32 | kResidue.recon[d][0];
        const uint64_t h = static_cast<uint64_t>(kResidue.recon[d][3]) << 32 | kResidue.recon[d][2];
        const uint64_t p = kResidue.minus_p[d];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const bool mine = (lane >> 4) == g;
            lo[g] = mine ? static_cast<int64_t>(l) : 0;
            hi[g] = mine ? static_cast<int64_t>(h) : 0;
            mp[g] = mine ? static_cast<int64_t>(p) : 0;
        }
    }
    uint32_t o[4][4];   // residue bytes of output u: o[g][u], moduli 4 g .. 4 g + 3
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint32_t in[4] = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        transpose_bytes(in, o[g]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        // T / P is within 0.39 of an integer q = round(sum_i r_i R_i / P);
        // the rounded fractions are off by at most 2^-6 in all
        int f1 = 0, f0 = 32768;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f1 = dot4(o[g][u], tab.frac1[g], f1);
            f0 = dot4(o[g][u], tab.frac0[g], f0);
        }
        const int q = ((f1 << 8) + f0) >> 16;
        const int64_t bq = static_cast<uint32_t>((q + 128) ^ 128) & 0xffffu;
        const int64_t b0 = static_cast<int64_t>(static_cast<uint64_t>(o[1][u]) << 32 | o[0][u]);
        const int64_t b1 = static_cast<int64_t>(static_cast<uint64_t>(o[3][u]) << 32 | o[2][u]);
        const i32x4 zero = {0, 0, 0, 0};
        i32x4 s[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            s[g] = __builtin_amdgcn_mfma_i32_16x16x32_i8(lo[g], b0, zero, 0, 0, 0);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            s[g] = __builtin_amdgcn_mfma_i32_16x16x32_i8(hi[g], b1, s[g], 0, 0, 0);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            s[g] = __builtin_amdgcn_mfma_i32_16x16x32_i8(mp[g], bq, s[g], 0, 0, 0);
        // digits below 2^18.2 in absolute value, in pairs: 2^26.3
        uint32_t low[4], high[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            low[g] = static_cast<uint32_t>(s[g][0] + (s[g][1] << 8));
            high[g] = static_cast<uint32_t>(s[g][2] + (s[g][3] << 8));
        }
        transpose_lane_groups(low);
        transpose_lane_groups(high);
        uint32_t t[4];
        int carry = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int l = static_cast<int>(low[w]) + carry, h = static_cast<int>(high[w]);
            const int64_t x = static_cast<int64_t>(l) + (static_cast<int64_t>(h) << 16);
            t[w] = static_cast<uint32_t>(x);
            carry = static_cast<int>(x >> 32);
        }
        const int64_t i = i0 + u;
        if (i >= M || j >= N)
            continue;
        float h, l;
        int128_to_ff(t, rowexp[i] + fj, h, l);
        float *const ph = Ch + i * ldc + j, *const pl = Cl + i * ldc + j;
        if (accumulate)
            ffd::add22(*ph, *pl, h, l, h, l);
        *ph = h;
        *pl = l;
    }
}

__global__ __launch_bounds__(256) void zero_matrix(int64_t M, int64_t N, float *__restrict__ Ch,
                                                   float *__restrict__ Cl, int64_t ldc)
{
    const int64_t n = M * N;
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; e < n;
         e += static_cast<int64_t>(gridDim.x) * 256) {
        Ch[e / N * ldc + e % N] = 0.0f;
        Cl[e / N * ldc + e % N] = 0.0f;
    }
}

// The planes are this much more than their contents apart: with 16 MiB
// between planes the sixteen stores (or loads) of one position would all meet
// the same memory channel (residue planes of 4096 x 4096: 292 us against 252).
constexpr int64_t kPlaneSkew = 4096 + 256;

// Planes are held for one panel of C at a time, at most this many rows by columns,
// and of K for the chunk that one accumulation covers: 12.9 GB of them at most
// (21.5 in BF16).  Planes of whole operands took 206 GB at 65536^3, which the
// matrices (103 GB) left no room for.  Where there are several panels both ways,
// A's planes are formed anew for each panel of columns.  ms against planes of
// whole operands: 20000 x 20000 x 1000 8.96 / 9.06 (BF16 13.0 / 13.4), 32768 x 32768 x
// 2048 37.2 / 37.4, 4096 x 4096 x 40000 10.3 both.
constexpr int64_t kPanel = 16384;

struct ResidueGeom {
    int tm, tn;                // 32 x 32 blocks per wavefront: 1 x 1, 2 x 2, 4 x 2 or 4 x 4
    int64_t rows, cols;        // of a panel
    int64_t nseg, nband;       // partial maxima per row / column
    int64_t plane_a, plane_b, plane_c;
    size_t off_colpart, off_rowexp, off_colexp, off_a, off_b, off_c, total;
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline int64_t padded_steps(int64_t K, int frag_k)
{
    return ffh::cdiv(K, static_cast<int64_t>(frag_k) * kStageFrags) * kStageFrags;
}

inline ResidueGeom residue_geom(int64_t M, int64_t N, int64_t K, int frag_k)
{
    ResidueGeom g;
    g.rows = M < kPanel ? M : kPanel;
    g.cols = N < kPanel ? N : kPanel;
    // The tile of the least estimated time: the rounds of one workgroup per
    // compute unit that the tiles of a die make, times the cost of a round in
    // units of half a 256 x 128 one.  The costs were fitted to per-call times of
    // all four tiles at 40 shapes (int8 unless said): 4 x 2 against 4 x 4 and
    // 2 x 2 takes 45.4, 47.0 and 46.6 us at 1024^3, 347, 357 and 376 at 2560^3,
    // 447, 485 and 490 at 5000 x 5000 x 512; whole rounds matter between 2 x 2
    // and 4 x 2 (84.8 against 87.5 us at 1300^3, 101.4 against 97.1 at 1536^3);
    // 1 x 1 against 2 x 2 takes 16.8 and 17.3 us at 200 x 300 x 257, 48.9 and
    // 53.5 at 64 x 5000 x 1000, 23.2 and 22.2 at 512^3.  4 x 4 leaves the
    // start and end of a tile to one workgroup per compute unit and so pays
    // only from 96 K-steps on: 1166 against 1182 us at 4096^3 and 311 against
    // 315 at 2048^3 in BF16, but 690 against 675 at 4096 x 4096 x 2048.
    const int64_t nkb = padded_steps(K < kMaxKChunk ? K : kMaxKChunk, frag_k);
    constexpr struct {
        int tm, tn;
        double round;
    } kTiles[] = {{1, 1, 0.45}, {2, 2, 1.15}, {4, 2, 2.0}, {4, 4, 3.88}};
    double best = 0;
    for (const auto &t : kTiles) {
        if (t.tn == 4 && nkb < 96)
            break;
        const int64_t per_die =
            ffh::cdiv(g.rows, 64 * t.tm) * ffh::cdiv(g.cols, 64 * t.tn) * (kModuli / kXcds);
        const double cost = t.round * static_cast<double>(ffh::cdiv(per_die, 32));
        if (best == 0 || cost <= best) {
            best = cost;
            g.tm = t.tm;
            g.tn = t.tn;
        }
    }
    // The workspace holds whole 256 x 256 tiles whatever the tile, so that it grows
    // with every dimension and one for a caller's largest product serves the others.
    const int64_t blocks_a = ffh::cdiv(g.rows, 256) * 8, blocks_b = ffh::cdiv(g.cols, 256) * 8;
    g.nseg = ffh::cdiv(K, kRowSegment);
    g.nband = ffh::cdiv(K, kColBand);
    g.plane_a = blocks_a * nkb * kFragBytes + kPlaneSkew;
    g.plane_b = blocks_b * nkb * kFragBytes + kPlaneSkew;
    g.plane_c = blocks_a * blocks_b * kFragBytes + kPlaneSkew;
    size_t off = align256(sizeof(uint32_t) * g.nseg * M);
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    g.off_colpart = take(sizeof(uint32_t) * g.nband * N);
    g.off_rowexp = take(sizeof(int) * M);
    g.off_colexp = take(sizeof(int) * N);
    g.off_a = take(static_cast<size_t>(kModuli) * g.plane_a);
    g.off_b = take(static_cast<size_t>(kModuli) * g.plane_b);
    g.off_c = take(static_cast<size_t>(kModuli) * g.plane_c);
    g.total = off;
    return g;
}

template <class Dg>
ff_status sliced_gemm(int64_t M, int64_t N, int64_t K, const float *Ah, const float *Al,
                      int64_t lda, const float *Bh, const float *Bl, int64_t ldb, float *Ch,
                      float *Cl, int64_t ldc, void *ws, size_t ws_bytes, hipStream_t st)
{
    const ResidueGeom g = residue_geom(M, N, K, Dg::kFragK);
    if (!ws)
        return FF_ERR_NULL;
    if (ws_bytes < g.total)
        return FF_ERR_WORKSPACE;
    if (!ffh::aligned(ws, 256))
        return FF_ERR_ALIGN;
    if (M > int64_t(65535) * 4 || N > int64_t(65535) * 64 || K > int64_t(65535) * 64)
        return FF_ERR_SIZE;
    const int64_t row_groups = ffh::cdiv(M, 4), col_groups = ffh::cdiv(N, 64);
    const int64_t max_grid = row_groups * g.nseg + col_groups * g.nband;
    if (max_grid > INT32_MAX)
        return FF_ERR_SIZE;
    if (K == 0) {
        const int64_t blocks = ffh::cdiv(M * N, 256);
        hipLaunchKernelGGL(zero_matrix, dim3(static_cast<unsigned>(blocks < 4096 ? blocks : 4096)),
                           dim3(256), 0, st, M, N, Ch, Cl, ldc);
        return ffh::launch_status();
    }
    char *base = static_cast<char *>(ws);
    uint32_t *rowpart = reinterpret_cast<uint32_t *>(base);
    uint32_t *colpart = reinterpret_cast<uint32_t *>(base + g.off_colpart);
    int *rowexp = reinterpret_cast<int *>(base + g.off_rowexp);
    int *colexp = reinterpret_cast<int *>(base + g.off_colexp);
    uint8_t *Ap = reinterpret_cast<uint8_t *>(base + g.off_a);
    uint8_t *Bp = reinterpret_cast<uint8_t *>(base + g.off_b);
    uint8_t *Cr = reinterpret_cast<uint8_t *>(base + g.off_c);
    hipLaunchKernelGGL(absmax_partials, dim3(static_cast<unsigned>(max_grid)), dim3(256), 0, st, M, N, K,
                       Ah, lda, Bh, ldb, row_groups, col_groups, rowpart, colpart);
    auto product = g.tn == 4   ? gemm_residues<Dg, 4, 4>
                   : g.tm == 4 ? gemm_residues<Dg, 4, 2>
                   : g.tm == 2 ? gemm_residues<Dg, 2, 2>
                               : gemm_residues<Dg, 1, 1>;
    // One modulus's planes pass through one die's L2 while its tiles are few;
    // with more, each die's share of them is enough (447 against 470 us at
    // 5000 x 5000 x 512, 97 against 100 at 2500 x 2500 x 300), with fewer it
    // would fetch nearly all of both operands (57.6 against 45.4 us at 1024^3,
    // 18.5 against 16.8 at 200 x 300 x 257, 143 against 139 at 1700^3).
    auto panel = [&](int64_t i0, int64_t j0, int64_t k0) {
        const int64_t rows = M - i0 < g.rows ? M - i0 : g.rows;
        const int64_t cols = N - j0 < g.cols ? N - j0 : g.cols;
        const int64_t depth = K - k0 < kMaxKChunk ? K - k0 : kMaxKChunk;
        const int nKB = static_cast<int>(padded_steps(depth, Dg::kFragK));
        const int nTI = static_cast<int>(ffh::cdiv(rows, 64 * g.tm));
        const int nTJ = static_cast<int>(ffh::cdiv(cols, 64 * g.tn));
        const int nCB = nTJ * 2 * g.tn;
        // planes that an earlier panel left are used again
        const int form_rb = j0 == 0 || M > g.rows ? nTI * 2 * g.tm : 0;
        const int form_cb = i0 == 0 ? nCB : 0;
        if (form_rb + form_cb > 0) {
            // up to 8 spans per workgroup, as long as that leaves four per compute unit
            const int64_t all_spans = ffh::cdiv(nKB * Dg::kFragK, kResidueSpan);
            int spans = 8;
            while (spans > 1 && (form_rb + form_cb) * ffh::cdiv(all_spans, spans) < 1024)
                spans /= 2;
            const int64_t grid = (form_rb + form_cb) * ffh::cdiv(all_spans, spans);
            hipLaunchKernelGGL(residue_planes<Dg>, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                               st, rows, cols, depth, Ah + i0 * lda + k0, Al + i0 * lda + k0, lda,
                               Bh + k0 * ldb + j0, Bl + k0 * ldb + j0, ldb, form_rb, form_cb, nKB,
                               spans, rowpart + i0, M, colpart + j0, N, static_cast<int>(g.nseg),
                               static_cast<int>(g.nband), rowexp + i0, colexp + j0, Ap, Bp,
                               g.plane_a, g.plane_b);
        }
        const int own_xcd = nTI * nTJ <= 128 ? 1 : 0;
        hipLaunchKernelGGL(product, dim3(static_cast<unsigned>(kModuli * nTI * nTJ)), dim3(256), 0,
                           st, Ap, Bp, g.plane_a, g.plane_b, nKB, nTI, nTJ, Cr, g.plane_c,
                           nKB * Dg::kFragK > 4096 ? 1 : 0, own_xcd);
        const int64_t nBJ = ffh::cdiv(cols, kBlk);
        hipLaunchKernelGGL(combine_residues,
                           dim3(static_cast<unsigned>(ffh::cdiv(rows, kBlk) * nBJ)), dim3(256), 0,
                           st, rows, cols, nBJ, Cr, static_cast<int64_t>(nCB), g.plane_c,
                           rowexp + i0, colexp + j0, Ch + i0 * ldc + j0, Cl + i0 * ldc + j0, ldc,
                           k0 > 0 ? 1 : 0);
    };
    for (int64_t k0 = 0; k0 < K; k0 += kMaxKChunk)
        for (int64_t j0 = 0; j0 < N; j0 += g.cols)
            for (int64_t i0 = 0; i0 < M; i0 += g.rows)
                panel(i0, j0, k0);
    return ffh::launch_status();
}

} // namespace ffk

using namespace ffk;

extern "C" {

size_t ff_gemm_workspace_size(int64_t M, int64_t N, int64_t K, int32_t algo)
{
    if (M < 0 || N < 0 || K < 0)
        return 0;
    switch (algo) {
    case FF_GEMM_FMA_LOOP: return 0;
    case FF_GEMM_SLICED_BF16: return residue_geom(M, N, K, ResiduesBF16::kFragK).total;
    case FF_GEMM_SLICED_I8: return residue_geom(M, N, K, ResiduesI8::kFragK).total;
    default: return 0;
    }
}

ff_status ff_gemm(int64_t M, int64_t N, int64_t K, const float *A_hi, const float *A_lo,
                  int64_t lda, const float *B_hi, const float *B_lo, int64_t ldb, float *C_hi,
                  float *C_lo, int64_t ldc, int32_t algo, void *ws, size_t ws_bytes, void *stream)
{
    if (M < 0 || N < 0 || K < 0 || lda < K || ldb < N || ldc < N)
        return FF_ERR_SIZE;
    if (algo != FF_GEMM_FMA_LOOP && algo != FF_GEMM_SLICED_BF16 && algo != FF_GEMM_SLICED_I8)
        return FF_ERR_ARG;
    if (M == 0 || N == 0)
        return FF_OK;
    if (!C_hi || !C_lo || (K > 0 && (!A_hi || !A_lo || !B_hi || !B_lo)))
        return FF_ERR_NULL;
    for (const void *p : {static_cast<const void *>(A_hi), static_cast<const void *>(A_lo),
                          static_cast<const void *>(B_hi), static_cast<const void *>(B_lo),
                          static_cast<const void *>(C_hi), static_cast<const void *>(C_lo)})
        if (!ffh::aligned(p, 4))
            return FF_ERR_ALIGN;
    if (ffh::cdiv(M, 64) > 65535 || ffh::cdiv(N, 64) > INT32_MAX)
        return FF_ERR_SIZE;
    hipStream_t st = ffh::as_stream(stream);
    switch (algo) {
    case FF_GEMM_FMA_LOOP:
    {
        auto launch = [&](auto kernel, int tile) {
            ffh::in_parts(N, ffh::kMostThreads / 256 * tile, [&](int64_t at, int64_t cols) {
                hipLaunchKernelGGL(kernel,
                                   dim3(static_cast<unsigned>(ffh::cdiv(cols, tile)),
                                        static_cast<unsigned>(ffh::cdiv(M, tile))),
                                   dim3(256), 0, st, M, cols, K, A_hi, A_lo, lda, B_hi + at,
                                   B_lo + at, ldb, C_hi + at, C_lo + at, ldc);
            });
        };
        // as many outputs per thread (less LDS traffic each) as leave four
        // workgroups per compute unit; us with 1, 4 and 16: 1024^3 530 / 516 /
        // 890, 2048 x 2048 x 512 1024 / 959 / 940, 700 x 900 x 800 272 / 333 / 693
        if (ffh::cdiv(M, 64) * ffh::cdiv(N, 64) >= 1024)
            launch(gemm_fma_loop<4, 16>, 64);
        else if (ffh::cdiv(M, 32) * ffh::cdiv(N, 32) >= 1024)
            launch(gemm_fma_loop<2, 32>, 32);
        else
            launch(gemm_fma_loop<1, 32>, 16);
    }
        return ffh::launch_status();
    case FF_GEMM_SLICED_BF16:
        return sliced_gemm<ResiduesBF16>(M, N, K, A_hi, A_lo, lda, B_hi, B_lo, ldb, C_hi, C_lo, ldc,
                                       ws, ws_bytes, st);
    default:
        return sliced_gemm<ResiduesI8>(M, N, K, A_hi, A_lo, lda, B_hi, B_lo, ldb, C_hi, C_lo, ldc,
                                     ws, ws_bytes, st);
    }
}

} // extern "C"
