// ff_gemm_residue.h -- the residue number system of the matrix-core product:
// sixteen pairwise coprime moduli, their constants, and the device steps that
// take a fixed-point entry to its residues and sixteen residues of an output
// back to the integer they stand for.
//
// Notation: m_i the moduli, P their product (2^125.37), R_i the integer below
// P in absolute value with R_i = 1 mod m_i and 0 mod the others, so that
// T = sum_i r_i R_i mod P for residues r_i of T.
#pragma once

#include "ff_device.h"

namespace ffk {

constexpr int kModuli = 16;
// The sixteen pairwise coprime integers up to 256 with the largest product:
// a balanced residue then fits a signed byte, and fifteen of them (2^117.8)
// would not hold the 2^124 that a product of K = 16384 terms needs.
constexpr int kModulus[kModuli] = {256, 255, 253, 251, 247, 241, 239, 233,
                                   229, 227, 223, 217, 211, 199, 197, 193};

typedef unsigned __int128 u128;

struct ResidueTables {
    // 256^t mod m_i, balanced, as signed bytes: t = 0..3 and t = 4..6
    uint32_t digit_lo[kModuli], digit_hi[kModuli];
    // signed base-256 digits (mod 2^128) of R_i: byte i % 4 of
    // recon[j][i / 4] is digit j of R_i
    uint32_t recon[16][kModuli / 4];
    // round(2^16 R_i / P) = 256 frac1 + frac0, signed bytes packed alike
    uint32_t frac1[kModuli / 4], frac0[kModuli / 4];
    // signed base-256 digits of -P (byte 0) and -256 P (byte 1), mod 2^128
    uint32_t minus_p[16];
};

constexpr int balanced(int r, int m) { return 2 * r > m - (m & 1 ? 0 : 1) ? r - m : r; }

constexpr ResidueTables make_residue_tables()
{
    ResidueTables t{};
    u128 P = 1;
    for (int i = 0; i < kModuli; ++i)
        P *= static_cast<u128>(kModulus[i]);
    for (int i = 0; i < kModuli; ++i) {
        const int m = kModulus[i];
        int power = 1 % m;
        for (int d = 0; d < 7; ++d) {
            const uint32_t byte = static_cast<uint32_t>(balanced(power, m)) & 0xffu;
            if (d < 4)
                t.digit_lo[i] |= byte << (8 * d);
            else
                t.digit_hi[i] |= byte << (8 * (d - 4));
            power = power * 256 % m;
        }
        const u128 rest = P / static_cast<u128>(m);
        const int rm = static_cast<int>(rest % static_cast<u128>(m));
        int inv = 1;
        while (rm * inv % m != 1)
            ++inv;
        u128 R = rest * static_cast<u128>(inv);   // < P
        const bool neg = R > P / 2;
        const u128 mag = neg ? P - R : R;         // |R_i|, at most P / 2
        // round(2^16 |R_i| / P), one doubling at a time
        u128 rem = mag;
        int f = 0;
        for (int b = 0; b < 16; ++b) {
            rem *= 2;
            f *= 2;
            if (rem >= P) {
                rem -= P;
                f += 1;
            }
        }
        if (2 * rem >= P)
            f += 1;
        if (neg)
            f = -f;
        const int f0 = ((f + 128) & 255) - 128;
        const int f1 = (f - f0) / 256;
        t.frac0[i / 4] |= (static_cast<uint32_t>(f0) & 0xffu) << (8 * (i % 4));
        t.frac1[i / 4] |= (static_cast<uint32_t>(f1) & 0xffu) << (8 * (i % 4));
        if (f1 < -128 || f1 > 127)
            t.frac1[0] = 1 / (f1 - f1);           // not a constant: fails to compile
        u128 v = neg ? ~mag + 1 : mag;
        for (int j = 0; j < 16; ++j) {
            const int d = ((static_cast<int>(v & 255) + 128) & 255) - 128;
            t.recon[j][i / 4] |= (static_cast<uint32_t>(d) & 0xffu) << (8 * (i % 4));
            v = (v >> 8) + (d < 0 ? 1 : 0);
        }
    }
    u128 v = ~P + 1;
    int below = 0;
    for (int j = 0; j < 16; ++j) {
        const int d = ((static_cast<int>(v & 255) + 128) & 255) - 128;
        t.minus_p[j] = (static_cast<uint32_t>(d) & 0xffu) |
                       ((static_cast<uint32_t>(below) & 0xffu) << 8);
        below = d;
        v = (v >> 8) + (d < 0 ? 1 : 0);
    }
    return t;
}

constexpr ResidueTables kResidue = make_residue_tables();

__device__ __forceinline__ int dot4(uint32_t a, uint32_t b, int c)
{
    return __builtin_amdgcn_sdot4(static_cast<int>(a), static_cast<int>(b), c, false);
}

// q = the integer nearest f / m, read from the low bits of the sum with
// 1.5 2^23: the float and its 23 low bits 2^22 + q.
constexpr float kRoundMagic = 12582912.0f;

__device__ __forceinline__ int times24(float t, int neg_m)
{
    // (2^22 + q) (-m) as a 24-bit product (one multiply-add with the sum):
    // the low 24 bits of the float hold 2^22 + q with bit 23 clear
    const int n = static_cast<int>(__float_as_uint(t) << 8) >> 8;
    return static_cast<int>(static_cast<uint32_t>(n) *
                            static_cast<uint32_t>((neg_m << 8) >> 8));
}

// s - q m for q = the integer nearest fl(fl(s) / m), in the low byte of the
// result (the magic number adds 2^22 m, a multiple of 256).  |s| < 2^22 m.
__device__ __forceinline__ uint32_t reduce_low_byte(int s, int m, float inv)
{
    const float t = __builtin_fmaf(static_cast<float>(s), inv, kRoundMagic);
    return static_cast<uint32_t>(s) + static_cast<uint32_t>(times24(t, -m));
}

// The same difference itself, as a signed integer.
__device__ __forceinline__ int reduce_once(int s, int m, float inv)
{
    return static_cast<int>(reduce_low_byte(s, m, inv) + (static_cast<uint32_t>(m) << 22));
}

// Bytes 0 of four words, packed.
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
    const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// 4 x 4 byte transpose: word o of the result holds byte o of each input word.
__device__ __forceinline__ void transpose_bytes(const uint32_t (&v)[4], uint32_t (&o)[4])
{
    const uint32_t a = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u);   // bytes 0, 1 of v0, v1
    const uint32_t b = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u);
    const uint32_t c = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);   // bytes 2, 3
    const uint32_t d = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(b, a, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(d, c, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(d, c, 0x07060302u);
}

// A float-float entry as the integer X = round(hi 2^(54 - e)) + round(lo
// 2^(54 - e)), returned as its seven signed base-256 digits (X = sum_t d_t
// 256^t, digit t in byte t of the two words).  Each word is split at weight
// 2^30 with exact binary32 steps: its upper part is an integer of at most 24
// significant bits, and the remainder times 2^30 is rounded to nearest.  The
// upper sum is clamped so that |X| <= 127 2^48 + 2^31, which seven digits hold
// (entries with |hi| < 2^e and |lo| <= ulp(hi) never reach it).
__device__ __forceinline__ void entry_digits(float hi, float lo, int e, uint32_t &d_lo,
                                             uint32_t &d_hi)
{
    constexpr float kTop = 33292288.0f;    // 127 2^18
    constexpr float kRest = 536870912.0f;  // 2^29: half a unit of the upper part
    const float h = __builtin_ldexpf(hi, 24 - e), l = __builtin_ldexpf(lo, 24 - e);
    const float hu = __builtin_rintf(h), lu = __builtin_rintf(l);
    const float hr = __builtin_rintf((h - hu) * 1073741824.0f);
    const float lr = __builtin_rintf((l - lu) * 1073741824.0f);
    int top = static_cast<int>(__builtin_amdgcn_fmed3f(hu, -kTop, kTop)) +
              static_cast<int>(__builtin_amdgcn_fmed3f(lu, -kTop, kTop));
    top = min(max(top, -33292288), 33292288);
    const int rest = static_cast<int>(__builtin_amdgcn_fmed3f(hr, -kRest, kRest)) +
                     static_cast<int>(__builtin_amdgcn_fmed3f(lr, -kRest, kRest));
    const int64_t X = (static_cast<int64_t>(top) << 30) + rest;
    // adding 128 to every digit makes the digits plain bytes; flipping bit 7
    // of each byte takes the 128 off again
    const uint64_t b = static_cast<uint64_t>(X) + 0x0080808080808080ull;
    d_lo = static_cast<uint32_t>(b) ^ 0x80808080u;
    d_hi = static_cast<uint32_t>(b >> 32) ^ 0x00808080u;
}

// (hi, lo) = (RN(T), RN(T - RN(T))) 2^scale for the 128-bit two's complement
// integer T = sum_k t[k] 2^(32 k).
__device__ __forceinline__ int normalise(uint32_t (&n)[4])
{
    // shifts the leading one bit to bit 31 of n[3]; returns the shift
    int sh = 0;
    if (n[3] == 0) {
        n[3] = n[2]; n[2] = n[1]; n[1] = n[0]; n[0] = 0;
        sh = 32;
    }
    if (n[3] == 0) {
        n[3] = n[2]; n[2] = n[1]; n[1] = 0;
        sh = 64;
    }
    if (n[3] == 0) {
        n[3] = n[2]; n[2] = 0;
        sh = 96;
    }
    const int z = n[3] ? __builtin_clz(n[3]) : 0;
    // funnel shifts right by 32 - z, of which the low five bits count: z = 0
    // is a shift by 0 of the lower word pair, so it takes its own select
    const uint32_t a3 = z ? __builtin_amdgcn_alignbit(n[3], n[2], 32 - z) : n[3];
    const uint32_t a2 = z ? __builtin_amdgcn_alignbit(n[2], n[1], 32 - z) : n[2];
    const uint32_t a1 = z ? __builtin_amdgcn_alignbit(n[1], n[0], 32 - z) : n[1];
    n[0] <<= z;
    n[3] = a3;
    n[2] = a2;
    n[1] = a1;
    return sh + z;
}

__device__ __forceinline__ void negate(uint32_t (&n)[4])
{
    const uint64_t lo = ~(static_cast<uint64_t>(n[1]) << 32 | n[0]) + 1;
    uint64_t hi = ~(static_cast<uint64_t>(n[3]) << 32 | n[2]);
    hi += lo == 0 ? 1 : 0;
    n[0] = static_cast<uint32_t>(lo);
    n[1] = static_cast<uint32_t>(lo >> 32);
    n[2] = static_cast<uint32_t>(hi);
    n[3] = static_cast<uint32_t>(hi >> 32);
}

__device__ __forceinline__ void int128_to_ff(uint32_t (&t)[4], int scale, float &hi, float &lo)
{
    const bool neg = static_cast<int32_t>(t[3]) < 0;
    if (neg)
        negate(t);
    const int s1 = normalise(t);
    // the top 32 bits with a sticky bit for the rest convert to the nearest
    // binary32 of the whole (32 >= 24 + 2)
    const uint32_t top = t[3];
    const float f = static_cast<float>(top | ((t[2] | t[1] | t[0]) ? 1u : 0u));
    // rounded up: the remainder is the low 104 bits minus 2^104
    const bool up = static_cast<uint32_t>(f * 0.00390625f) != top >> 8;
    t[3] = up ? (top & 255u) - 256u : top & 255u;
    if (up)
        negate(t);
    const int s2 = normalise(t);
    const float g = static_cast<float>(t[3] | ((t[2] | t[1] | t[0]) ? 1u : 0u));
    const float h = __builtin_ldexpf(f, scale + 96 - s1);
    const float l = __builtin_ldexpf(g, scale + 96 - s1 - s2);
    hi = neg ? -h : h;
    lo = (neg != up ? -l : l) + 0.0f;   // an exact zero comes back +0
}

} // namespace ffk
