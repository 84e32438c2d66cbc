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

__host__ __device__ __forceinline__ int times24(float t, int neg_m)
{
    // (2^22 + q) (-m) as a 24-bit product (one multiply-add with the sum):
    // the low 24 bits of the float hold 2^22 + q with bit 23 clear
    const int n = static_cast<int>(__builtin_bit_cast(uint32_t, t) << 8) >> 8;
    return static_cast<int>(static_cast<uint32_t>(n) *
                            static_cast<uint32_t>((neg_m << 8) >> 8));
}

// s - q m for q = the integer nearest fl(fl(s) / m), in the low byte of the
// result (the magic number adds 2^22 m, a multiple of 256).  |s| < 2^22 m.
__host__ __device__ __forceinline__ uint32_t reduce_low_byte(int s, int m, float inv)
{
    const float t = __builtin_fmaf(static_cast<float>(s), inv, kRoundMagic);
    return static_cast<uint32_t>(s) + static_cast<uint32_t>(times24(t, -m));
}

// The same difference itself, as a signed integer.
__host__ __device__ __forceinline__ int reduce_once(int s, int m, float inv)
{
    return static_cast<int>(reduce_low_byte(s, m, inv) + (static_cast<uint32_t>(m) << 22));
}

// FP32 sums start at kFoldUnits m and are brought back to the m integers around
// it, exactly, before 640 products more can move them by 640 2^14.
constexpr int kFoldUnits = 16384;

__host__ __device__ __forceinline__ float reduce_float(float c, int m, float inv)
{
    const float n = __builtin_fmaf(c, inv, kRoundMagic) - (kRoundMagic + kFoldUnits);
    return __builtin_fmaf(n, -static_cast<float>(m), c);
}

// The residue of such a sum in the low byte.  1 / m in binary32 is off by up to
// 2^-24 of itself, so that the quotient of a sum beyond 2^23 can be the one next
// to the nearest, and the difference pass m / 2 by less than 1.  Only for 255 has a
// byte no room for that, above (128, at -8454907 and below); 1 / 255 rounds up,
// which takes differences of positive sums down and of negative ones up, and the
// sums lie above -6.4 10^6 because they start at 4.2 10^6.  (Up to 1.5 10^7, below
// 2^24: all exact.)
__host__ __device__ __forceinline__ uint32_t residue_of_float(float c, int m, float inv)
{
    const float t = __builtin_fmaf(c, inv, kRoundMagic);
    return static_cast<uint32_t>(static_cast<int>(c)) + static_cast<uint32_t>(times24(t, -m));
}

// A sum s of digit products, |s| < 2^17, read from the integer that an
// accumulation starting at the bits of the binary32 number `base` leaves: as a
// float it is base + s exactly.  base is a multiple of 256 m near 1.5 2^23, so
// that base / m is an integer and the low byte is that of s.
struct BiasedModulus {
    int bits;         // of base
    float base;
    float inv;        // 1 / m
    float offset;     // 1.5 2^23 - base / m, an integer
    int neg_m;
};

struct BiasedTable {
    BiasedModulus of[kModuli];
};

constexpr BiasedTable make_biased_table()
{
    BiasedTable b{};
    for (int i = 0; i < kModuli; ++i) {
        const int m = kModulus[i], units = 49152 / m;   // base = 256 m units
        const int base = 256 * m * units;
        b.of[i].bits = 0x4b000000 + (base - (1 << 23));  // of a float in [2^23, 2^24)
        b.of[i].base = static_cast<float>(base);
        b.of[i].inv = 1.0f / static_cast<float>(m);
        b.of[i].offset = kRoundMagic - static_cast<float>(256 * units);
        b.of[i].neg_m = -m;
    }
    return b;
}

constexpr BiasedTable kBiased = make_biased_table();

// s minus a multiple of m, in the low byte: the residue nearest zero, or the
// next one where the rounding of 1 / m (up to 2^-24 of base / m, 0.75 / m)
// moves a quotient over one half.  It stays within [-128, 127]: only 255 has no
// room above its largest balanced residue, and 1 / 255 rounds up, which moves
// quotients up and residues down.
__host__ __device__ __forceinline__ uint32_t residue_from_biased(int v, const BiasedModulus &b)
{
    const float t = __builtin_fmaf(__builtin_bit_cast(float, v), b.inv, b.offset);
    return static_cast<uint32_t>(v) + static_cast<uint32_t>(times24(t, b.neg_m));
}

// The same residue as a float.
__host__ __device__ __forceinline__ float residue_float_from_biased(int v, const BiasedModulus &b)
{
    const float x = __builtin_bit_cast(float, v), s = x - b.base;
    const float n = __builtin_fmaf(x, b.inv, b.offset) - kRoundMagic;
    return __builtin_fmaf(n, static_cast<float>(b.neg_m), s);
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

// Leading bits equal to the sign bit, counting it; -1 for 0 and -1
// (v_ffbh_i32, which no builtin names).
extern "C" __device__ int sign_bits(int x) __asm("llvm.amdgcn.sffbh.i32");

// Shifts the two's complement number n[3] .. n[0] left by 24 as long as its
// leading word holds 28 sign bits or more (a number of few bits: rare, so the
// wavefront tests for it together).  Returns the shift.
__device__ __forceinline__ int shift_out_signs(uint32_t (&n)[4])
{
    int sh = 0;
    for (int pass = 0; pass < 5; ++pass) {
        const bool few =
            static_cast<unsigned>(sign_bits(static_cast<int>(n[3]))) >= 28u;
        if (!__any(few))
            break;
        if (few) {
            n[3] = __builtin_amdgcn_alignbit(n[3], n[2], 8);
            n[2] = __builtin_amdgcn_alignbit(n[2], n[1], 8);
            n[1] = __builtin_amdgcn_alignbit(n[1], n[0], 8);
            n[0] <<= 24;
            sh += 24;
        }
    }
    return sh;
}

// (hi, lo) = (RN(T), RN(T - RN(T))) 2^scale for the 128-bit two's complement
// integer T = sum_k t[k] 2^(32 k), |T| < 2^124.  Signed words throughout: a
// leading word with a sticky bit for all that follows it converts to the
// nearest binary32 of the whole in two's complement too (the truncated part
// is positive and the rounding points are even).
__device__ __forceinline__ void int128_to_ff(uint32_t (&t)[4], int scale, float &hi, float &lo)
{
    scale += 96 - shift_out_signs(t);
    // two sign bits left, so |top| <= 2^30 and its rounding converts back;
    // T has at least four, so the funnel shifts are by 2 to 30
    const int z = sign_bits(static_cast<int>(t[3])) - 2;
    const int top = static_cast<int>(__builtin_amdgcn_alignbit(t[3], t[2], 32 - z));
    const uint32_t n2 = __builtin_amdgcn_alignbit(t[2], t[1], 32 - z);
    const uint32_t n1 = __builtin_amdgcn_alignbit(t[1], t[0], 32 - z);
    const uint32_t n0 = t[0] << (z & 31);
    const float f = static_cast<float>(top | static_cast<int>(min(n2 | n1 | n0, 1u)));
    const uint32_t d = static_cast<uint32_t>(top - static_cast<int>(f));   // |d| <= 32
    // T - hi = d 2^96 + ..., its leading word 24 bits up: at most 2^29
    uint32_t r[4] = {n0 << 24, __builtin_amdgcn_alignbit(n1, n0, 8),
                     __builtin_amdgcn_alignbit(n2, n1, 8), __builtin_amdgcn_alignbit(d, n2, 8)};
    const int sh = shift_out_signs(r);
    const int y = sign_bits(static_cast<int>(r[3])) - 1;      // 1 to 26
    const int low = static_cast<int>(__builtin_amdgcn_alignbit(r[3], r[2], 32 - y));
    const uint32_t rest = r[2] << (y & 31) | r[1] | r[0];
    const float g = static_cast<float>(low | static_cast<int>(min(rest, 1u)));
    scale -= z;
    hi = __builtin_ldexpf(f, scale);
    lo = __builtin_ldexpf(g, scale - 24 - sh - y);
}

} // namespace ffk
