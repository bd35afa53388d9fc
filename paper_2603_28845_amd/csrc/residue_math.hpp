// Arithmetic of the products by residues (residue.hip): moduli, scales, an entry's residues, a sum's residue, the value that residues
// stand for.  Shared by the kernels and a host check (tests/residue_check.cpp); what the bounds in the comments rest on is asserted here.
#pragma once
#include <stdint.h>
#include <string.h>

#if defined(__HIPCC__)
#define ONECOMP_RES __host__ __device__ __forceinline__
#else
#define ONECOMP_RES inline
#endif

namespace onecomp {
namespace residue {

constexpr int MODULI = 14;
constexpr int MAX_K = 1 << 15;   // longest inner range, see product_kernel
// shift of a row whose entries no scale fits: every product with it is NaN
constexpr int32_t NO_SHIFT = INT32_MIN;

// Pairwise coprime; 256 needs no reduction, what the others leave of an entry has to fit 8 bits with the error of its quotient (see
// entry_margin: 251 leaves up to 127.3).
constexpr int MOD[MODULI] = {256, 251, 249, 247, 245, 241, 239, 233, 229, 227, 223, 211, 199, 197};   // 2^109.94
constexpr int BOUND_EXP = 109;            // BOUND = 2^108.8 = 0.8705 2^109
constexpr double BOUND_MANT = 0.87;

constexpr bool coprime() {
    for (int i = 0; i < MODULI; ++i)
        for (int j = 0; j < i; ++j) {
            int a = MOD[i], b = MOD[j];
            while (b != 0) { const int t = a % b; a = b; b = t; }
            if (a != 1) return false;
        }
    return true;
}
static_assert(coprime(), "two moduli share a factor");

struct Tables {
    float inv[MODULI];                  // 1 / m
    int c1[MODULI], c2[MODULI];         // 2^18 and 2^36 mod m, balanced
    double hi[MODULI], lo[MODULI];      // q / m in two parts, q the inverse of M / m: x / M = sum r q / m mod 1
    double M;
};
constexpr int balanced(int64_t x, int m) { return int(x % m) > m / 2 ? int(x % m) - m : int(x % m); }
constexpr Tables make_tables() {
    Tables t{};
    t.M = 1.0;
    for (int i = 0; i < MODULI; ++i) {
        const int m = MOD[i];
        t.inv[i] = 1.0f / float(m);
        t.c1[i] = balanced(int64_t(1) << 18, m);
        t.c2[i] = balanced(int64_t(1) << 36, m);
        int64_t p = 1;
        for (int j = 0; j < MODULI; ++j)
            if (j != i) p = p * MOD[j] % m;
        int64_t q = 1;
        while (p * q % m != 1) ++q;
        // the upper part in units of 2^-40, so that MODULI products with 8-bit residues add up exactly in 53 bits
        t.hi[i] = double((q << 40) / m) * 0x1p-40;
        t.lo[i] = double((q << 40) % m) / m * 0x1p-40;
        t.M *= m;
    }
    return t;
}
constexpr Tables TAB = make_tables();

// ---- how far a remainder by an fp32 quotient may lie from zero -------------------------------------------------------------
// q is the integer nearest to float(v) inv, so v - q m is off zero by m / 2, by what float(v) lost and by |v| |m inv - 1|, which the
// rounding of 1 / m costs.
constexpr double quotient_margin(int i, int64_t largest, double conversion) {
    const double e = double(MOD[i]) * double(TAB.inv[i]) - 1.0;
    return MOD[i] / 2.0 + conversion + double(largest) * (e < 0 ? -e : e);
}
constexpr int64_t magnitude(int c) { return c < 0 ? -int64_t(c) : c; }
// |n0|, |n1| and |n2| of an entry: no entry is longer than its row, whose square is at most BOUND (convert_columns_kernel allows it
// 2^-10.8 more), so |N| < 1.32 2^54
constexpr int64_t ENTRY_N1 = 1 << 17, ENTRY_N2 = 346000;
static_assert(BOUND_EXP == 109 && BOUND_MANT * (1.0 + 0x1p-10) * 2.0 < double(ENTRY_N2 - 1) * double(ENTRY_N2 - 1) * 0x1p-36, "n2 of the longest entry");
constexpr int64_t largest_entry(int i) { return ENTRY_N2 * magnitude(TAB.c2[i]) + ENTRY_N1 * (1 + magnitude(TAB.c1[i])); }
constexpr double entry_margin(int i) {   // float(v) is off by half a unit of its 24 bits: 2 below 2^26, 1 below 2^25, ..
    double half = 2.0;
    for (int64_t top = int64_t(1) << 25; half > 0.25 && largest_entry(i) <= top; top /= 2) half /= 2;
    return quotient_margin(i, largest_entry(i), half);
}
constexpr int64_t LARGEST_SUM = int64_t(MAX_K) << 14;   // products of two residues in [-128, 128)
constexpr double sum_margin(int i) { return quotient_margin(i, LARGEST_SUM, 16.0); }
constexpr bool margins_hold() {
    for (int i = 0; i < MODULI; ++i) {
        if (i > 0 && !(largest_entry(i) < (int64_t(1) << 26) && entry_margin(i) < 128.0)) return false;   // 8 bits hold it
        if (!(sum_margin(i) < MOD[i])) return false;                                                     // one m short at most
        // the quotient stays below 2^22, and with it the accumulator, which starts at 2^22 m, inside (0, 2^31)
        if (!(LARGEST_SUM < (int64_t(MOD[i]) << 22) && (int64_t(MOD[i]) << 22) + LARGEST_SUM < (int64_t(1) << 31))) return false;
    }
    return true;
}
static_assert(LARGEST_SUM == int64_t(1) << 29, "float(sum) is off by 16 at most");
static_assert(margins_hold(), "a residue leaves 8 bits, or a sum's remainder its modulus");

// ---- scales -------------------------------------------------------------------------------------------------------------
// the scale of a row of squared norm s
ONECOMP_RES int32_t shift_of(double s) {
    if (!(s < __builtin_inf())) return NO_SHIFT;
    if (!(s > 0.0)) return s == 0.0 ? 0 : NO_SHIFT;
    int e;
    const double f = __builtin_frexp(s, &e);          // s = f 2^e, f in [0.5, 1)
    const int d = BOUND_EXP - e;                      // f 2^(e + 2 shift) <= BOUND_MANT 2^BOUND_EXP
    return (d & 1) ? (d - 1) / 2 : f <= BOUND_MANT ? d / 2 : d / 2 - 1;
}

// ---- residues of an entry -------------------------------------------------------------------------------------------------
// a c + b, 24-bit factors: two of these are what the compiler makes two products and a sum of three of
ONECOMP_RES int mad24(int a, int c, int b) {
#if defined(__HIP_DEVICE_COMPILE__)
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(c), "v"(b));
    return r;
#else
    auto low = [](int x) { return int64_t(int32_t(uint32_t(x) << 8) >> 8); };
    return int(uint32_t(low(a) * low(c) + b));
#endif
}
ONECOMP_RES int low_word(double x) { return int(uint32_t(__builtin_bit_cast(uint64_t, x))); }

// N = rint(x) = n2 2^36 + n1 2^18 + n0 with |n0|, |n1| <= 2^17 and |n2| <= ENTRY_N2, each rounded by adding 1.5 2^52, whose sum holds
// it in its low word
ONECOMP_RES void split_entry(double x, int& n0, int& n1, int& n2) {
    constexpr double MAGIC = 0x1.8p52;
    const double h = __builtin_fma(x, 0x1p-36, MAGIC);
    const double l = __builtin_fma(-(h - MAGIC), 0x1p36, x);
    const double g = __builtin_fma(l, 0x1p-18, MAGIC);
    n2 = low_word(h);
    n1 = low_word(g);
    n0 = low_word(__builtin_fma(-(g - MAGIC), 0x1p18, l) + MAGIC);
}
// N mod MOD[i] in the low byte, in [-128, 128): n2 c2 + n1 c1 + n0 stays below 2^26, its quotient by m comes from fp32 (entry_margin).
// 1.5 2^23 + q holds q in its low bits; the offset 2^22 m it brings into the product leaves the low byte alone.
ONECOMP_RES uint32_t entry_residue(int n0, int n1, int n2, int i) {
    if (MOD[i] == 256) return uint32_t(n0);   // 2^18 and 2^36 are zero mod 256
    const int v = mad24(n2, TAB.c2[i], mad24(n1, TAB.c1[i], n0));
    const float t = __builtin_fmaf(float(v), TAB.inv[i], 12582912.0f);
    return uint32_t(mad24(int(__builtin_bit_cast(uint32_t, t)), -MOD[i], v));
}

// ---- residue of a sum -------------------------------------------------------------------------------------------------------
// (s - 2^22 m) mod m in [0, m) of an accumulator s that started at 2^22 m.  What the fp32 quotient leaves lies inside (-m, m)
// (sum_margin) and is one m short where negative.  1.5 2^23 + q holds q + 2^22 in its low 24 bits, and 2^22 m is what the
// accumulator started with.
ONECOMP_RES uint32_t sum_residue(int s, int m, float inv) {
    const float t = __builtin_fmaf(float(s - (m << 22)), inv, 12582912.0f);
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t v = uint32_t(s - __mul24(int(__builtin_bit_cast(uint32_t, t)), m));
#else
    const uint32_t v = uint32_t(s) - uint32_t(int32_t(__builtin_bit_cast(uint32_t, t) << 8) >> 8) * uint32_t(m);
#endif
    return v < v + uint32_t(m) ? v : v + uint32_t(m);
}

// ---- the value ------------------------------------------------------------------------------------------------------------
// x / M in [-1/2, 1/2] from x's residues, exactly but for 2^-82: the upper parts of q / m add up without rounding
struct Fraction {
    double hi = 0.0, lo = 0.0;
    ONECOMP_RES void add(uint32_t residue, int i) {
        const double r = double(residue);
        hi = __builtin_fma(r, TAB.hi[i], hi);
        lo = __builtin_fma(r, TAB.lo[i], lo);
    }
    ONECOMP_RES double value() const { return (hi - __builtin_rint(hi)) + lo; }
};
// a product of rows with scales ea and eb without them
ONECOMP_RES double unscaled(double v, int32_t ea, int32_t eb) {
    const bool none = ea == NO_SHIFT || eb == NO_SHIFT;   // sums with NO_SHIFT overflow
    v = __builtin_ldexp(v, none ? 0 : -(ea + eb));
    return none ? __builtin_nan("") : v;
}

}  // namespace residue
}  // namespace onecomp
