// Host check of csrc/residue_math.hpp: the kernels' own functions against 128-bit integers.
#include "../paper_2603_28845_amd/csrc/residue_math.hpp"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

using namespace onecomp::residue;
typedef __int128 i128;

static long checked = 0;
#define REQUIRE(c, ...)                                                                                          \
    do {                                                                                                         \
        ++checked;                                                                                               \
        if (!(c)) { std::printf("FAILED %s: ", #c); std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } \
    } while (0)

static int mod(i128 x, int m) { return int((x % m + m) % m); }

static void check_entry(double x) {
    int n0, n1, n2;
    split_entry(x, n0, n1, n2);
    const i128 n = i128(std::nearbyint(x));
    REQUIRE(i128(n2) * (i128(1) << 36) + i128(n1) * (1 << 18) + n0 == n, "parts of %a", x);
    REQUIRE(std::abs(n0) <= ENTRY_N1 && std::abs(n1) <= ENTRY_N1 && std::abs(n2) <= ENTRY_N2, "sizes of %a's parts", x);
    for (int i = 0; i < MODULI; ++i) {
        const int r = int8_t(entry_residue(n0, n1, n2, i));   // what the kernel stores
        REQUIRE(mod(r, MOD[i]) == mod(n, MOD[i]), "residue %d of %a mod %d", r, x, MOD[i]);
    }
}

int main() {
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> unit(-1.0, 1.0);
    for (int i = 0; i < MODULI; ++i) {
        const double q = (TAB.hi[i] + TAB.lo[i]) * MOD[i];
        int64_t p = 1;
        for (int j = 0; j < MODULI; ++j)
            if (j != i) p = p * MOD[j] % MOD[i];
        REQUIRE(q == std::nearbyint(q) && p * int64_t(q) % MOD[i] == 1, "inverse mod %d", MOD[i]);
    }

    const double longest = std::sqrt(BOUND_MANT * 2.0) * 0x1p54;
    for (double x : {0.0, 0.5, 1.5, 131072.0, 131071.5, 0x1p35, 0x1p35 + 131072.0, 0x1p36, 0x1p53, longest}) {
        check_entry(x);
        check_entry(-x);
    }
    for (int k = 0; k < 200000; ++k) check_entry(unit(rng) * std::exp2(std::uniform_real_distribution<double>(0.0, 54.399)(rng)));
    // parts at and near their ends, and values whose quotients by m lie next to a half
    for (int i = 1; i < MODULI; ++i) {
        const int m = MOD[i], top = int(largest_entry(i));
        auto check = [&](int n0, int n1, int n2) {
            const int r = int8_t(entry_residue(n0, n1, n2, i));
            REQUIRE(mod(r, m) == mod(i128(n2) * (i128(1) << 36) + i128(n1) * (1 << 18) + n0, m), "%d %d %d mod %d", n0, n1, n2, m);
        };
        const int s1 = TAB.c1[i] < 0 ? -1 : 1, s2 = TAB.c2[i] < 0 ? -1 : 1;
        for (int sign : {1, -1})
            for (int d2 = 0; d2 < 40; ++d2)
                for (int d1 = 0; d1 < 40; ++d1)
                    for (int d0 = 0; d0 < 2 * m; ++d0)
                        check(sign * int(ENTRY_N1 - d0), sign * s1 * int(ENTRY_N1 - d1), sign * s2 * int(ENTRY_N2 - d2));
        REQUIRE(top < 1 << 26, "largest entry mod %d", m);
    }

    for (int i = 0; i < MODULI; ++i) {
        const int m = MOD[i], start = m << 22;
        auto check = [&](int64_t s) {
            if (s < -LARGEST_SUM || s > LARGEST_SUM) return;
            REQUIRE(int(sum_residue(int(start + s), m, TAB.inv[i])) == mod(s, m), "sum %lld mod %d", (long long)s, m);
        };
        for (int64_t s = -LARGEST_SUM; s <= LARGEST_SUM; s += 9973) check(s);
        for (int64_t k = -(LARGEST_SUM / m); k <= LARGEST_SUM / m; k += 331)   // next to multiples and to halves between them
            for (int d = -2; d <= 2; ++d) { check(k * m + d); check(k * m + m / 2 + d); }
        for (int64_t d = 0; d < 4 * m; ++d) { check(LARGEST_SUM - d); check(d - LARGEST_SUM); }
    }

    for (int k = 0; k < 200000; ++k) {   // integers up to BOUND from their residues
        i128 x = i128(int64_t(rng())) * (i128(1) << 45) + int64_t(rng() >> 19);
        const int down = int(rng() % 108);
        x = k % 2 ? x : x / (i128(1) << down);
        Fraction f;
        for (int i = 0; i < MODULI; ++i) f.add(uint32_t(mod(x, MOD[i])), i);
        const double got = f.value() * TAB.M, want = double(x);
        REQUIRE(std::fabs(got - want) <= 0x1p-80 * TAB.M + 0x1p-51 * std::fabs(want), "value %a for %a", got, want);
    }

    const double bound = BOUND_MANT * std::ldexp(1.0, BOUND_EXP);
    for (int k = 0; k < 200000; ++k) {
        const double s = std::ldexp(0.5 + 0.5 * std::fabs(unit(rng)), int(rng() % 1200) - 600);
        const double scaled = std::ldexp(s, 2 * shift_of(s));
        REQUIRE(scaled <= bound && 4.0 * scaled > bound, "scale of %a", s);
    }
    REQUIRE(shift_of(0.0) == 0, "scale of zero");
    for (double s : {-1.0, double(INFINITY), double(NAN)}) REQUIRE(shift_of(s) == NO_SHIFT, "scale of %a", s);

    // rows without a scale, beside each other and beside ordinary ones, give NaN; no exponent is formed of theirs
    for (int32_t a : {NO_SHIFT, -640, -1, 0, 1, 640})
        for (int32_t b : {NO_SHIFT, -640, -1, 0, 1, 640}) {
            const double v = unscaled(0.75, a, b);
            if (a == NO_SHIFT || b == NO_SHIFT) REQUIRE(std::isnan(v), "%d, %d", a, b);
            else REQUIRE(v == std::ldexp(0.75, -(a + b)), "%d, %d", a, b);
        }
    std::printf("ok %ld\n", checked);
    return 0;
}
