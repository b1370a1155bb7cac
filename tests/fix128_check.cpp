// The device encoder's fixed-point transform (csrc/fix128.hpp) and the host encoder's 113-bit one on the same values
// (one per line on stdin, after <log_n> on the command line): per coefficient, before the scale and the rounding,
// the fixed-point word, then the 113-bit value as mantissa and exponent; the first line is the shift of the fixed-point words.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2207_04620_amd/csrc/fix128.hpp"
#include "../paper_2207_04620_amd/csrc/host_math.hpp"

static void put(i128 v) {
    const u128 a = (u128)(v < 0 ? -v : v);
    printf("%s0x%016llx%016llx", v < 0 ? "-" : "", (unsigned long long)(a >> 64), (unsigned long long)a);
}

int main(int argc, char** argv) {
    if (argc != 2) return 1;
    const int log_n = atoi(argv[1]);
    const int64_t n = (int64_t)1 << log_n;
    std::vector<double> vals;
    double v, mx = 0;
    while (scanf("%lf", &v) == 1) vals.push_back(v), mx = std::fmax(mx, std::fabs(v));
    if (vals.empty() || (n / 2) % (int64_t)vals.size()) return 1;
    hm::Encoder E;
    E.init(log_n);
    int e;
    (void)std::frexp(mx, &e);
    const int shift = 125 - e;
    printf("%d\n", shift - log_n);
    std::vector<i128> xr(n), xi(n, 0), zr(n), zi(n);
    std::vector<f128> re(n), im(n, 0);
    twist_fix(log_n, zr.data(), zi.data());
    for (int64_t j = 0; j < n / 2; ++j) {
        const double z = vals[j % vals.size()];
        re[E.slot_pos[j]] = re[E.slot_neg[j]] = z;
        xr[E.slot_pos[j]] = xr[E.slot_neg[j]] = to_fix(z, shift);
    }
    for (int64_t half = n / 2, stride = 1; half >= 1; half >>= 1, stride <<= 1)
        for (int64_t b = 0; b < n; b += 2 * half)
            for (int64_t j = 0; j < half; ++j)
                bfly_fix(xr[b + j], xi[b + j], xr[b + j + half], xi[b + j + half], zr[2 * j * stride],
                         zi[2 * j * stride]);
    E.dif(re, im);
    for (int64_t i = 0; i < n; ++i) {
        const int64_t u = hm::bitrev((uint32_t)i, log_n);
        put(mul_fix<126>(xr[u], zr[i]) - mul_fix<126>(xi[u], zi[i]));
        const f128 y = re[u] * E.zr[i] - im[u] * E.zi[i];
        u128 bits;
        memcpy(&bits, &y, 16);
        const int ex = (int)(bits >> 112) & 0x7fff;
        const i128 m = (i128)((bits & (((u128)1 << 112) - 1)) | ((u128)(ex != 0) << 112));
        putchar(' ');
        put((bits >> 127) ? -m : m);
        printf(" %d\n", (ex ? ex : 1) - 16383 - 112);
    }
    return 0;
}
