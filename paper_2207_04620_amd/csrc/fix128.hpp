// 128-bit fixed point of the device encoder: host and device code, so that the error of the transform is checked
// on the CPU in the arithmetic that the kernels run.
#pragma once
#include <stdint.h>
#include <string.h>

#ifdef __HIP__
#define FIX_FN __host__ __device__ __forceinline__
#else
#define FIX_FN inline
#endif

typedef __int128 i128;
typedef unsigned __int128 u128;

// a b 2^-S (S = 126 or 127) for |b| <= 2^126, rounded to nearest (a half up).  Rounded down instead, the bias
// of half a unit adds up coherently along the transform.
template <int S>
FIX_FN i128 mul_fix(i128 a, i128 b) {
    const uint64_t al = (uint64_t)a, ah = (uint64_t)((u128)a >> 64), bl = (uint64_t)b, bh = (uint64_t)((u128)b >> 64);
    const u128 p0 = (u128)al * bl, p1 = (u128)al * bh, p2 = (u128)ah * bl, p3 = (u128)ah * bh;
    // word 1 of the product and its carries, with half a unit added
    const u128 mid = (p0 >> 64) + (uint64_t)p1 + (uint64_t)p2 + ((uint64_t)1 << (S - 65));
    u128 top = p3 + (uint64_t)(p1 >> 64) + (uint64_t)(p2 >> 64) + (uint64_t)(mid >> 64);
    if (a < 0) top -= (u128)b;  // the two's-complement words as signed numbers
    if (b < 0) top -= (u128)a;
    return (i128)((top << (128 - S)) | ((uint64_t)mid >> (S - 64)));
}

// Half a decimation-in-frequency butterfly, (p, q) <- ((p + q) / 2, (p - q) (c + i s) / 2), c and s times 2^126:
// magnitudes up to 2^125 stay there, so every stage keeps the whole word (with the growth of all stages left
// free from the start, the first ones round at the last one's unit).
FIX_FN void bfly_fix(i128& pr, i128& pi, i128& qr, i128& qi, i128 c, i128 s) {
    const i128 ur = pr - qr, ui = pi - qi;
    pr = (pr + qr + 1) >> 1;
    pi = (pi + qi + 1) >> 1;
    qr = mul_fix<127>(ur, c) - mul_fix<127>(ui, s);
    qi = mul_fix<127>(ur, s) + mul_fix<127>(ui, c);
}

// z 2^shift as an integer, truncated
FIX_FN i128 to_fix(double z, int shift) {
    uint64_t b;
    memcpy(&b, &z, 8);
    const int eb = (int)(b >> 52) & 2047;
    const uint64_t m = (b & 0xfffffffffffffull) | (eb ? 1ull << 52 : 0);
    const int s = (eb ? eb : 1) - 1075 + shift;
    const i128 v = s >= 0 ? (i128)((u128)m << s) : s > -64 ? (i128)(m >> -s) : 0;
    return (int64_t)b < 0 ? -v : v;
}

// exp(-i pi k / N) 2^126 for k < N: the first octant by Taylor series (errors of a few units, 2^-122), the others by
// symmetry.  The 113-bit tables' own errors, 2^-114 an entry, would be the largest part of the transform's.
inline void twist_fix(int log_n, i128* c, i128* s) {
    const int64_t n = (int64_t)1 << log_n;
    const int m = log_n - 2;
    const u128 pi = ((u128)0x3243F6A8885A308Dull << 64) | 0x313198A2E0370734ull;  // 2^124
    for (int64_t k = 0; k <= n / 4; ++k) {
        // pi k / N, at most pi / 4, times 2^126
        const i128 x = (i128)((pi >> m) * (u128)k + (((pi & (((u128)1 << m) - 1)) * (u128)k) >> m)), x2 = mul_fix<126>(x, x);
        i128 tc = (i128)1 << 126, ts = x, C = tc, S = x;
        for (int j = 1; tc || ts; ++j) {
            tc = -mul_fix<126>(tc, x2) / ((2 * j - 1) * (2 * j));
            ts = -mul_fix<126>(ts, x2) / ((2 * j) * (2 * j + 1));
            C += tc;
            S += ts;
        }
        c[k] = C, s[k] = -S;
        c[n / 2 - k] = S, s[n / 2 - k] = -C;
        c[n / 2 + k] = -S, s[n / 2 + k] = -C;
        if (k) c[n - k] = -C, s[n - k] = -S;
    }
}
