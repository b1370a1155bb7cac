// Encoding and decoding on the device.
//
// Ecd (Fig. 1 item 3) is m_i = round(scale / N Re(zeta^-i sum_u W_u omega^(-u i))) with the slot
// values at the odd exponents 2u + 1 = +-5^j.  The transform runs in 128-bit fixed point (fix128.hpp):
// values scaled by the power of two that brings the largest below 2^125, halved in every stage, twiddles by
// 2^126, every product rounded once, and the last product with the scale exact before the one rounding (half
// away from zero).  Its error is below that of the 113-bit floating-point form on the host, and both
// round to the same integers.
//
// The work is N / 2 log2 N butterflies of four 128-bit products (about 270 instructions each): nothing for the device, so
// the time is launches and their latency, and a pass takes two stages per thread (three would halve
// the threads again).  N = 2^15: 9 launches, about 50 us, against 14 ms on one host core.
//
// Dec + Dcd: the residues are lifted to integers (the plaintext is below q_0 q_1 / 2; the other
// limbs check that), rounded to doubles and transformed in double precision in the host
// decoder's order of operations.
#include "kernels.hpp"
#include "fix128.hpp"

#include <stdexcept>

#define TPB 256

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct FixOps {
    typedef FixC C;
    static __device__ __forceinline__ C ld(const C* p) { return *p; }
    static __device__ __forceinline__ i128 val(u64 lo, u64 hi) { return (i128)(((u128)hi << 64) | lo); }
    static __device__ __forceinline__ C pack(i128 re, i128 im) {
        return C{(u64)re, (u64)((u128)re >> 64), (u64)im, (u64)((u128)im >> 64)};
    }
    static __device__ __forceinline__ void bfly(C& p, C& q, const C& w) {
        i128 pr = val(p.rl, p.rh), pi = val(p.il, p.ih), qr = val(q.rl, q.rh), qi = val(q.il, q.ih);
        bfly_fix(pr, pi, qr, qi, val(w.rl, w.rh), val(w.il, w.ih));
        p = pack(pr, pi);
        q = pack(qr, qi);
    }
};
// the host decoder's arithmetic: no contraction into fused multiply-adds
struct DblOps {
    typedef DblC C;
    static __device__ __forceinline__ C ld(const C* p) { return *p; }
    static __device__ __forceinline__ C mul(const C& a, const C& b) {
#pragma clang fp contract(off)
        return C{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
    }
    static __device__ __forceinline__ void bfly(C& p, C& q, const C& w) {
#pragma clang fp contract(off)
        const C u = {p.re - q.re, p.im - q.im};
        p = C{p.re + q.re, p.im + q.im};
        q = mul(u, w);
    }
};

// R (1 or 2) stages of the decimation-in-frequency transform from distance 'half' (the first one),
// natural input, bit-reversed output; load(position) and store(position, value) are the ends
template <class O, int R, class L, class S>
__device__ __forceinline__ void fft_pass(int log_n, int log_half, const typename O::C* W, L&& load, S&& store) {
    const int g = blockIdx.x * TPB + threadIdx.x;
    if (g >= (1 << (log_n - R))) return;
    const int ld = log_half - (R - 1), d = 1 << ld;  // the last stage's distance
    const int j = g & (d - 1), p = ((g >> ld) << (ld + R)) + j;
    const int ls = log_n - 1 - log_half;  // twiddle stride of the first stage
    if constexpr (R == 2) {
        typename O::C a = load(p), b = load(p + d), c = load(p + 2 * d), e = load(p + 3 * d);
        O::bfly(a, c, O::ld(W + ((int64_t)j << ls)));
        O::bfly(b, e, O::ld(W + ((int64_t)(j + d) << ls)));
        const typename O::C w = O::ld(W + ((int64_t)j << (ls + 1)));
        O::bfly(a, b, w);
        O::bfly(c, e, w);
        store(p, a);
        store(p + d, b);
        store(p + 2 * d, c);
        store(p + 3 * d, e);
    } else {
        typename O::C a = load(p), b = load(p + d);
        O::bfly(a, b, O::ld(W + ((int64_t)j << ls)));
        store(p, a);
        store(p + d, b);
    }
}

template <int R, bool FIRST, bool LAST>
__global__ __launch_bounds__(TPB) void k_encode_pass(EncTables E, EncArgs A, int log_half, FixC* x, int64_t* out) {
    const auto load = [&](int p) {
        if constexpr (FIRST) return FixOps::pack(to_fix(A.z[E.slot[p] & A.vmask], A.shift), 0);
        else return x[p];
    };
    const auto store = [&](int p, const FixC& v) {
        if constexpr (!LAST) {
            x[p] = v;
        } else {
            const int i = (int)brev_bits((u32)p, E.log_n);
            const FixC z = E.twist[i];
            const i128 y = mul_fix<126>(FixOps::val(v.rl, v.rh), FixOps::val(z.rl, z.rh)) -
                           mul_fix<126>(FixOps::val(v.il, v.ih), FixOps::val(z.il, z.ih));
            // |y| mant 2^-sh, rounded half up
            const u128 a = (u128)(y < 0 ? -y : y);
            u64 p0, p1, c, t;
            mul_wide((u64)a, A.mant, p0, c);
            mul_wide((u64)(a >> 64), A.mant, p1, t);
            const u128 mid = (u128)p1 + c;
            const u64 w1 = (u64)mid, w2 = t + (u64)(mid >> 64);  // words 1 and 2; word 0 is below the shift
            const auto shr = [&](int s) {  // bits from s >= 64 on
                return s >= 128 ? w2 >> (s - 128) : s > 64 ? (w1 >> (s - 64)) | (w2 << (128 - s)) : w1;
            };
            const int64_t r = (int64_t)(shr(A.sh) + (shr(A.sh - 1) & 1));
            out[i] = y < 0 ? -r : r;
        }
    };
    fft_pass<FixOps, R>(E.log_n, log_half, E.w, load, store);
}

template <int R, bool FIRST, bool LAST>
static void encode_pass(const EncTables& E, const EncArgs& A, int lh, FixC* x, int64_t* out, hipStream_t st) {
    const dim3 grid((unsigned)ceil_div((int64_t)1 << (E.log_n - R), TPB));
    ProfScope prof_(PK_EW, (FIRST ? 1.0 : 2.0) * sizeof(FixC) * (double)((int64_t)1 << E.log_n), st);
    HE_LAUNCH((k_encode_pass<R, FIRST, LAST>), grid, dim3(TPB), 0, st, E, A, lh, x, out);
}

void launch_encode(const EncTables& E, const EncArgs& A, FixC* x, int64_t* out, hipStream_t st) {
    if (E.log_n < 4 || A.sh < 66 || A.sh > 191) throw std::runtime_error("encode: unsupported shape");
    // two stages per pass; an odd count starts with one of one stage
    int lh = E.log_n - 1;
    if (E.log_n & 1) {
        encode_pass<1, true, false>(E, A, lh, x, out, st);
        lh -= 1;
    } else {
        encode_pass<2, true, false>(E, A, lh, x, out, st);
        lh -= 2;
    }
    for (; lh > 1; lh -= 2) encode_pass<2, false, false>(E, A, lh, x, out, st);
    encode_pass<2, false, true>(E, A, lh, x, out, st);
}

// ------------------------------------------------------------------ decryption's integers, Dcd
// (double)v of a signed 128-bit integer, rounded to nearest even as the host conversion does
__device__ __forceinline__ double to_double(i128 v) {
    u128 a = (u128)(v < 0 ? -v : v);
    const u64 hi = (u64)(a >> 64);
    int s = 0;
    if (hi) {  // 64 leading bits, the dropped ones as a sticky bit
        s = 64 - __clzll((long long)hi);
        const u128 rest = a & (((u128)1 << s) - 1);
        a = (a >> s) | (rest ? 1 : 0);
    }
    const u64 m = (u64)a;
    // both halves are exact, so the sum is rounded once
    const double d = ldexp((double)(u32)(m >> 32) * 4294967296.0 + (double)(u32)m, s);
    return v < 0 ? -d : d;
}

__global__ __launch_bounds__(TPB) void k_lift_centred(DevTables T, int nl, const u64* m, u64 q0inv, u64 half_lo, u64 half_hi,
                                                      double* out, u32* bad) {
    const int N = 1 << T.log_n;
    const int i = blockIdx.x * TPB + threadIdx.x;
    const ModP m0 = T.mods[0];
    const u64 x0 = m[i];
    if (nl == 1) {
        out[i] = to_double(x0 > (m0.q >> 1) ? (i128)x0 - (i128)m0.q : (i128)x0);
        return;
    }
    // x0 + q0 ((x1 - x0) q0^-1 mod q1), centred modulo q0 q1
    const ModP m1 = T.mods[1];
    const u64 k = mul_plain(sub_mod(m[N + i], reduce64(x0, m1), m1.q), q0inv, m1);
    u64 lo, hi;
    mul_wide(m0.q, k, lo, hi);
    const u128 w = (((u128)hi << 64) | lo) + x0;
    const bool neg = w > (((u128)half_hi << 64) | half_lo);
    mul_wide(m0.q, m1.q, lo, hi);
    const i128 v = neg ? (i128)w - (i128)(((u128)hi << 64) | lo) : (i128)w;
    bool wrong = false;
    for (int t = 2; t < nl; ++t) {
        const ModP mt = T.mods[t];
        const u64 q0t = reduce64(m0.q, mt);
        // w = x0 + q0 k, less q0 q1 when negative
        u64 kk = reduce64(k, mt);
        if (neg) kk = sub_mod(kk, reduce64(m1.q, mt), mt.q);
        const u64 r = add_mod(reduce64(x0, mt), mul_plain(q0t, kk, mt), mt.q);
        wrong = wrong || r != m[(int64_t)t * N + i];
    }
    if (wrong) *bad = 1;
    out[i] = to_double(v);
}

void launch_lift_centred(const DevTables& T, int nl, const u64* m, u64 q0inv, u64 half_lo, u64 half_hi, double* out,
                         u32* bad, hipStream_t st) {
    const int N = 1 << T.log_n;
    ProfScope prof_(PK_EW, (nl + 1.0) * 8.0 * N, st);
    HE_LAUNCH(k_lift_centred, dim3(ceil_div(N, TPB)), dim3(TPB), 0, st, T, nl, m, q0inv, half_lo, half_hi, out, bad);
}

template <int R, bool FIRST>
__global__ __launch_bounds__(TPB) void k_decode_pass(DecTables D, int log_half, const double* coeffs, DblC* x) {
    const auto load = [&](int p) {
        if constexpr (FIRST) {
            const double c = coeffs[p];
            return DblC{c * D.twist[p].re, c * D.twist[p].im};
        } else {
            return x[p];
        }
    };
    fft_pass<DblOps, R>(D.log_n, log_half, D.w, load, [&](int p, const DblC& v) { x[p] = v; });
}

__global__ __launch_bounds__(TPB) void k_decode_slots(DecTables D, const DblC* x, double scale, int n, double* out) {
    const int j = blockIdx.x * TPB + threadIdx.x;
    if (j < n) out[j] = x[D.pos[j]].re / scale;
}

template <int R, bool FIRST>
static void decode_pass(const DecTables& D, int lh, const double* c, DblC* x, hipStream_t st) {
    const dim3 grid((unsigned)ceil_div((int64_t)1 << (D.log_n - R), TPB));
    ProfScope prof_(PK_EW, (FIRST ? 1.5 : 2.0) * sizeof(DblC) * (double)((int64_t)1 << D.log_n), st);
    HE_LAUNCH((k_decode_pass<R, FIRST>), grid, dim3(TPB), 0, st, D, lh, c, x);
}

void launch_decode(const DecTables& D, const double* coeffs, double scale, DblC* x, int n_out, double* out,
                   hipStream_t st) {
    int lh = D.log_n - 1;
    if (D.log_n & 1) {
        decode_pass<1, true>(D, lh, coeffs, x, st);
        lh -= 1;
    } else {
        decode_pass<2, true>(D, lh, coeffs, x, st);
        lh -= 2;
    }
    for (; lh > 0; lh -= 2) decode_pass<2, false>(D, lh, coeffs, x, st);
    if (n_out <= 0) return;
    ProfScope prof_(PK_EW, 24.0 * n_out, st);
    HE_LAUNCH(k_decode_slots, dim3(ceil_div(n_out, TPB)), dim3(TPB), 0, st, D, x, scale, n_out, out);
}
