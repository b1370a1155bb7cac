// libhe host runtime: context (primes, twiddles, keys, masks), the Fig. 1 operations,
// the packed product HE-MatMult (Alg. 3 + App. B) with hoisted rotations, the
// composite sign approximation (Sec. 4.2) and the C ABI declared in include/he.h.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <stdexcept>
#include <thread>
#include <unordered_map>
#include <vector>

#include "../../include/he.h"
#include "fix128.hpp"
#include "he_internal.hpp"

using namespace hm;

// ====================================================================== errors
const char* he_status_string(he_status s) {
    switch (s) {
        case HE_OK: return "ok";
        case HE_EINVAL: return "invalid argument";
        case HE_ENOMEM: return "out of memory";
        case HE_ELEVEL: return "level too low";
        case HE_ESCALE: return "scale out of range";
        case HE_EKEY: return "rotation key missing";
        case HE_ESHAPE: return "bad matrix shape";
        case HE_EMISMATCH: return "mismatched handles";
        case HE_EDEVICE: return "device error";
        default: return "unsupported";
    }
}

void hip_check(hipError_t e, const char* what) {
    if (e != hipSuccess) {
        fprintf(stderr, "libhe: HIP error %s in %s\n", hipGetErrorString(e), what);
        throw HeError(HE_EDEVICE);
    }
}

// ====================================================================== device pool
void* Pool::alloc(size_t bytes) {
    std::lock_guard<std::mutex> lk(m);
    bytes = (bytes + 255) & ~(size_t)255;
    if (capture) {  // a graph reuses its own blocks first; whatever it takes becomes its own
        auto gi = capture->free_.find(bytes);
        if (gi != capture->free_.end() && !gi->second.empty()) {
            void* p = gi->second.back();
            gi->second.pop_back();
            return p;
        }
    }
    void* p0 = alloc_locked(bytes);
    if (capture) capture->owned[p0] = bytes;
    return p0;
}
void* Pool::alloc_locked(size_t bytes) {
    auto it = free_.find(bytes);
    if (it != free_.end() && !it->second.empty()) {
        void* p = it->second.back();
        it->second.pop_back();
        cached -= bytes;
        peak = std::max(peak, held - cached);
        return p;
    }
    // the stream of a recording capture cannot be waited for (and nothing runs on it)
    const bool wait = !capture && !(sibling && sibling->capture);
    if (limit && held + bytes > limit) {
        trim_locked(wait);  // cached blocks of other sizes go back to the device first
        if (held + bytes > limit) throw HeError(HE_ENOMEM);
    }
    const auto take = [&]() -> void* {
        if (dev_alloc) return dev_alloc(bytes, user);
        void* p = nullptr;
        if (hipMalloc(&p, bytes) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    };
    void* p = take();
    if (!p) {  // the cached blocks of other sizes go back, the other cache's too
        trim_locked(wait);
        if (sibling) {
            std::lock_guard<std::mutex> lk2(sibling->m);
            sibling->trim_locked(wait);
        }
        p = take();
    }
    if (!p) throw HeError(HE_ENOMEM);
    held += bytes;
    peak = std::max(peak, held - cached);
    return p;
}
void Pool::release(void* p, size_t bytes) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(m);
    bytes = (bytes + 255) & ~(size_t)255;
    if (capture) {  // released while capturing: the graph's, reused only by that capture
        capture->owned[p] = bytes;
        capture->free_[bytes].push_back(p);
        return;
    }
    free_[bytes].push_back(p);
    cached += bytes;
}
void Pool::trim() {
    std::lock_guard<std::mutex> lk(m);
    trim_locked();
}
void Pool::trim_locked(bool wait) {
    // hipFree waits for the device; a caller's free need not
    if (dev_free && wait && owner && !free_.empty()) owner->drain();
    for (auto& kv : free_)
        for (void* p : kv.second) {
            if (dev_free) dev_free(p, user);
            else (void)hipFree(p);
            held -= kv.first;
            cached -= kv.first;
        }
    free_.clear();
}

void Ctx::drain() {
    (void)hipStreamSynchronize(home);
    if (side) (void)hipStreamSynchronize(side);
}

DBuf::DBuf(Ctx* c, size_t n_u64) : ctx(c), pool(c->alloc_side ? &c->pool_side : &c->pool), n(n_u64) {
    p = (u64*)pool->alloc(n_u64 * 8);
}
DBuf::~DBuf() {
    if (p) pool->release(p, n * 8);
}
// ====================================================================== context setup
static void gen_primes(int log_n, const std::vector<uint32_t>& bits, std::vector<uint64_t>& out) {
    const uint64_t m2n = 2ull << log_n;
    for (uint32_t b : bits) {
        if (b < 20 || b > 60) throw HeError(HE_EINVAL);
        const uint64_t top = 1ull << b;
        uint64_t cand = (top - 1) / m2n * m2n + 1;
        for (;; cand -= m2n) {
            if (cand <= (top >> 1)) throw HeError(HE_EINVAL);
            if (std::find(out.begin(), out.end(), cand) != out.end()) continue;
            if (is_prime(cand)) break;
        }
        out.push_back(cand);
    }
}

// smallest primitive 2N-th root of unity modulo q
static uint64_t min_root(uint64_t q, int64_t N) {
    uint64_t g = 0;
    for (uint64_t x = 2;; ++x) {
        const uint64_t r = powmod(x, (q - 1) / (2 * N), q);
        if (powmod(r, N, q) == q - 1) {
            g = r;
            break;
        }
    }
    uint64_t best = g, cur = g;
    const uint64_t g2 = mulmod(g, g, q);
    for (int64_t k = 1; k < N; ++k) {
        cur = mulmod(cur, g2, q);
        best = std::min(best, cur);
    }
    return best;
}

// host buffers handed to upload() may be freed right after it returns
static void upload(Ctx* c, void* dst, const void* src, size_t bytes) {
    hip_check(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, c->stream), "upload");
    hip_check(hipStreamSynchronize(c->stream), "upload sync");
}

// CDT thresholds T[k] = floor(2^63 Pr[|e| <= k]) of the rounded Gaussian on [-19, 19],
// rho(x) = exp(-x^2 / (2 sigma^2)), sigma = 3.2, computed in __float128
static void gauss_cdt(uint64_t out[19]) {
    auto exp128 = [](f128 x) {  // exp(x) = (exp(x / 2^10))^(2^10)
        f128 y = x / 1024, t = 1, s = 1;
        for (int k = 1; k < 40; ++k) {
            t *= y / (f128)k;
            s += t;
        }
        for (int k = 0; k < 10; ++k) s *= s;
        return s;
    };
    const f128 sigma = (f128)32 / (f128)10;
    f128 rho[20], tot = 0;
    for (int x = 0; x < 20; ++x) rho[x] = exp128(-(f128)(x * x) / (2 * sigma * sigma));
    tot = rho[0];
    for (int x = 1; x < 20; ++x) tot += 2 * rho[x];
    f128 cum = rho[0];
    const f128 two63 = (f128)(1ull << 62) * 2;
    for (int k = 0; k < 19; ++k) {
        if (k) cum += 2 * rho[k];
        out[k] = (uint64_t)(cum / tot * two63);
    }
}

int Ctx::ext_mod(int level, int i) const { return i <= level ? i : n_q + (i - level - 1); }

void Ctx::build_tables() {
    const int M = n_q + n_p;
    std::vector<ModP> mp(M);
    std::vector<u64> psi(M * (size_t)N), psi_sh(M * (size_t)N), ipsi(M * (size_t)N), ipsi_sh(M * (size_t)N);
    for (int m = 0; m < M; ++m) {
        const u64 q = mods[m];
        const u64 r = min_root(q, N), ri = invmod(r, q);
        roots.push_back(r);
        ModP& e = mp[m];
        e.q = q;
        e.qninv = mont_neg_inv(q);
        const u64 rm = r_mod(q);
        e.r2 = mulmod(rm, rm, q);
        e.bar = ~0ull / q;
        e.ninv = invmod((u64)N % q, q);
        e.ninv_sh = shoup(e.ninv, q);
        const int bits = 64 - __builtin_clzll(q);
        e.sh = (u32)(bits - 16);
        e.c = (u32)(((unsigned __int128)1 << (bits + 16)) / q);
        e.qinv = 1.0 / (double)q;
        // psi^(bitrev k)
        std::vector<u64> pw(N), ipw(N);
        u64 a = 1, b = 1;
        for (int64_t k = 0; k < N; ++k) {
            pw[k] = a;
            ipw[k] = b;
            a = mulmod(a, r, q);
            b = mulmod(b, ri, q);
        }
        for (int64_t k = 0; k < N; ++k) {
            const uint32_t br = bitrev((uint32_t)k, log_n);
            const size_t o = (size_t)m * N + k;
            psi[o] = pw[br];
            psi_sh[o] = shoup(pw[br], q);
            ipsi[o] = ipw[br];
            ipsi_sh[o] = shoup(ipw[br], q);
        }
    }
    d_mods = std::make_unique<DBuf>(this, (M * sizeof(ModP) + 7) / 8);
    d_psi = std::make_unique<DBuf>(this, (size_t)M * N);
    d_psi_sh = std::make_unique<DBuf>(this, (size_t)M * N);
    d_ipsi = std::make_unique<DBuf>(this, (size_t)M * N);
    d_ipsi_sh = std::make_unique<DBuf>(this, (size_t)M * N);
    upload(this, d_mods->p, mp.data(), M * sizeof(ModP));
    upload(this, d_psi->p, psi.data(), psi.size() * 8);
    upload(this, d_psi_sh->p, psi_sh.data(), psi.size() * 8);
    upload(this, d_ipsi->p, ipsi.data(), psi.size() * 8);
    upload(this, d_ipsi_sh->p, ipsi_sh.data(), psi.size() * 8);
    T.mods = (const ModP*)d_mods->p;
    T.psi = d_psi->p;
    T.psi_sh = d_psi_sh->p;
    T.ipsi = d_ipsi->p;
    T.ipsi_sh = d_ipsi_sh->p;
    T.log_n = log_n;
    T.n2_log = std::min(log_n, 11);
    T.n1_log = log_n - T.n2_log;
    T.fp64_mods = 0;
    for (int m = 0; m < M; ++m)
        if (fp64_limb(mp[m].q, T.n1_log, 1 << T.n2_log)) T.fp64_mods |= 1ull << m;
    host_mods = mp;

    // ---- row-pass twiddles in consumption order (N >= 2^11): row r of the second pass works
    // on twiddle exponents (N1 + r) 2^st + j; a group J of a round starting at stage s0 uses, for
    // its stages s0 + i (forward) or s0 - i (inverse), the pairs at (N1 + r) 2^st + (J << shift) + b
    T.rtw = T.irtw = nullptr;
    T.rtwd = T.irtwd = T.cold = T.icold = nullptr;
    if (T.n2_log == 11) {
        const int N1 = 1 << T.n1_log;
        std::vector<u64> rtw((size_t)M * N1 * ROW_TW * 2), irtw((size_t)M * N1 * ROW_TW * 2);
        static const int fr[4][2] = {{0, 3}, {3, 3}, {6, 3}, {9, 2}};
        static const int ir[4][2] = {{10, 3}, {7, 3}, {4, 3}, {1, 2}};
        for (int m = 0; m < M; ++m)
            for (int r = 0; r < N1; ++r) {
                const int64_t X = N1 + r;
                const size_t o = ((size_t)m * N1 + r) * ROW_TW * 2;
                size_t pos = 0;
                for (const auto& rd : fr) {
                    const int s0 = rd[0], R = rd[1];
                    for (int J = 0; J < (1 << s0); ++J)
                        for (int i = 0; i < R; ++i)
                            for (int b = 0; b < (1 << i); ++b) {
                                const size_t k = (size_t)m * N + (X << (s0 + i)) + ((int64_t)J << i) + b;
                                rtw[o + 2 * pos] = psi[k];
                                rtw[o + 2 * pos + 1] = psi_sh[k];
                                ++pos;
                            }
                }
                if (pos != ROW_TW) throw HeError(HE_EINVAL);
                pos = 0;
                for (const auto& rd : ir) {
                    const int s0 = rd[0], R = rd[1], G = 1 << R;
                    for (int J = 0; J < ((2048 / G) >> (11 - s0 - 1)); ++J)
                        for (int i = 0; i < R; ++i)
                            for (int b = 0; b < (G >> (i + 1)); ++b) {
                                const size_t k = (size_t)m * N + (X << (s0 - i)) + ((int64_t)J << (R - 1 - i)) + b;
                                irtw[o + 2 * pos] = ipsi[k];
                                irtw[o + 2 * pos + 1] = ipsi_sh[k];
                                ++pos;
                            }
                }
                if (pos != ROW_TW) throw HeError(HE_EINVAL);
            }
        d_rtw = std::make_unique<DBuf>(this, rtw.size());
        d_irtw = std::make_unique<DBuf>(this, irtw.size());
        upload(this, d_rtw->p, rtw.data(), rtw.size() * 8);
        upload(this, d_irtw->p, irtw.data(), irtw.size() * 8);
        T.rtw = d_rtw->p;
        T.irtw = d_irtw->p;
        // FP64 forms for primes below 2^46 (exact as doubles), each group of 2^R - 1 padded to 2^R
        std::vector<double> rtwd((size_t)M * N1 * ROW_TWD, 0.0), irtwd((size_t)M * N1 * ROW_TWD, 0.0),
            cold((size_t)M * N1, 0.0), icold((size_t)M * N1, 0.0);
        static const int fgroups[4][2] = {{1, 7}, {8, 7}, {64, 7}, {512, 3}}, igroups[4][2] = {{256, 7}, {32, 7}, {4, 7}, {1, 3}};
        for (int m = 0; m < M; ++m) {
            if (mods[m] >= (1ull << 46)) continue;
            for (int r = 0; r < N1; ++r) {
                const size_t src = ((size_t)m * N1 + r) * ROW_TW, dst = ((size_t)m * N1 + r) * ROW_TWD;
                const auto pad = [&](const int (&groups)[4][2], const std::vector<u64>& from, std::vector<double>& to) {
                    size_t i = src, o = dst;
                    for (const auto& g : groups)
                        for (int j = 0; j < g[0]; ++j, o += g[1] + 1)
                            for (int e = 0; e < g[1]; ++e) to[o + e] = (double)from[2 * i++];
                };
                pad(fgroups, rtw, rtwd);
                pad(igroups, irtw, irtwd);
            }
            for (int j = 0; j < N1; ++j) {
                cold[(size_t)m * N1 + j] = (double)psi[(size_t)m * N + j];
                icold[(size_t)m * N1 + j] = (double)ipsi[(size_t)m * N + j];
            }
        }
        d_rtwd = std::make_unique<DBuf>(this, rtwd.size());
        d_irtwd = std::make_unique<DBuf>(this, irtwd.size());
        d_cold = std::make_unique<DBuf>(this, cold.size());
        d_icold = std::make_unique<DBuf>(this, icold.size());
        upload(this, d_rtwd->p, rtwd.data(), rtwd.size() * 8);
        upload(this, d_irtwd->p, irtwd.data(), irtwd.size() * 8);
        upload(this, d_cold->p, cold.data(), cold.size() * 8);
        upload(this, d_icold->p, icold.data(), icold.size() * 8);
        T.rtwd = (const double*)d_rtwd->p;
        T.irtwd = (const double*)d_irtwd->p;
        T.cold = (const double*)d_cold->p;
        T.icold = (const double*)d_icold->p;
    }

    // ---- rescale constants: qinv[l][i] = q_l^-1 mod q_i
    std::vector<u64> qi((size_t)n_q * n_q, 0), qis((size_t)n_q * n_q, 0);
    for (int l = 1; l < n_q; ++l)
        for (int i = 0; i < l; ++i) {
            const u64 v = invmod(mods[l] % mods[i], mods[i]);
            qi[(size_t)l * n_q + i] = v;
            qis[(size_t)l * n_q + i] = shoup(v, mods[i]);
        }
    d_rs = std::make_unique<DBuf>(this, 2 * (size_t)n_q * n_q);
    upload(this, d_rs->p, qi.data(), qi.size() * 8);
    upload(this, d_rs->p + qi.size(), qis.data(), qis.size() * 8);

    // ---- ModDown: sources P, targets every Q limb; P^-1 mod q_t
    {
        std::vector<u64> tab((size_t)n_p * n_q * 2), pinv(n_q), pinv_sh(n_q);
        for (int s = 0; s < n_p; ++s) {
            const u64 qs = mods[n_q + s];
            u64 hs = 1;
            for (int r = 0; r < n_p; ++r)
                if (r != s) hs = mulmod(hs, mods[n_q + r] % qs, qs);
            md_hinv.push_back(invmod(hs, qs));
            md_hinv_sh.push_back(shoup(md_hinv.back(), qs));
            for (int t = 0; t < n_q; ++t) {
                const u64 qt = mods[t];
                u64 ht = 1;
                for (int r = 0; r < n_p; ++r)
                    if (r != s) ht = mulmod(ht, mods[n_q + r] % qt, qt);
                tab[((size_t)s * n_q + t) * 2 + 0] = to_mont(ht, qt);
                tab[((size_t)s * n_q + t) * 2 + 1] = to_mont((qt - mulmod(qs % qt, ht, qt)) % qt, qt);
            }
        }
        for (int t = 0; t < n_q; ++t) {
            u64 P = 1;
            for (int k = 0; k < n_p; ++k) P = mulmod(P, mods[n_q + k] % mods[t], mods[t]);
            pmod.push_back(P);
            pinv[t] = invmod(P, mods[t]);
            pinv_sh[t] = shoup(pinv[t], mods[t]);
        }
        d_md_tab = std::make_unique<DBuf>(this, tab.size());
        upload(this, d_md_tab->p, tab.data(), tab.size() * 8);
        d_pinv = std::make_unique<DBuf>(this, 2 * (size_t)n_q);
        upload(this, d_pinv->p, pinv.data(), n_q * 8);
        upload(this, d_pinv->p + n_q, pinv_sh.data(), n_q * 8);
    }

    // ---- ModUp: for each level l and digit j, sources I_j = [j a, min((j+1) a, l+1)),
    // targets all ext limbs (tab rows indexed by ext limb t in [0, l+1+K))
    mu.assign(n_q, {});
    size_t total = 0;
    for (int l = 0; l < n_q; ++l) {
        const int nl = l + 1, ne = nl + n_p, beta = (nl + alpha - 1) / alpha;
        for (int j = 0; j < beta; ++j) {
            ModUpInfo inf;
            inf.lo = j * alpha;
            inf.hi = std::min((j + 1) * alpha, nl);
            inf.off = total;
            total += (size_t)(inf.hi - inf.lo) * ne * 2;
            mu[l].push_back(inf);
        }
    }
    std::vector<u64> tab(total, 0);
    for (int l = 0; l < n_q; ++l) {
        const int nl = l + 1, ne = nl + n_p;
        for (auto& inf : mu[l]) {
            const int ns = inf.hi - inf.lo;
            for (int s = 0; s < ns; ++s) {
                const u64 qs = mods[inf.lo + s];
                u64 hs = 1;
                for (int r = 0; r < ns; ++r)
                    if (r != s) hs = mulmod(hs, mods[inf.lo + r] % qs, qs);
                inf.hinv[s] = invmod(hs, qs);
                inf.hinv_sh[s] = shoup(inf.hinv[s], qs);
                for (int t = 0; t < ne; ++t) {
                    const int tm = ext_mod(l, t);
                    const u64 qt = mods[tm];
                    u64 ht = 1;
                    for (int r = 0; r < ns; ++r)
                        if (r != s) ht = mulmod(ht, mods[inf.lo + r] % qt, qt);
                    tab[inf.off + ((size_t)s * ne + t) * 2 + 0] = to_mont(ht, qt);
                    tab[inf.off + ((size_t)s * ne + t) * 2 + 1] = to_mont((qt - mulmod(qs % qt, ht, qt)) % qt, qt);
                }
            }
        }
    }
    d_mu_tab = std::make_unique<DBuf>(this, std::max<size_t>(total, 1));
    upload(this, d_mu_tab->p, tab.data(), total * 8);

    // ---- output constants of the inverse transforms that feed a fused base conversion:
    // N^-1 (D/q_s)^-1 mod q_s as Shoup pairs, ModUp per (level, limb), ModDown per P prime
    {
        std::vector<u64> mus((size_t)n_q * n_q * 2, 0), mds((size_t)n_p * 2);
        for (int l = 0; l < n_q; ++l)
            for (const auto& inf : mu[l])
                for (int i = inf.lo; i < inf.hi; ++i) {
                    const u64 q = mods[i], f = mulmod(invmod((u64)N % q, q), inf.hinv[i - inf.lo], q);
                    mus[((size_t)l * n_q + i) * 2] = f;
                    mus[((size_t)l * n_q + i) * 2 + 1] = shoup(f, q);
                }
        for (int k = 0; k < n_p; ++k) {
            const u64 q = mods[n_q + k], f = mulmod(invmod((u64)N % q, q), md_hinv[k], q);
            mds[2 * k] = f;
            mds[2 * k + 1] = shoup(f, q);
        }
        d_mu_scale = std::make_unique<DBuf>(this, mus.size());
        upload(this, d_mu_scale->p, mus.data(), mus.size() * 8);
        d_md_scale = std::make_unique<DBuf>(this, mds.size());
        upload(this, d_md_scale->p, mds.data(), mds.size() * 8);
    }
    gauss_cdt(cdt);
    for (int t = 0; t < n_q; ++t) pmod_key.push_back((u64)((unsigned __int128)pmod[t] * (1ull << 60) % mods[t]));
    if (rescale_mfma_fits(T)) build_plans();
}

// Conversion plans of every level.  The constants of target t and source s are w_d = centred((D/q_s)
// 2^(8d) mod q_t), d < 8, each in signed bytes w_de; a set's A operands put byte e = 4 tile + r of
// target g at row 4 g + r, and digit d of source b at byte d of word 0 of the lanes of k block b (the
// layout in which the kernel holds the source words as B operands); source 4 + s is word 1 of the
// xs k blocks from xs s.  A set of fewer than four targets repeats its first.
void Ctx::build_plans() {
    const auto signed_byte = [](int64_t w, int e) { return (u64)(((uint64_t)w + 0x8080808080808080ull) >> (8 * e) & 255) ^ 128; };
    std::vector<ConvSet> sets;
    std::vector<u64> tab, rs_scale(2 * (size_t)n_q);
    // one digit: ns sources from limb slo with primes smod .., to the targets (limb offset, prime)
    const auto add_digit = [&](ConvPlan& P, int slo, int ns, int smod, const std::vector<std::pair<int, int>>& targets) {
        ConvDig& dg = P.dig[P.ndig++];
        dg = ConvDig{slo, ns, smod, P.nset, 0};
        P.src_limbs += ns;
        std::vector<std::pair<int, int>> kind[2];  // integer targets, FP64 targets
        for (auto& t : targets) kind[(T.fp64_mods >> t.second) & 1].push_back(t);
        P.dst_limbs += (double)targets.size();
        P.fp_limbs += (double)kind[1].size();
        for (int fp = 1; fp >= 0; --fp)
            for (size_t t0 = 0; t0 < kind[fp].size(); t0 += 4) {
                ConvSet S;
                memset(&S, 0, sizeof S);
                S.tab = (uint32_t)tab.size();
                S.nt = (uint8_t)std::min<size_t>(4, kind[fp].size() - t0);
                S.fp = (uint8_t)fp;
                const int ks = P.xs ? 2 : 1;
                tab.resize(tab.size() + 128 * (size_t)ks, 0);
                for (int g = 0; g < 4; ++g) {
                    const auto& t = kind[fp][t0 + (g < S.nt ? g : 0)];
                    const u64 q = mods[t.second];
                    S.doff[g] = (uint16_t)t.first;
                    S.dmod[g] = (uint8_t)t.second;
                    if (q < (1ull << 43)) S.small = 1;
                    const u64 c32 = (1ull << 32) % q;
                    S.w32[g] = c32;
                    S.w32_sh[g] = shoup(c32, q);
                    const u64 c77 = mulmod(mulmod(c32, c32, q), (1ull << 13) % q, q);
                    S.off[g] = (q - c77) % q;
                    if (S.off[g] < (1ull << 45)) S.off[g] += q;
                    for (int s = 0; s < ns; ++s) {
                        u64 w = 1 % q;  // D / q_s mod q, then times 2^8 per byte of the source
                        for (int r = 0; r < ns; ++r)
                            if (r != s) w = mulmod(w, mods[smod + r] % q, q);
                        for (int d = 0; d < 8; ++d) {
                            const int64_t wc = w > (q - 1) / 2 ? (int64_t)w - (int64_t)q : (int64_t)w;
                            for (int e = 0; e < 8; ++e) {
                                const int word = s >> 2, rep = word ? P.xs : 1;
                                for (int b = (word ? s - 4 : s) * rep, n = 0; n < rep; ++n, ++b)
                                    tab[S.tab + ((size_t)(e >> 2) * 64 + b * 16 + 4 * g + (e & 3)) * ks + word] |=
                                        signed_byte(wc, e) << (8 * d);
                            }
                            w = mulmod(w, 256 % q, q);
                        }
                    }
                }
                sets.push_back(S);
                ++dg.nset;
                ++P.nset;
            }
    };
    std::vector<size_t> first;  // each plan's first set
    plan_mu.assign(n_q, ConvPlan());
    plan_md.assign(n_q, ConvPlan());
    plan_rs.assign(n_q, ConvPlan());
    for (int l = 0; l < n_q; ++l) {
        const int nl = l + 1, ne = nl + n_p;
        first.push_back(sets.size());
        ConvPlan& U = plan_mu[l];
        U.xs = conv_mfma_share(T, std::min(alpha, nl));
        for (size_t j = 0; j < mu[l].size() && conv_mfma_fits(T, std::max(alpha, n_p), 1 << 16); ++j) {
            std::vector<std::pair<int, int>> t;
            for (int i = 0; i < ne; ++i)
                if (i < mu[l][j].lo || i >= mu[l][j].hi) t.push_back({(int)j * ne + i, ext_mod(l, i)});
            add_digit(U, mu[l][j].lo, mu[l][j].hi - mu[l][j].lo, mu[l][j].lo, t);
        }
        first.push_back(sets.size());
        ConvPlan& D = plan_md[l];
        D.xs = conv_mfma_share(T, n_p);
        std::vector<std::pair<int, int>> t;
        for (int i = 0; i < nl; ++i) t.push_back({i, i});
        if (conv_mfma_fits(T, std::max(alpha, n_p), 1 << 16)) add_digit(D, 0, n_p, n_q, t);
        first.push_back(sets.size());
        ConvPlan& R = plan_rs[l];
        t.pop_back();
        add_digit(R, 0, 1, l, t);
        rs_scale[2 * l] = host_mods[l].ninv;
        rs_scale[2 * l + 1] = host_mods[l].ninv_sh;
    }
    d_plan_sets = std::make_unique<DBuf>(this, (sets.size() * sizeof(ConvSet) + 7) / 8);
    d_plan_tab = std::make_unique<DBuf>(this, tab.size());
    d_rs_scale = std::make_unique<DBuf>(this, rs_scale.size());
    upload(this, d_plan_sets->p, sets.data(), sets.size() * sizeof(ConvSet));
    upload(this, d_plan_tab->p, tab.data(), tab.size() * 8);
    upload(this, d_rs_scale->p, rs_scale.data(), rs_scale.size() * 8);
    for (int l = 0; l < n_q; ++l) {
        ConvPlan* P[3] = {&plan_mu[l], &plan_md[l], &plan_rs[l]};
        const u64* sc[3] = {d_mu_scale->p + (size_t)l * n_q * 2, d_md_scale->p, d_rs_scale->p + 2 * (size_t)l};
        for (int k = 0; k < 3; ++k) {
            P[k]->sets = (const ConvSet*)d_plan_sets->p + first[3 * (size_t)l + k];
            P[k]->tab = d_plan_tab->p;
            P[k]->scale = sc[k];
        }
    }
}

// ====================================================================== small helpers
// src: the inverse transform reads limb k from there (same layout) instead of from base
void Ctx::ntt(u64* base, int npoly, int64_t pstride_limbs, int nl, bool inverse, int level_for_ext, const u64* src) {
    // job lists are capped; long ones are split
    Jobs J;
    J.base = base;
    J.src = src;
    J.cstride = 0;
    J.nct = 1;
    J.n = 0;
    for (int p = 0; p < npoly; ++p)
        for (int i = 0; i < nl; ++i) {
            J.off[J.n] = (uint16_t)(p * pstride_limbs + i);
            J.mod[J.n] = (uint8_t)(level_for_ext < 0 ? i : ext_mod(level_for_ext, i));
            if (++J.n == HE_MAXJ) {
                launch_ntt(T, J, inverse, stream);
                J.n = 0;
            }
        }
    if (J.n) launch_ntt(T, J, inverse, stream);
}

static ModMap qmap(const Ctx* c) { return ModMap{1 << 20, c->n_q}; }

// ====================================================================== keys
void Ctx::sample_into(u64* dst, int nl_modidx_count, const int* modidx, int kind, uint32_t purpose, u64 index,
                      const u64* uidx) {
    Jobs J;
    J.base = dst;
    J.cstride = 0;
    J.nct = 1;
    J.n = nl_modidx_count;
    for (int k = 0; k < J.n; ++k) {
        J.off[k] = (uint16_t)k;
        J.mod[k] = (uint8_t)modidx[k];
    }
    SampleArgs A;
    memset(&A, 0, sizeof A);
    A.seed = seed;
    A.poly[0] = {purpose, kind, index};
    if (uidx)
        for (int k = 0; k < J.n; ++k) A.uidx[k] = uidx[k];
    memcpy(A.cdt, cdt, sizeof cdt);
    launch_sample(T, J, A, stream);
}

void Ctx::keygen_base() {
    const int M = n_q + n_p;
    std::vector<int> all(M);
    for (int m = 0; m < M; ++m) all[m] = m;
    s_eval = std::make_unique<DBuf>(this, (size_t)M * N);
    sample_into(s_eval->p, M, all.data(), 0, P_SK, 0, nullptr);
    ntt(s_eval->p, 1, 0, M, false, -1);
    s2_eval = std::make_unique<DBuf>(this, (size_t)M * N);
    launch_ew(T, ModMap{1 << 20, n_q}, M, 1, s2_eval->p, 0, s_eval->p, 0, s_eval->p, 0, EW_MUL_PLAIN, stream);
    // public key over Q
    pk = std::make_unique<DBuf>(this, 2 * (size_t)n_q * N);
    u64* pk0 = pk->p;
    u64* pk1 = pk->p + (size_t)n_q * N;
    std::vector<u64> uidx(n_q);
    for (int i = 0; i < n_q; ++i) uidx[i] = (u64)i;
    sample_into(pk1, n_q, all.data(), 2, P_PK_A, 0, uidx.data());
    sample_into(pk0, n_q, all.data(), 1, P_PK_E, 0, nullptr);
    ntt(pk->p, 2, n_q, n_q, false, -1);
    // pk0 = e - a s
    DBuf as(this, (size_t)n_q * N);
    launch_ew(T, qmap(this), n_q, 1, as.p, 0, pk1, 0, s_eval->p, 0, EW_MUL_PLAIN, stream);
    launch_ew(T, qmap(this), n_q, 1, pk0, 0, pk0, 0, as.p, 0, EW_SUB, stream);
    launch_to_mont(T, qmap(this), n_q, 2, pk->p, (int64_t)n_q * N, stream);
    keys_bytes += (size_t)(2 * M + 2 * n_q) * N * 8;
}

// switching key from s' (evaluation form over all M primes) to s, words times 2^60; layout [beta][2][M][N]
std::unique_ptr<DBuf> Ctx::make_swk(u64 key_id, const u64* sp) {
    const int M = n_q + n_p, beta = (n_q + alpha - 1) / alpha;
    auto key = std::make_unique<DBuf>(this, (size_t)beta * 2 * M * N);
    std::vector<int> all(M);
    for (int m = 0; m < M; ++m) all[m] = m;
    DBuf e(this, (size_t)M * N);
    std::vector<uint8_t> flag(M);
    DBuf d_flag(this, (M + 7) / 8 + 1);
    DBuf d_pm(this, M);
    std::vector<u64> pm(M, 0);
    for (int t = 0; t < n_q; ++t) pm[t] = pmod[t];
    upload(this, d_pm.p, pm.data(), M * 8);
    for (int j = 0; j < beta; ++j) {
        u64* b = key->p + ((size_t)j * 2 + 0) * M * N;
        u64* a = key->p + ((size_t)j * 2 + 1) * M * N;
        std::vector<u64> uidx(M);
        for (int m = 0; m < M; ++m) uidx[m] = (key_id << 16) | ((u64)j << 8) | (u64)m;
        sample_into(a, M, all.data(), 2, P_SWK_A, 0, uidx.data());
        sample_into(e.p, M, all.data(), 1, P_SWK_E, (key_id << 8) | (u64)j, nullptr);
        ntt(a, 1, 0, M, false, -1);
        ntt(e.p, 1, 0, M, false, -1);
        for (int m = 0; m < M; ++m) flag[m] = (m < n_q && m / alpha == j) ? 1 : 0;
        upload(this, d_flag.p, flag.data(), M);
        launch_swk_finish(T, M, b, a, e.p, s_eval->p, sp, d_pm.p, (const uint8_t*)d_flag.p, stream);
        launch_to_key(T, ModMap{1 << 20, n_q}, M, 2, b, (int64_t)M * N, stream);
        hip_check(hipStreamSynchronize(stream), "swk");  // flag buffer reused
    }
    keys_bytes += (size_t)beta * 2 * M * N * 8;
    return key;
}

const u64* Ctx::relin_key() {
    if (!rlk) rlk = make_swk(0, s2_eval->p);
    return rlk->p;
}

u64 Ctx::galois(int64_t k) const {
    const int64_t half = N / 2;
    const int64_t kk = ((k % half) + half) % half;
    return powmod(5, (u64)kk, 2 * (u64)N);
}

const u64* Ctx::rot_key(u64 g, bool create) {
    auto it = rot_keys.find(g);
    if (it != rot_keys.end()) return it->second->p;
    if (!create) throw HeError(HE_EKEY);
    const int M = n_q + n_p;
    DBuf sp(this, (size_t)M * N);
    launch_automorph(T, M, 1, sp.p, 0, s_eval->p, 0, g, stream);
    auto key = make_swk(g, sp.p);
    const u64* p = key->p;
    rot_keys[g] = std::move(key);
    return p;
}

// ====================================================================== ciphertexts
CtPtr Ctx::new_ct(int level, int deg, double scale) {
    auto c = std::make_shared<CtData>();
    c->level = level;
    c->deg = deg;
    c->scale = scale;
    c->buf = std::make_unique<DBuf>(this, (size_t)(deg + 1) * (level + 1) * N);
    return c;
}

CtPtr Ctx::encrypt_coeffs(const int64_t* m_host, int level, double scale, u64 nonce) {
    if (level < 0 || level >= n_q) throw HeError(HE_ELEVEL);
    DBuf dm(this, N);
    upload(this, dm.p, m_host, N * 8);
    return encrypt_dev((const int64_t*)dm.p, level, scale, nonce);
}

// Enc of N device coefficients: v, e0 and e1 in one block, one sampling launch and one transform for the three
CtPtr Ctx::encrypt_dev(const int64_t* dev_coeffs, int level, double scale, u64 nonce) {
    if (level < 0 || level >= n_q) throw HeError(HE_ELEVEL);
    const int nl = level + 1;
    const size_t ps = (size_t)nl * N;
    DBuf x(this, 3 * ps);
    Jobs J;
    J.base = x.p;
    J.cstride = (int64_t)ps;
    J.nct = 3;
    J.n = nl;
    for (int i = 0; i < nl; ++i) {
        J.off[i] = (uint16_t)i;
        J.mod[i] = (uint8_t)i;
    }
    SampleArgs A;
    memset(&A, 0, sizeof A);
    A.seed = seed;
    A.poly[0] = {P_ENC_V, 0, nonce};
    A.poly[1] = {P_ENC_E0, 1, nonce};
    A.poly[2] = {P_ENC_E1, 1, nonce};
    memcpy(A.cdt, cdt, sizeof cdt);
    launch_sample(T, J, A, stream);
    launch_add_signed(T, nl, x.p + ps, dev_coeffs, stream);
    launch_ntt(T, J, false, stream);
    CtPtr c = new_ct(level, 1, scale);
    u64* c0 = c->buf->p;
    launch_enc_combine(T, nl, x.p, pk->p, pk->p + (size_t)n_q * N, x.p + ps, x.p + 2 * ps, c0, c0 + ps, stream);
    return c;
}

// Ecd of host values into N device coefficients, on the device where its fixed point holds them: finite
// values, a positive scale, results below 2^62, and memory for the transform; the 113-bit host encoder takes
// the rest
void Ctx::encode_into(const double* vals, int64_t n_vals, double sc, int64_t* dev_out) {
    double mx = 0;
    bool finite = true;
    for (int64_t j = 0; j < n_vals; ++j) {
        const double a = std::fabs(vals[j]);
        finite = finite && a <= 1.7976931348623157e308;  // false for NaN
        mx = a > mx ? a : mx;
    }
    int e = 0, es = 0;
    const double f = std::frexp(sc, &es);
    (void)std::frexp(mx, &e);
    std::unique_ptr<DBuf> z, x;
    const bool fixed = finite && sc >= 2.2250738585072014e-308 && sc <= 1.7976931348623157e308 && !(mx > 0 && e + es > 62);
    try {
        if (fixed) {
            z = std::make_unique<DBuf>(this, (size_t)n_vals);
            x = std::make_unique<DBuf>(this, (size_t)N * (sizeof(FixC) / 8));
        }
    } catch (const HeError& err) {
        if (err.s != HE_ENOMEM) throw;
    }
    if (!x) {
        std::vector<int64_t> m(N);
        enc.encode(vals, n_vals, sc, m.data());
        upload(this, dev_out, m.data(), N * 8);
        return;
    }
    if (mx == 0) e = 62 - es;  // any range will do
    upload(this, z->p, vals, n_vals * 8);
    EncArgs A;
    A.z = (const double*)z->p;
    A.vmask = (uint32_t)(n_vals - 1);
    A.shift = 125 - e;  // |values| 2^shift < 2^125, and every stage halves
    A.mant = (u64)std::ldexp(f, 53);
    A.sh = std::min(191, A.shift + 53 - es);  // 116 and up; at 191 every result rounds to 0
    launch_encode(E, A, (FixC*)x->p, dev_out, stream);
}

// device tables of the encoder and decoder
void Ctx::build_encoder() {
    const size_t n = (size_t)N;
    std::vector<i128> zr(n), zi(n);
    twist_fix(log_n, zr.data(), zi.data());
    std::vector<FixC> f(n + n / 2);  // w, then twist
    for (size_t i = 0; i < n; ++i) {
        const FixC z = {(u64)zr[i], (u64)((u128)zr[i] >> 64), (u64)zi[i], (u64)((u128)zi[i] >> 64)};
        f[n / 2 + i] = z;
        if (i % 2 == 0) f[i / 2] = z;
    }
    std::vector<uint32_t> slot(n), pos(n / 2);
    for (size_t j = 0; j < n / 2; ++j) {
        slot[enc.slot_pos[j]] = slot[enc.slot_neg[j]] = (uint32_t)j;
        pos[j] = bitrev((uint32_t)enc.slot_pos[j], log_n);
    }
    const size_t fw = f.size() * sizeof(FixC) / 8;
    d_enc = std::make_unique<DBuf>(this, fw + n / 2);
    upload(this, d_enc->p, f.data(), fw * 8);
    upload(this, d_enc->p + fw, slot.data(), n * 4);
    E.log_n = log_n;
    E.w = (const FixC*)d_enc->p;
    E.twist = E.w + n / 2;
    E.slot = (const uint32_t*)(d_enc->p + fw);
    static_assert(sizeof(std::complex<double>) == sizeof(DblC), "double tables");
    d_dec = std::make_unique<DBuf>(this, 3 * n + n / 4);
    upload(this, d_dec->p, enc.dw.data(), n * 8);
    upload(this, d_dec->p + n, enc.dz.data(), 2 * n * 8);
    upload(this, d_dec->p + 3 * n, pos.data(), n * 2);
    D.log_n = log_n;
    D.w = (const DblC*)d_dec->p;
    D.twist = (const DblC*)(d_dec->p + n);
    D.pos = (const uint32_t*)(d_dec->p + 3 * n);
}

// Dec: the N centred integers as doubles, and one word after them that is set when they do not fit q_0 q_1
std::unique_ptr<DBuf> Ctx::decrypt_lifted(const CtData& c) {
    const int nl = c.level + 1;
    DBuf m(this, (size_t)nl * N);
    launch_dec_dot(T, nl, c.deg, c.buf->p, (int64_t)nl * N, s_eval->p, s2_eval->p, m.p, stream);
    ntt(m.p, 1, 0, nl, true, -1);
    auto out = std::make_unique<DBuf>(this, (size_t)N + 1);
    launch_zero(out->p + N, 1, stream);
    const u64 q1 = nl > 1 ? mods[1] : 1;
    const u128h half = (u128h)mods[0] * q1 / 2;
    launch_lift_centred(T, nl, m.p, nl > 1 ? invmod(mods[0] % q1, q1) : 0, (u64)half, (u64)(half >> 64), (double*)out->p,
                        (uint32_t*)(out->p + N), stream);
    return out;
}

// The same on the host, with no more device memory than the residues take
void Ctx::decrypt_lifted_host(const CtData& c, double* out) {
    const int nl = c.level + 1;
    DBuf m(this, (size_t)nl * N);
    launch_dec_dot(T, nl, c.deg, c.buf->p, (int64_t)nl * N, s_eval->p, s2_eval->p, m.p, stream);
    ntt(m.p, 1, 0, nl, true, -1);
    std::vector<u64> h((size_t)nl * N);
    hip_check(hipMemcpyAsync(h.data(), m.p, h.size() * 8, hipMemcpyDeviceToHost, stream), "dec copy");
    hip_check(hipStreamSynchronize(stream), "dec sync");
    const u64 q0 = mods[0], q1 = nl > 1 ? mods[1] : 1, q0inv = nl > 1 ? invmod(q0 % q1, q1) : 0;
    const u128h Q = (u128h)q0 * q1;
    for (int64_t t = 0; t < N; ++t) {
        u128h w = h[t];
        if (nl > 1) w += (u128h)q0 * mulmod((h[N + t] + q1 - h[t] % q1) % q1, q0inv, q1);
        const __int128 v = w > Q / 2 ? (__int128)w - (__int128)Q : (__int128)w;
        for (int i = 2; i < nl; ++i) {
            const __int128 r = v % (__int128)mods[i];
            if ((u64)(r < 0 ? r + (__int128)mods[i] : r) != h[(size_t)i * N + t]) throw HeError(HE_ESCALE);
        }
        out[t] = (double)v;
    }
}

void Ctx::decrypt_coeffs(const CtData& c, double* out) {
    std::unique_ptr<DBuf> v;
    try {
        v = decrypt_lifted(c);
    } catch (const HeError& e) {
        if (e.s != HE_ENOMEM) throw;
        decrypt_lifted_host(c, out);
        return;
    }
    std::vector<double> h((size_t)N + 1);
    hip_check(hipMemcpyAsync(h.data(), v->p, h.size() * 8, hipMemcpyDeviceToHost, stream), "dec copy");
    hip_check(hipStreamSynchronize(stream), "dec sync");
    uint32_t bad;
    memcpy(&bad, &h[N], 4);
    if (bad) throw HeError(HE_ESCALE);
    std::copy(h.begin(), h.begin() + N, out);
}

// Dec + Dcd: the first n_out slot values (at most N / 2)
void Ctx::decrypt_values(const CtData& c, double* out, size_t n_out) {
    const size_t n = std::min(n_out, (size_t)N / 2);
    // the transform's buffer x [N] complex, then values [n] and the flag
    std::unique_ptr<DBuf> v, x, vals;
    try {
        v = decrypt_lifted(c);
        x = std::make_unique<DBuf>(this, 2 * (size_t)N);
        vals = std::make_unique<DBuf>(this, n + 1);
    } catch (const HeError& e) {  // does not fit: the residues alone may
        if (e.s != HE_ENOMEM) throw;
        v.reset();
        x.reset();
        std::vector<double> m((size_t)N);
        decrypt_lifted_host(c, m.data());
        enc.decode(m.data(), c.scale, out, (int64_t)n);
        return;
    }
    launch_decode(D, (const double*)v->p, c.scale, (DblC*)x->p, (int)n, (double*)vals->p, stream);
    hip_check(hipMemcpyAsync(vals->p + n, v->p + N, 8, hipMemcpyDeviceToDevice, stream), "dec flag");
    std::vector<double> h(n + 1);
    hip_check(hipMemcpyAsync(h.data(), vals->p, h.size() * 8, hipMemcpyDeviceToHost, stream), "dec copy");
    hip_check(hipStreamSynchronize(stream), "dec sync");
    uint32_t bad;
    memcpy(&bad, &h[n], 4);
    if (bad) throw HeError(HE_ESCALE);
    std::copy(h.begin(), h.begin() + n, out);
}

// Device to the caller's memory by way of pinned slots, all of the queue's copies issued before the first
// wait.  A copy straight to pageable memory takes the runtime's own staging, and the pages of a fresh
// array fault one by one while the device idles: they are populated here while the queued work runs.
// One ciphertext of two limbs at N = 2^15 (1 MB): 289 us into a fresh array straight, 151 so
// (N = 2^16: 389 and 230); slots of 256 KiB or 1 MiB take as long or longer.
void Ctx::read_back(void* dst, const void* src, size_t bytes) {
    char* d = (char*)dst;
    const char* s = (const char*)src;
    if (!stage && bytes > STAGE_SLOT / 8) {
        if (hipHostMalloc((void**)&stage, STAGE_SLOTS * STAGE_SLOT, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            stage = nullptr;
        }
        for (int i = 0; stage && i < STAGE_SLOTS; ++i)
            if (hipEventCreateWithFlags(&stage_ev[i], hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                free_stage();
            }
    }
    if (!stage || bytes <= STAGE_SLOT / 8) {
        hip_check(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, stream), "read back");
        hip_check(hipStreamSynchronize(stream), "read back sync");
        return;
    }
    struct Drain {  // an error path: nothing is left writing to the slots
        Ctx* c;
        bool busy = true;
        ~Drain() {
            if (busy) (void)hipStreamSynchronize(c->stream);
        }
    } drain{this};
    const size_t n = (bytes + STAGE_SLOT - 1) / STAGE_SLOT;
    auto len = [&](size_t i) { return std::min(STAGE_SLOT, bytes - i * STAGE_SLOT); };
    auto issue = [&](size_t i) {
        const int k = (int)(i % STAGE_SLOTS);
        hip_check(hipMemcpyAsync(stage + k * STAGE_SLOT, s + i * STAGE_SLOT, len(i), hipMemcpyDeviceToHost, stream),
                  "read back");
        hip_check(hipEventRecord(stage_ev[k], stream), "read back event");
    };
    for (size_t i = 0; i < std::min(n, (size_t)STAGE_SLOTS); ++i) issue(i);
    const uintptr_t page = 4096, p0 = ((uintptr_t)d + page - 1) / page * page, p1 = ((uintptr_t)d + bytes) / page * page;
#ifdef MADV_POPULATE_WRITE
    if (p1 > p0) (void)madvise((void*)p0, p1 - p0, MADV_POPULATE_WRITE);  // only earlier than the copy would
#endif
    for (size_t i = 0; i < n; ++i) {
        const int k = (int)(i % STAGE_SLOTS);
        hip_check(hipEventSynchronize(stage_ev[k]), "read back wait");
        memcpy(d + i * STAGE_SLOT, stage + k * STAGE_SLOT, len(i));
        if (i + STAGE_SLOTS < n) issue(i + STAGE_SLOTS);
    }
    drain.busy = false;
}

void Ctx::free_stage() {
    for (auto& e : stage_ev) {
        if (e) (void)hipEventDestroy(e);
        e = nullptr;
    }
    if (stage) (void)hipHostFree(stage);
    stage = nullptr;
}

CtPtr Ctx::drop(const CtData& a, int level) {
    if (level > a.level || level < 0) throw HeError(HE_ELEVEL);
    CtPtr r = new_ct(level, a.deg, a.scale);
    CopyDesc D;
    D.src[0] = a.buf->p;
    D.dst[0] = r->buf->p;
    D.width[0] = D.dpitch[0] = (int64_t)(level + 1) * N;
    D.spitch[0] = (int64_t)(a.level + 1) * N;
    D.rows[0] = a.deg + 1;
    D.n = 1;
    launch_copy(D, stream);
    return r;
}

CtPtr Ctx::add_sub(const CtData& a, const CtData& b, bool sub) {
    const int level = std::min(a.level, b.level);
    const int deg = std::max(a.deg, b.deg);
    CtPtr r = new_ct(level, deg, std::max(a.scale, b.scale));
    const int nl = level + 1;
    const int64_t ps = (int64_t)nl * N, pa = (int64_t)(a.level + 1) * N, pb = (int64_t)(b.level + 1) * N;
    const int common = std::min(a.deg, b.deg) + 1;
    launch_ew(T, qmap(this), nl, common, r->buf->p, ps, a.buf->p, pa, b.buf->p, pb, sub ? EW_SUB : EW_ADD, stream);
    for (int p = common; p <= deg; ++p) {
        const CtData& src = a.deg >= p ? a : b;
        const int64_t psrc = (int64_t)(src.level + 1) * N;
        if (a.deg >= p || !sub) {
            hip_check(hipMemcpyAsync(r->buf->p + p * ps, src.buf->p + p * psrc, (size_t)nl * N * 8,
                                     hipMemcpyDeviceToDevice, stream),
                      "add copy");
        } else {  // 0 - b_p
            hip_check(hipMemsetAsync(r->buf->p + p * ps, 0, (size_t)nl * N * 8, stream), "sub zero");
            launch_ew(T, qmap(this), nl, 1, r->buf->p + p * ps, 0, r->buf->p + p * ps, 0, src.buf->p + p * psrc, 0,
                      EW_SUB, stream);
        }
    }
    cnt[C_ADD]++;
    return r;
}

// (a0 b0, a0 b1 + a1 b0, a1 b1) at the lower level (Fig. 1 Mul_ct before relinearisation)
CtPtr Ctx::tensor(const CtData& a, const CtData& b) {
    if (a.deg != 1 || b.deg != 1) throw HeError(HE_EMISMATCH);
    const int level = std::min(a.level, b.level), nl = level + 1;
    CtPtr r = new_ct(level, 2, a.scale * b.scale);
    TensorSumDesc D;
    memset(&D, 0, sizeof D);
    D.a[0] = a.buf->p;
    D.a_ps[0] = (int64_t)(a.level + 1) * N;
    D.b[0] = b.buf->p;
    D.b_ps[0] = (int64_t)(b.level + 1) * N;
    D.d = r->buf->p;
    D.d_ps = (int64_t)nl * N;
    D.n = D.nct = 1;
    launch_tensor_each(T, nl, D, stream);
    cnt[C_MULCT]++;
    return r;
}

// ---------------------------------------------------------------- key switching
// out (two polynomials of nl limbs, out_ps apart) = ModDown(<digits of d permuted by g, key>) (+ sigma_g(c0) in
// out_0 for a rotation, + add [2][nl][N] for a relinearisation), on the caller's lift [beta][ne][N], u
// [2][ne][N] and tmp [2][nl][N]
void Ctx::ks_single_into(const u64* d, int level, const u64* key, u64 g, const u64* c0, const u64* add, u64* out,
                         int64_t out_ps, u64* lift, u64* u, u64* tmp) {
    const int64_t ps = (int64_t)(level + 1) * N;
    lift_into(d, 0, 1, level, lift, tmp);
    IpSet S;
    memset(&S, 0, sizeof S);
    S.key = key;
    S.g = g;
    ip_into(u, lift, d, 0, 1, level, {S}, 1, c0, 0, false);
    Epi E;
    memset(&E, 0, sizeof E);
    if (add) {
        E.add[0] = add;
        E.add[1] = add + ps;
    }
    E.out[0] = out;
    E.out[1] = out + out_ps;
    moddown_into(u, tmp, 1, level, E);
}

// the same with buffers of the context's allocation cache
void Ctx::ks_single(const u64* d, int level, const u64* key, u64 g, const u64* c0, const u64* add, u64* out) {
    const int nl = level + 1, ne = nl + n_p;
    DBuf lift(this, mu[level].size() * (size_t)ne * N), u(this, 2 * (size_t)ne * N), tmp(this, 2 * (size_t)nl * N);
    ks_single_into(d, level, key, g, c0, add, out, (int64_t)nl * N, lift.p, u.p, tmp.p);
}

CtPtr Ctx::relin(const CtData& a) {
    if (a.deg != 2) throw HeError(HE_EMISMATCH);
    const u64* key = relin_key();
    CtPtr r = new_ct(a.level, 1, a.scale);
    ks_single(a.buf->p + 2 * (int64_t)(a.level + 1) * N, a.level, key, 1, nullptr, a.buf->p, r->buf->p);
    return r;
}

CtPtr Ctx::rescale(const CtData& a) {
    if (a.level < 1) throw HeError(HE_ELEVEL);
    const int l = a.level;
    CtPtr r = new_ct(l - 1, a.deg, a.scale / (double)mods[l]);
    rescale_into(a.buf->p, (int64_t)(l + 1) * N, l, a.deg + 1, 1, r->buf->p, (int64_t)l * N);
    cnt[C_RS]++;
    return r;
}

CtPtr Ctx::rotate(const CtData& a, int64_t k) {
    if (a.deg != 1) throw HeError(HE_EMISMATCH);
    const u64 g = galois(k);
    if (g == 1) return drop(a, a.level);
    const u64* key = rot_key(g, false);
    CtPtr r = new_ct(a.level, 1, a.scale);
    ks_single(a.buf->p + (int64_t)(a.level + 1) * N, a.level, key, g, a.buf->p, nullptr, r->buf->p);
    cnt[C_ROT]++;
    return r;
}

CtPtr Ctx::mul_int(const CtData& a, int64_t k) {
    const int nl = a.level + 1;
    CtPtr r = new_ct(a.level, a.deg, a.scale);
    MulIntDesc D;
    D.a = a.buf->p;
    D.out = r->buf->p;
    D.ps = (int64_t)nl * N;
    D.a_cs = D.out_ks = 0;
    D.n = D.nct = 1;
    D.npoly = a.deg + 1;
    D.k[0] = k;
    launch_mul_ints(T, nl, D, stream);
    return r;
}

// plaintext (signed integer coefficients) to Montgomery evaluation form over all Q limbs
// a plaintext's residues on every modulus (Q and P, so that it can also multiply a value
// in the extended basis), evaluation form, Montgomery form: [M][N]
std::unique_ptr<DBuf> Ctx::plaintext_mont(const int64_t* coeffs) {
    DBuf dm(this, N);
    upload(this, dm.p, coeffs, N * 8);
    auto pt = plaintext_mont_dev((const int64_t*)dm.p);
    hip_check(hipStreamSynchronize(stream), "plaintext");
    return pt;
}

std::unique_ptr<DBuf> Ctx::plaintext_mont_dev(const int64_t* dev_coeffs) {
    const int M = n_q + n_p;
    auto pt = std::make_unique<DBuf>(this, (size_t)M * N);
    launch_zero(pt->p, (int64_t)M * N, stream);
    launch_add_signed(T, M, pt->p, dev_coeffs, stream);
    ntt(pt->p, 1, 0, M, false, -1);
    launch_to_mont(T, ModMap{1 << 20, n_q}, M, 1, pt->p, 0, stream);
    return pt;
}

// Alg. 6 aggregation: W - coeff sum_i G_i.  The n gradients are summed in one pass over HBM
// (16 inputs per launch), multiplied by the constant coeff = eta / (B N) encoded at the scale
// q_l of the prime the rescale removes (Mul_pt; the product returns exactly to the gradients'
// scale), rescaled, and subtracted from W dropped to the result's level.
CtPtr Ctx::fl_update(const CtData& w, const std::vector<const CtData*>& grads, double coeff) {
    if (grads.empty()) throw HeError(HE_EINVAL);
    int lvl = grads[0]->level;
    double sc = grads[0]->scale;
    for (auto* g : grads) {
        if (g->deg != 1) throw HeError(HE_EMISMATCH);
        lvl = std::min(lvl, g->level);
        sc = std::max(sc, g->scale);
    }
    if (lvl < 1 || w.deg != 1) throw HeError(lvl < 1 ? HE_ELEVEL : HE_EMISMATCH);
    const int nl = lvl + 1;
    CtPtr sum = new_ct(lvl, 1, sc);
    for (size_t base = 0; base < grads.size(); base += 16) {
        SumDesc D;
        memset(&D, 0, sizeof D);
        D.n = (int)std::min<size_t>(16, grads.size() - base);
        for (int t = 0; t < D.n; ++t) {
            D.in[t] = grads[base + t]->buf->p;
            D.in_ps[t] = (int64_t)(grads[base + t]->level + 1) * N;
        }
        launch_sum_many(T, nl, 2, D, sum->buf->p, (int64_t)nl * N, base > 0, stream);
    }
    cnt[C_ADD] += (int64_t)grads.size() - 1;
    const double ql = (double)mods[lvl];
    auto m = std::make_unique<DBuf>(this, N);
    encode_into(&coeff, 1, ql, (int64_t*)m->p);
    auto pt = plaintext_mont_dev((const int64_t*)m->p);
    m.reset();
    CtPtr t = mask_sum({{sum.get(), pt->p}}, ql);
    CtPtr u = rescale(*t);
    CtPtr wd = drop(w, std::min(u->level, w.level));
    return add_sub(*wd, *u, true);
}

// sum_r in_r * mask_r (Mul_pt terms of one diagonal sum, Alg. 2 / Eq. 1)
CtPtr Ctx::mask_sum(const std::vector<std::pair<const CtData*, const u64*>>& terms, double mask_scale) {
    const CtData& a0 = *terms[0].first;
    const int level = a0.level, nl = level + 1;
    CtPtr r = new_ct(level, 1, a0.scale * mask_scale);
    for (size_t base = 0; base < terms.size(); base += 16) {
        MacDesc D;
        memset(&D, 0, sizeof D);
        D.nct = 1;
        D.nterm = (int)std::min<size_t>(16, terms.size() - base);
        for (int t = 0; t < D.nterm; ++t) {
            const CtData* c = terms[base + t].first;
            if (c->level != level || c->deg != 1) throw HeError(HE_EMISMATCH);
            D.in[t] = c->buf->p;
            D.in_ps[t] = (int64_t)nl * N;
            D.mask[t] = terms[base + t].second;
        }
        launch_mask_mac(T, nl, 2, D, r->buf->p, (int64_t)nl * N, base > 0, stream);
    }
    cnt[C_MULPT] += (int64_t)terms.size();
    cnt[C_ADD] += (int64_t)terms.size() - 1;
    return r;
}

// ====================================================================== masks (Sec. 3.5-3.6, App. B)
static void mask_slots(int kind, int h, int k, std::vector<double>& out) {
    const int n = h * h;
    out.assign(n, 0.0);
    for (int t = 0; t < n; ++t) {
        bool v;
        switch (kind) {
            case 0:  // u^mu_k
                v = k >= 0 ? (t - h * k >= 0 && t - h * k < h - k) : (-k <= t - (h + k) * h && t - (h + k) * h < h);
                break;
            case 1: v = (t % h) == k; break;      // u^zeta_{h k}
            case 2: v = (t % h) < h - k; break;   // v_k (all ones for k = 0)
            case 3: v = (t % h) >= h - k; break;  // v_{k-h}
            default:  // App. C: diagonal (h-1) k of the transpose map (output h i + j reads h j + i)
                v = (t % h) - (t / h) == k;
                break;
        }
        out[t] = v ? 1.0 : 0.0;
    }
}

const u64* Ctx::mask(int kind, int h, int k, int64_t rot, int beta) {
    const MaskKey key{kind, h, beta, k, rot};
    auto it = masks.find(key);
    if (it != masks.end()) return it->second->p;
    prepare_masks({key});
    return masks.at(key)->p;
}

void Ctx::prepare_masks(const std::vector<MaskKey>& keys) {
    std::vector<MaskKey> todo;
    for (auto& k : keys)
        if (!masks.count(k) && std::find(todo.begin(), todo.end(), k) == todo.end()) todo.push_back(k);
    if (todo.empty()) return;
    std::vector<double> u, ur;
    DBuf coeffs(this, N);
    for (const MaskKey& m : todo) {
        mask_slots(m.kind, m.h, m.k, u);
        const int n = m.h * m.h;
        // R(u, rot), each entry repeated beta times (packing iota_beta: entry t of every
        // matrix sits at slots beta t .. beta t + beta - 1)
        ur.resize((size_t)n * m.beta);
        for (int t = 0; t < n; ++t)
            for (int e = 0; e < m.beta; ++e)
                ur[(size_t)m.beta * t + e] = u[(size_t)((((t + m.rot) % n) + n) % n)];
        encode_into(ur.data(), (int64_t)n * m.beta, scale, (int64_t*)coeffs.p);
        masks[m] = plaintext_mont_dev((const int64_t*)coeffs.p);
        keys_bytes += (size_t)(n_q + n_p) * N * 8;
    }
}

static int ilog2i(int h) {
    int l = 0;
    while ((1 << l) < h) ++l;
    return l;
}
static int floordiv(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }
int Ctx::bsgs(int h) const { return 1 << ((ilog2i(h) + 1) / 2); }
// baby steps bg of the Step-3 split k = bg i + j (2^ceil((log2 h + 1) / 2), at most h); one
// block of h terms without the flag
int Ctx::step3_baby(int h) const {
    if (!(schedule & HE_SCHED_STEP3_BSGS)) return h;
    return std::min(h, 1 << ((ilog2i(h) + 2) / 2));
}

// masks of HE-LinTrans with BSGS over diagonals [dlo, dhi] at unit u: R(mask_d, -u b floor(d/b))
static void lintrans_masks(std::vector<MaskKey>& out, int kind, int h, int beta, int64_t unit, int dlo, int dhi,
                           int b) {
    for (int d = dlo; d <= dhi; ++d) out.push_back({kind, h, beta, d, -unit * b * floordiv(d, b)});
}
// rotation amounts of the same: baby steps u j, giant steps u b i (i != 0)
static void lintrans_rotations(std::vector<int64_t>& r, int b, int64_t unit, int dlo, int dhi) {
    for (int j = 1; j < b; ++j) r.push_back(unit * j);
    for (int i = floordiv(dlo, b); i <= floordiv(dhi, b); ++i)
        if (i) r.push_back(unit * b * i);
}

void Ctx::check_shape(const MatShape& s) const {
    const auto pow2 = [](int x) { return x >= 1 && !(x & (x - 1)); };
    if (!pow2(s.h) || !pow2(s.t) || s.t > s.h || !pow2(s.beta) || (int64_t)s.beta * s.h * s.h > N / 2)
        throw HeError(HE_ESHAPE);
}

std::vector<MaskKey> Ctx::matmul_masks(const MatShape& s) const {
    std::vector<MaskKey> out;
    const int h = s.h, b = bsgs(h), bg = step3_baby(s.t);
    lintrans_masks(out, 0, h, s.beta, 1, 1 - h, h - 1, b);
    lintrans_masks(out, 1, h, s.beta, h, 0, h - 1, b);
    out.push_back({2, h, s.beta, 0, 0});
    for (int k = 1; k < s.t; ++k) {
        const int64_t shift = (int64_t)h * bg * (k / bg);
        out.push_back({2, h, s.beta, k, -shift});
        out.push_back({3, h, s.beta, k, -shift});
    }
    return out;
}

// amounts before the packing factor; every amount is multiplied by beta
std::vector<int64_t> Ctx::matmul_rotations(const MatShape& s) const {
    const int h = s.h, t = s.t, b = bsgs(h), bg = step3_baby(t);
    std::vector<int64_t> r;
    lintrans_rotations(r, b, 1, 1 - h, h - 1);
    lintrans_rotations(r, b, h, 0, h - 1);
    for (int k = 1; k < t; ++k) {
        const int64_t shift = (int64_t)h * bg * (k / bg);
        r.push_back(k - shift);
        r.push_back(k - h - shift);
    }
    for (int j = 1; j < bg; ++j) r.push_back((int64_t)h * j);
    for (int i = 1; i * bg < t; ++i) r.push_back((int64_t)h * bg * i);
    for (int sh = 0; (t << sh) < h; ++sh) r.push_back(((int64_t)t * h) << sh);
    for (auto& v : r) v *= s.beta;
    return r;
}

std::vector<MaskKey> Ctx::transpose_masks(int h, int beta) const {
    std::vector<MaskKey> out;
    lintrans_masks(out, 4, h, beta, h - 1, 1 - h, h - 1, bsgs(h));
    return out;
}

std::vector<int64_t> Ctx::transpose_rotations(int h, int beta) const {
    std::vector<int64_t> r;
    lintrans_rotations(r, bsgs(h), h - 1, 1 - h, h - 1);
    for (auto& v : r) v *= beta;
    return r;
}

void Ctx::prepare_shape(const MatShape& s) {
    check_shape(s);
    if (prepared.count(s)) return;
    for (int64_t k : matmul_rotations(s)) rot_key(galois(k), true);
    prepare_masks(matmul_masks(s));
    hip_check(hipStreamSynchronize(stream), "prepare_shape");
    prepared.insert(s);
    if (s.t == s.h && s.beta == 1) {
        int lg = 0;
        while ((1 << lg) < s.h) ++lg;
        prepared_mask.fetch_or(1u << lg);
    }
}

void Ctx::prepare_transpose(int h, int beta) {
    check_shape(MatShape{h, h, beta});
    if (prepared_tr.count({h, beta})) return;
    for (int64_t k : transpose_rotations(h, beta)) rot_key(galois(k), true);
    prepare_masks(transpose_masks(h, beta));
    hip_check(hipStreamSynchronize(stream), "prepare_transpose");
    prepared_tr.insert({h, beta});
}

// ====================================================================== C ABI


template <class F>
static he_status guard(F&& f);
template <class F>
static he_status guardc(he_ctx* ctx, F&& f) {
    std::lock_guard<std::recursive_mutex> lk(ctx->c->api_mu);
    return guard(std::forward<F>(f));
}
template <class F>
static he_status guard(F&& f) {
    try {
        f();
        return HE_OK;
    } catch (const HeError& e) {
        return e.s;
    } catch (const LaunchError&) {
        return HE_EDEVICE;
    } catch (const std::bad_alloc&) {
        return HE_ENOMEM;
    } catch (...) {
        return HE_EDEVICE;
    }
}

he_ct* wrap(Ctx* c, CtPtr p) { return new he_ct{c, std::move(p)}; }

extern "C" {

// iota_beta (App. E): entry e of matrix m at position beta e + m
he_status he_pack_beta(size_t beta, size_t n, const double* const* mats, double* out) {
    if (!mats || !out || beta == 0 || n == 0) return HE_EINVAL;
    for (size_t m = 0; m < beta; ++m)
        if (!mats[m]) return HE_EINVAL;
    for (size_t e = 0; e < n; ++e)
        for (size_t m = 0; m < beta; ++m) out[beta * e + m] = mats[m][e];
    return HE_OK;
}

// ====================================================================== allocation-free rotation
// Scratch of he_rotate_noalloc: file-scope device memory, one copy on every device the library
// runs on, held until the process ends.  Host code never passes the array's name to a kernel or
// a copy (on the host it only names the symbol); it uses the device address taken once per
// device by hipGetSymbolAddress with that device current.
#define HE_SCRATCH_BYTES (64ull << 20)
#define HE_MAX_DEVICES 64
static __device__ __align__(256) u64 scratch[HE_SCRATCH_BYTES / 8];
static std::mutex g_scratch_mu;
static u64* g_scratch_dev[HE_MAX_DEVICES];

// the current device's scratch address (taken on the first call for that device)
static u64* scratch_of_current_device(int* dev_out) {
    int dev = 0;
    hip_check(hipGetDevice(&dev), "scratch device");
    if (dev < 0 || dev >= HE_MAX_DEVICES) throw HeError(HE_EUNSUPPORTED);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "scratch address");
        g_scratch_dev[dev] = (u64*)p;
    }
    *dev_out = dev;
    return g_scratch_dev[dev];
}

he_status he_ctx_create(const he_params* prm, const he_device* dev, he_ctx** out) {
    if (!prm || !out || !prm->q_bits || (prm->n_p && !prm->p_bits)) return HE_EINVAL;
    return guard([&]() {
        if (prm->log_n < 8 || prm->log_n > 17 || prm->n_q < 1 || prm->n_p < 1 || prm->alpha < 1 ||
            prm->n_q + prm->n_p > HE_MAXT || prm->alpha > HE_MAXSRC || prm->n_p > HE_MAXSRC ||
            (prm->n_q + prm->alpha - 1) / prm->alpha > HE_MAXSRC || (prm->schedule & ~HE_SCHED_ALL))
            throw HeError(HE_EINVAL);
        auto c = std::make_unique<Ctx>();
        c->scratch = scratch_of_current_device(&c->device);
        c->log_n = (int)prm->log_n;
        c->N = (int64_t)1 << prm->log_n;
        c->n_q = (int)prm->n_q;
        c->n_p = (int)prm->n_p;
        c->alpha = (int)prm->alpha;
        c->scale = std::pow(2.0, prm->log_scale);
        c->seed = prm->seed;
        c->schedule = prm->schedule;
        if (dev) {
            c->pool.dev_alloc = c->pool_side.dev_alloc = dev->alloc;
            c->pool.dev_free = c->pool_side.dev_free = dev->free;
            c->pool.user = c->pool_side.user = dev->user;
        }
        if (dev && dev->stream) {
            c->stream = (hipStream_t)dev->stream;
        } else {
            hip_check(hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking), "stream");
            c->own_stream = true;
        }
        c->home = c->stream;
        c->pool.sibling = &c->pool_side;
        c->pool_side.sibling = &c->pool;
        c->pool.owner = c->pool_side.owner = c.get();

        std::vector<uint32_t> qb(prm->q_bits, prm->q_bits + prm->n_q), pb(prm->p_bits, prm->p_bits + prm->n_p);
        gen_primes(c->log_n, qb, c->mods);
        gen_primes(c->log_n, pb, c->mods);
        // the REDC accumulations need (terms) * q < 2^64
        for (u64 q : c->mods)
            if (q >= (1ull << 60) + 1) throw HeError(HE_EINVAL);
        c->enc.init(c->log_n);
        c->build_tables();
        c->build_encoder();
        c->keygen_base();
        c->relin_key();
        for (uint32_t i = 0; i < prm->n_h; ++i) c->prepare_h((int)prm->h_list[i]);
        hip_check(hipStreamSynchronize(c->stream), "create");
        *out = new he_ctx{std::move(c)};
    });
}

void he_ctx_destroy(he_ctx* ctx) {
    if (!ctx) return;
    try {
        (void)hipStreamSynchronize(ctx->c->stream);
        if (ctx->c->side) (void)hipStreamSynchronize(ctx->c->side);
        ctx->c->release_all();
        if (ctx->c->own_stream) (void)hipStreamDestroy(ctx->c->stream);
    } catch (...) {
    }
    delete ctx;
}

he_status he_ctx_moduli(const he_ctx* ctx, uint64_t* out, size_t n) {
    if (!ctx || !out || n < ctx->c->mods.size()) return HE_EINVAL;
    std::copy(ctx->c->mods.begin(), ctx->c->mods.end(), out);
    return HE_OK;
}

he_status he_sync(he_ctx* ctx) {
    if (!ctx) return HE_EINVAL;
    return guardc(ctx, [&]() { hip_check(hipStreamSynchronize(ctx->c->stream), "sync"); });
}

he_status he_counters(const he_ctx* ctx, int64_t out[6], int reset) {
    if (!ctx || !out) return HE_EINVAL;
    for (int i = 0; i < 6; ++i) out[i] = ctx->c->cnt[i];
    if (reset)
        for (int i = 0; i < 6; ++i) const_cast<Ctx*>(ctx->c.get())->cnt[i] = 0;
    return HE_OK;
}

he_status he_memory(const he_ctx* ctx, uint64_t* keys_bytes, uint64_t* pool_bytes) {
    if (!ctx) return HE_EINVAL;
    if (keys_bytes) *keys_bytes = ctx->c->keys_bytes;
    if (pool_bytes) *pool_bytes = ctx->c->pool.held + ctx->c->pool_side.held;
    return HE_OK;
}

he_status he_pool_limit(he_ctx* ctx, uint64_t bytes) {
    if (!ctx) return HE_EINVAL;
    return guardc(ctx, [&]() {
        // cached blocks above the new cap go back to the device once queued work is done
        hip_check(hipStreamSynchronize(ctx->c->stream), "pool limit");
        Pool& P = ctx->c->pool;
        std::lock_guard<std::mutex> lk(P.m);
        P.limit = bytes;
        if (bytes && P.held > bytes) P.trim_locked();
        if (bytes) ctx->c->pool_side.trim();
    });
}
he_status he_pool_stats(he_ctx* ctx, uint64_t* in_use, uint64_t* peak, int reset) {
    if (!ctx) return HE_EINVAL;
    Pool& P = ctx->c->pool;
    std::lock_guard<std::mutex> lk(P.m);
    if (in_use) *in_use = P.held - P.cached;
    if (peak) *peak = P.peak;
    if (reset) P.peak = P.held - P.cached;
    return HE_OK;
}

he_status he_encode(he_ctx* ctx, const double* vals, size_t n_vals, double scale, int64_t* out) {
    if (!ctx || !vals || !out || n_vals == 0 || (size_t)(ctx->c->N / 2) % n_vals) return HE_EINVAL;
    return guardc(ctx, [&]() {
        Ctx* c = ctx->c.get();
        std::unique_ptr<DBuf> m;
        try {
            m = std::make_unique<DBuf>(c, c->N);
        } catch (const HeError& e) {  // no device memory at all: on the host
            if (e.s != HE_ENOMEM) throw;
            c->enc.encode(vals, (int64_t)n_vals, scale, out);
            return;
        }
        c->encode_into(vals, (int64_t)n_vals, scale, (int64_t*)m->p);
        hip_check(hipMemcpyAsync(out, m->p, c->N * 8, hipMemcpyDeviceToHost, c->stream), "encode d2h");
        hip_check(hipStreamSynchronize(c->stream), "encode sync");
    });
}

he_status he_encrypt(he_ctx* ctx, const double* vals, size_t n_vals, uint32_t level, uint64_t nonce, he_ct** out) {
    if (!ctx || !vals || !out || n_vals == 0 || (size_t)(ctx->c->N / 2) % n_vals) return HE_EINVAL;
    return guardc(ctx, [&]() {
        Ctx* c = ctx->c.get();
        if ((int)level >= c->n_q || (int)level < 0) throw HeError(HE_ELEVEL);
        DBuf m(c, c->N);
        c->encode_into(vals, (int64_t)n_vals, c->scale, (int64_t*)m.p);
        *out = wrap(c, c->encrypt_dev((const int64_t*)m.p, (int)level, c->scale, nonce));
    });
}

he_status he_encrypt_coeffs(he_ctx* ctx, const int64_t* coeffs, uint32_t level, double scale, uint64_t nonce,
                            he_ct** out) {
    if (!ctx || !coeffs || !out) return HE_EINVAL;
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->encrypt_coeffs(coeffs, (int)level, scale, nonce)); });
}

he_status he_decrypt_coeffs(he_ctx* ctx, const he_ct* ct, double* out, size_t n) {
    if (!ctx || !ct || !out || n < (size_t)ctx->c->N) return HE_EINVAL;
    if (ct->ctx != ctx->c.get()) return HE_EMISMATCH;
    return guardc(ctx, [&]() { ctx->c->decrypt_coeffs(*ct->c, out); });
}

he_status he_decrypt(he_ctx* ctx, const he_ct* ct, double* out, size_t n_out) {
    if (!ctx || !ct || !out) return HE_EINVAL;
    if (ct->ctx != ctx->c.get()) return HE_EMISMATCH;
    return guardc(ctx, [&]() { ctx->c->decrypt_values(*ct->c, out, n_out); });
}

void he_ct_free(he_ct* ct) {
    if (!ct) return;
    std::lock_guard<std::recursive_mutex> lk(ct->ctx->api_mu);
    delete ct;
}

he_status he_ct_info(const he_ct* ct, uint32_t* level, uint32_t* degree, double* scale) {
    if (!ct) return HE_EINVAL;
    if (level) *level = (uint32_t)ct->c->level;
    if (degree) *degree = (uint32_t)ct->c->deg;
    if (scale) *scale = ct->c->scale;
    return HE_OK;
}

he_status he_ct_export(he_ctx* ctx, const he_ct* ct, uint64_t* buf, size_t n) {
    if (!ctx || !ct || !buf) return HE_EINVAL;
    if (ct->ctx != ctx->c.get()) return HE_EMISMATCH;
    Ctx* c = ctx->c.get();
    const CtData& d = *ct->c;
    const size_t tot = (size_t)(d.deg + 1) * (d.level + 1) * c->N;
    if (n < tot) return HE_EINVAL;
    return guardc(ctx, [&]() {
        DBuf tmp(c, tot);
        c->ntt(tmp.p, d.deg + 1, d.level + 1, d.level + 1, true, -1, d.buf->p);
        c->read_back(buf, tmp.p, tot * 8);
    });
}

he_status he_ct_import(he_ctx* ctx, const uint64_t* buf, size_t n, uint32_t level, uint32_t degree, double scale,
                       he_ct** out) {
    if (!ctx || !buf || !out || degree < 1 || degree > 2) return HE_EINVAL;
    Ctx* c = ctx->c.get();
    if ((int)level >= c->n_q) return HE_ELEVEL;
    const size_t tot = (size_t)(degree + 1) * (level + 1) * c->N;
    if (n < tot) return HE_EINVAL;
    // every residue of limb i must lie in [0, q_i): the transform takes canonical words (its
    // FP64 butterflies convert a word exactly only below 2^52), so a corrupt or foreign
    // checkpoint is refused here instead of becoming a silently wrong ciphertext
    for (size_t p = 0; p <= degree; ++p)
        for (size_t i = 0; i <= level; ++i) {
            const uint64_t q = c->mods[i];
            const uint64_t* w = buf + (p * (level + 1) + i) * c->N;
            uint64_t over = 0;  // no early exit: the loop runs as vector code
            for (int64_t t = 0; t < c->N; ++t) over |= (uint64_t)(w[t] >= q);
            if (over) return HE_EINVAL;
        }
    return guardc(ctx, [&]() {
        CtPtr r = c->new_ct((int)level, (int)degree, scale);
        upload(c, r->buf->p, buf, tot * 8);
        c->ntt(r->buf->p, degree + 1, level + 1, level + 1, false, -1);
        hip_check(hipStreamSynchronize(c->stream), "import");
        *out = wrap(c, r);
    });
}

#define CHECK2(a, b)                                                  \
    if (!ctx || !(a) || !(b) || !out) return HE_EINVAL;               \
    if ((a)->ctx != ctx->c.get() || (b)->ctx != ctx->c.get()) return HE_EMISMATCH;
#define CHECK1(a)                               \
    if (!ctx || !(a) || !out) return HE_EINVAL; \
    if ((a)->ctx != ctx->c.get()) return HE_EMISMATCH;

he_status he_add(he_ctx* ctx, const he_ct* a, const he_ct* b, he_ct** out) {
    CHECK2(a, b);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->add_sub(*a->c, *b->c, false)); });
}
he_status he_sub(he_ctx* ctx, const he_ct* a, const he_ct* b, he_ct** out) {
    CHECK2(a, b);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->add_sub(*a->c, *b->c, true)); });
}
he_status he_drop(he_ctx* ctx, const he_ct* a, uint32_t level, he_ct** out) {
    CHECK1(a);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->drop(*a->c, (int)level)); });
}
he_status he_mul_plain(he_ctx* ctx, const he_ct* a, const int64_t* coeffs, double pt_scale, he_ct** out) {
    CHECK1(a);
    if (!coeffs) return HE_EINVAL;
    return guardc(ctx, [&]() {
        Ctx* c = ctx->c.get();
        auto pt = c->plaintext_mont(coeffs);
        if (a->c->deg != 1) throw HeError(HE_EMISMATCH);
        CtPtr r = c->mask_sum({{a->c.get(), pt->p}}, pt_scale);
        hip_check(hipStreamSynchronize(c->stream), "mul_plain");
        *out = wrap(c, r);
    });
}
he_status he_mul_int(he_ctx* ctx, const he_ct* a, int64_t k, he_ct** out) {
    CHECK1(a);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->mul_int(*a->c, k)); });
}
he_status he_tensor(he_ctx* ctx, const he_ct* a, const he_ct* b, he_ct** out) {
    CHECK2(a, b);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->tensor(*a->c, *b->c)); });
}
he_status he_relin(he_ctx* ctx, const he_ct* a, he_ct** out) {
    CHECK1(a);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->relin(*a->c)); });
}
he_status he_mul(he_ctx* ctx, const he_ct* a, const he_ct* b, he_ct** out) {
    CHECK2(a, b);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->relin(*ctx->c->tensor(*a->c, *b->c))); });
}
he_status he_rescale(he_ctx* ctx, const he_ct* a, he_ct** out) {
    CHECK1(a);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->rescale(*a->c)); });
}
he_status he_rotate(he_ctx* ctx, const he_ct* a, int64_t k, he_ct** out) {
    CHECK1(a);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->rotate(*a->c, k)); });
}

// Rot(a, k) with every temporary in the static scratch: the digit lift [beta][ne][N], the
// inner product over Q_l and P [2][ne][N], and one region shared by the digits' coefficient
// form (used while lifting) and the converted P part (used by ModDown afterwards) [2][nl][N].
// Every scratch word a call reads was written earlier in that call, so nothing is cleared.
he_status he_rotate_noalloc(he_ctx* ctx, const uint64_t* in, uint32_t level, int64_t k, uint64_t* out) {
    if (!ctx || !in || !out) return HE_EINVAL;
    Ctx* c = ctx->c.get();
    if ((int)level >= c->n_q) return HE_ELEVEL;
    const int nl = (int)level + 1, ne = nl + c->n_p;
    const int64_t N = c->N;
    const size_t ct_words = 2 * (size_t)nl * N;
    if (in < out + ct_words && out < in + ct_words) return HE_EINVAL;  // in and out overlap
    const int beta = (int)c->mu[level].size();
    const size_t lift_w = (size_t)beta * ne * N, u_w = 2 * (size_t)ne * N, tmp_w = 2 * (size_t)nl * N;
    if ((lift_w + u_w + tmp_w) * 8 > HE_SCRATCH_BYTES) {
        fprintf(stderr, "libhe: he_rotate_noalloc needs %zu scratch bytes at level %u, more than the %llu it has\n",
                (lift_w + u_w + tmp_w) * 8, level, HE_SCRATCH_BYTES);
        return HE_ENOMEM;
    }
    return guardc(ctx, [&]() {
        int dev = 0;
        hip_check(hipGetDevice(&dev), "device");
        if (dev != c->device) throw HeError(HE_EMISMATCH);  // the scratch address is per device
        const u64 g = c->galois(k);
        if (g == 1) {
            hip_check(hipMemcpyAsync(out, in, ct_words * 8, hipMemcpyDeviceToDevice, c->stream), "rotate copy");
            return;
        }
        const u64* key = c->rot_key(g, false);
        u64 *lift = c->scratch, *u = lift + lift_w, *tmp = u + u_w;
        // the row pass stores 16 bytes a lane: a result at an odd multiple of 8 bytes is made in place of
        // the Q limbs of u (every lane reads its words of u before it writes them) and copied word by word
        const bool odd = ((uintptr_t)out & 15) != 0;
        c->ks_single_into(in + (size_t)nl * N, (int)level, key, g, in, nullptr, odd ? u : out,
                          odd ? (int64_t)ne * N : (int64_t)nl * N, lift, u, tmp);
        if (odd) launch_automorph(c->T, nl, 2, out, (int64_t)nl * N, u, (int64_t)ne * N, 1, c->stream);
        c->cnt[C_ROT]++;
    });
}
he_status he_gen_rotation_key(he_ctx* ctx, int64_t k) {
    if (!ctx) return HE_EINVAL;
    return guardc(ctx, [&]() {
        ctx->c->rot_key(ctx->c->galois(k), true);
        hip_check(hipStreamSynchronize(ctx->c->stream), "genkey");
    });
}
he_status he_matmul(he_ctx* ctx, const he_ct* a, const he_ct* b, uint32_t h, he_ct** out) {
    CHECK2(a, b);
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->matmul(*a->c, *b->c, (int)h)); });
}
he_status he_matmul_batch(he_ctx* ctx, size_t n, const he_ct* const* a, const he_ct* const* b, const uint32_t* h,
                          he_ct** out) {
    if (!ctx || (n && (!a || !b || !h || !out))) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!a[i] || !b[i]) return HE_EINVAL;
        if (a[i]->ctx != ctx->c.get() || b[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        std::vector<const CtData*> va(n), vb(n);
        std::vector<int> vh(n);
        for (size_t i = 0; i < n; ++i) {
            va[i] = a[i]->c.get();
            vb[i] = b[i]->c.get();
            vh[i] = (int)h[i];
        }
        std::vector<MatShape> sh(n);
        for (size_t i = 0; i < n; ++i) sh[i] = MatShape{vh[i], vh[i], 1};
        auto res = ctx->c->matmul_batch(va, vb, sh);
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), res[i]);
    });
}
he_status he_matmul_ex(he_ctx* ctx, const he_ct* a, const he_ct* b, const he_mat_shape* shape, he_ct** out) {
    return he_matmul_batch_ex(ctx, 1, &a, &b, shape, out);
}
he_status he_matmul_batch_ex(he_ctx* ctx, size_t n, const he_ct* const* a, const he_ct* const* b,
                             const he_mat_shape* shapes, he_ct** out) {
    if (!ctx || (n && (!a || !b || !shapes || !out))) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!a[i] || !b[i]) return HE_EINVAL;
        if (a[i]->ctx != ctx->c.get() || b[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        std::vector<const CtData*> va(n), vb(n);
        std::vector<MatShape> sh(n);
        for (size_t i = 0; i < n; ++i) {
            va[i] = a[i]->c.get();
            vb[i] = b[i]->c.get();
            sh[i] = MatShape{(int)shapes[i].h, (int)shapes[i].t, (int)shapes[i].beta};
        }
        auto res = ctx->c->matmul_batch(va, vb, sh);
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), res[i]);
    });
}
he_status he_transpose(he_ctx* ctx, const he_ct* a, uint32_t h, uint32_t beta, he_ct** out) {
    return he_transpose_batch(ctx, 1, &a, h, beta, out);
}
he_status he_transpose_batch(he_ctx* ctx, size_t n, const he_ct* const* a, uint32_t h, uint32_t beta,
                             he_ct** out) {
    if (!ctx || (n && (!a || !out))) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!a[i]) return HE_EINVAL;
        if (a[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        std::vector<const CtData*> va(n);
        for (size_t i = 0; i < n; ++i) va[i] = a[i]->c.get();
        auto res = ctx->c->transpose_batch(va, (int)h, (int)beta);
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), res[i]);
    });
}
he_status he_sign_approx(he_ctx* ctx, const he_ct* x, uint32_t d, uint32_t k, uint32_t mode, he_ct** out) {
    CHECK1(x);
    if (mode > 1) return HE_EINVAL;
    return guardc(ctx, [&]() { *out = wrap(ctx->c.get(), ctx->c->sign_group({x->c.get()}, (int)d, (int)k, (int)mode)[0]); });
}
he_status he_sign_approx_batch(he_ctx* ctx, size_t n, const he_ct* const* x, uint32_t d, uint32_t k, uint32_t mode,
                               he_ct** out) {
    if (!ctx || (n && (!x || !out)) || mode > 1) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!x[i]) return HE_EINVAL;
        if (x[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        // lockstep groups of equal level
        std::map<int, std::vector<size_t>> byl;
        for (size_t i = 0; i < n; ++i) byl[x[i]->c->level].push_back(i);
        std::vector<CtPtr> res(n);
        for (auto& kv : byl) {
            for (size_t s = 0; s < kv.second.size(); s += (size_t)ctx->c->max_group) {
                std::vector<const CtData*> v;
                const size_t e = std::min(kv.second.size(), s + (size_t)ctx->c->max_group);
                for (size_t t = s; t < e; ++t) v.push_back(x[kv.second[t]]->c.get());
                auto r = ctx->c->sign_group(v, (int)d, (int)k, (int)mode);
                for (size_t t = s; t < e; ++t) res[kv.second[t]] = r[t - s];
            }
        }
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), res[i]);
    });
}
he_status he_appmax(he_ctx* ctx, const he_ct* a, const he_ct* b, uint32_t d, uint32_t k, he_ct** out) {
    return he_appmax_batch(ctx, 1, &a, &b, d, k, out);
}
he_status he_appmax_batch(he_ctx* ctx, size_t n, const he_ct* const* a, const he_ct* const* b, uint32_t d,
                          uint32_t k, he_ct** out) {
    if (!ctx || (n && (!a || !b || !out))) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!a[i] || !b[i]) return HE_EINVAL;
        if (a[i]->ctx != ctx->c.get() || b[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        // lockstep groups of equal operand levels
        std::map<std::pair<int, int>, std::vector<size_t>> byl;
        for (size_t i = 0; i < n; ++i) byl[{a[i]->c->level, b[i]->c->level}].push_back(i);
        std::vector<CtPtr> res(n);
        for (auto& kv : byl) {
            for (size_t s = 0; s < kv.second.size(); s += (size_t)ctx->c->max_group) {
                std::vector<const CtData*> va, vb;
                const size_t e = std::min(kv.second.size(), s + (size_t)ctx->c->max_group);
                for (size_t t = s; t < e; ++t) {
                    va.push_back(a[kv.second[t]]->c.get());
                    vb.push_back(b[kv.second[t]]->c.get());
                }
                auto r = ctx->c->sign_group(va, (int)d, (int)k, 2, vb);
                for (size_t t = s; t < e; ++t) res[kv.second[t]] = r[t - s];
            }
        }
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), res[i]);
    });
}
he_status he_maxpool2(he_ctx* ctx, const he_ct* x, uint32_t h, uint32_t d, uint32_t k, he_ct** out) {
    return he_maxpool2_batch(ctx, 1, &x, h, d, k, out);
}
he_status he_maxpool2_batch(he_ctx* ctx, size_t n, const he_ct* const* x, uint32_t h, uint32_t d, uint32_t k,
                            he_ct** out) {
    if (!ctx || (n && (!x || !out))) return HE_EINVAL;
    for (size_t i = 0; i < n; ++i) {
        if (!x[i]) return HE_EINVAL;
        if (x[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        std::vector<const CtData*> v(n);
        for (size_t i = 0; i < n; ++i) v[i] = x[i]->c.get();
        auto r = ctx->c->maxpool_batch(v, (int)h, (int)d, (int)k);
        for (size_t i = 0; i < n; ++i) out[i] = wrap(ctx->c.get(), r[i]);
    });
}
he_status he_fl_update(he_ctx* ctx, const he_ct* w, size_t n, const he_ct* const* grads, double coeff, he_ct** out) {
    if (!ctx || !w || !out || n == 0 || !grads) return HE_EINVAL;
    if (w->ctx != ctx->c.get()) return HE_EMISMATCH;
    for (size_t i = 0; i < n; ++i) {
        if (!grads[i]) return HE_EINVAL;
        if (grads[i]->ctx != ctx->c.get()) return HE_EMISMATCH;
    }
    return guardc(ctx, [&]() {
        std::vector<const CtData*> g(n);
        for (size_t i = 0; i < n; ++i) g[i] = grads[i]->c.get();
        *out = wrap(ctx->c.get(), ctx->c->fl_update(*w->c, g, coeff));
    });
}
he_status he_profile_enable(he_ctx* ctx, int on, const char* only) {
    if (!ctx) return HE_EINVAL;
    return prof_enable(on != 0, only) ? HE_OK : HE_EINVAL;
}
he_status he_debug_fail_launch(uint64_t n) {
    launch_inject(n);
    return HE_OK;
}
he_status he_profile_report(he_ctx* ctx, char* buf, size_t n) {
    if (!ctx || !buf || n == 0) return HE_EINVAL;
    return guardc(ctx, [&]() {
        const std::string r = prof_report();
        const size_t m = std::min(n - 1, r.size());
        memcpy(buf, r.data(), m);
        buf[m] = 0;
    });
}
he_status he_ntt(he_ctx* ctx, uint64_t* dev_ptr, uint32_t n_limbs, const uint32_t* mod_idx, int inverse) {
    if (!ctx || !dev_ptr || !mod_idx || n_limbs == 0) return HE_EINVAL;
    Ctx* c = ctx->c.get();
    for (uint32_t i = 0; i < n_limbs; ++i)
        if (mod_idx[i] >= c->mods.size()) return HE_EINVAL;
    return guardc(ctx, [&]() {
        for (uint32_t start = 0; start < n_limbs; start += HE_MAXJ) {
            Jobs J;
            J.base = dev_ptr + (size_t)start * c->N;
            J.cstride = 0;
            J.nct = 1;
            J.n = (int)std::min<uint32_t>(HE_MAXJ, n_limbs - start);
            for (int k = 0; k < J.n; ++k) {
                J.off[k] = (uint16_t)k;
                J.mod[k] = (uint8_t)mod_idx[start + k];
            }
            launch_ntt(c->T, J, inverse != 0, c->stream);
        }
        hip_check(hipGetLastError(), "ntt launch");
    });
}

}  // extern "C"

