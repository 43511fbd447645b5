// Device code of the pair-count kernels, shared by the single-count kernel
// and the batched kernel (each translation unit instantiates what it uses).
#pragma once

#include <math.h>
#include <stdint.h>

#include "cute_internal.h"
#include "runtime.h"

namespace cute {

namespace {

constexpr uint32_t kNoBin = 0xffffffffu;
constexpr double kPi = 3.14159265358979323846264338327950288;

// Read-only device memory seen through the constant address space: loads at
// wave-uniform addresses become scalar (s_load) loads into SGPRs.
typedef const __attribute__((address_space(4))) float* cfp;
typedef const __attribute__((address_space(4))) double* cdp;
typedef const __attribute__((address_space(4))) uint32_t* cu32p;
typedef const __attribute__((address_space(4))) CountArgs* cargp;

// x, y, z of the U consecutive points h .. h+U-1 from one base address with
// constant offsets (the index is widened before the offsets are added, so the
// scalar loads share one address computation and can merge)
template <uint32_t U>
__device__ __forceinline__ void load_points32(const float4* p, uint32_t h, float* x, float* y,
                                              float* z) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(4))) f4v* cf4p;
    const cf4p f = (cf4p)(const void*)(p + h);
#pragma unroll
    for (uint32_t u = 0; u < U; u++) {
        const f4v q = f[u];
        x[u] = q.x;
        y[u] = q.y;
        z[u] = q.z;
    }
}
template <uint32_t U>
__device__ __forceinline__ void load_points64(const P64* p, uint32_t h, double* x, double* y,
                                              double* z) {
    const cdp f = (cdp)(const void*)(p + h);
#pragma unroll
    for (uint32_t u = 0; u < U; u++) {
        x[u] = f[4 * u];
        y[u] = f[4 * u + 1];
        z[u] = f[4 * u + 2];
    }
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int unii(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
// base plus the number of lower lanes set in a mask
__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t base = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}
// A lane mask as a lane's own truth value.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int floordiv(int a, int n) { return a >= 0 ? a / n : -((-a + n - 1) / n); }

// ---------------------------------------------------------------------------
// Canonical FP64 classification (identical predicates to a plain FP64 double
// loop: squared quantities against squared edges, explicit fused multiply-adds,
// no square root or division). dx, dy, dz are the separation p - q (minimum
// image already applied), l the sum p + q (midpoint line of sight).
// Returns the flattened bin or kNoBin.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int last_le64(const double* t, int n, double v, int k) {
    // largest k in [0, n-1] with t[k] <= v, given t[0] <= v < t[n]; k is a guess
    while (k > 0 && v < t[k]) k--;
    while (k < n - 1 && v >= t[k + 1]) k++;
    return k;
}

__device__ __forceinline__ int last_ratio64(const double* t, int n, double num, double den,
                                            int k) {
    // largest k in [0, n-1] with num >= t[k] * den, given it holds at 0
    while (k > 0 && !(num >= t[k] * den)) k--;
    while (k < n - 1 && num >= t[k + 1] * den) k++;
    return k;
}

template <int MODE>
__device__ __forceinline__ uint32_t classify64(const CountArgs& P, const double* T1,
                                               const double* T2, double dx, double dy, double dz,
                                               double lx, double ly, double lz, int k1g,
                                               int k2g) {
    const int n1 = P.n1, n2 = P.n2;
    double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
    if (MODE == M_MONO || MODE == M_THETA) {
        if (!(T1[0] <= d2 && d2 < T1[n1])) return kNoBin;
        return (uint32_t)last_le64(T1, n1, d2, k1g);
    }
    if (MODE == M_RMU_Z || MODE == M_RMU_MID) {
        if (!(T1[0] <= d2 && d2 < T1[n1])) return kNoBin;
        int ir = last_le64(T1, n1, d2, k1g);
        double num, den;
        if (MODE == M_RMU_Z) {
            num = dz * dz;
            den = d2;
        } else {
            double sl = fma(dz, lz, fma(dy, ly, dx * lx));
            double ll = fma(lz, lz, fma(ly, ly, lx * lx));
            if (ll == 0.0) {
                num = 0.0;
                den = 1.0;
            } else {
                num = sl * sl;
                den = d2 * ll;
            }
        }
        if (d2 == 0.0) {
            num = 0.0;
            den = 1.0;
        }
        if (!(num >= T2[0] * den)) return kNoBin;
        if (!P.mu_top_closed && num >= T2[n2] * den) return kNoBin;
        int im = last_ratio64(T2, n2, num, den, k2g);
        return (uint32_t)(ir * n2 + im);
    }
    // SIGMAPI, midpoint line of sight
    double sl = fma(dz, lz, fma(dy, ly, dx * lx));
    double ll = fma(lz, lz, fma(ly, ly, lx * lx));
    double cx = fma(dy, lz, -(dz * ly));
    double cy = fma(dz, lx, -(dx * lz));
    double cz = fma(dx, ly, -(dy * lx));
    double c2 = fma(cz, cz, fma(cy, cy, cx * cx));
    double sn, pn, den;
    if (ll == 0.0) {
        sn = d2;
        pn = 0.0;
        den = 1.0;
    } else {
        sn = c2;
        pn = sl * sl;
        den = ll;
    }
    if (!(sn >= T1[0] * den)) return kNoBin;
    if (sn >= T1[n1] * den) return kNoBin;
    if (!(pn >= T2[0] * den)) return kNoBin;
    if (pn >= T2[n2] * den) return kNoBin;
    int is = last_ratio64(T1, n1, sn, den, k1g);
    int ip = last_ratio64(T2, n2, pn, den, k2g);
    return (uint32_t)(is * n2 + ip);
}

// Guess of the dimension-1 bin from a float value (used to start the exact
// search; any guess in range gives the right answer).
template <int MODE, int EST>
__device__ __forceinline__ int guess1(const CountArgs& P, float v) {
    float t;
    if (MODE == M_THETA) {
        float c = __builtin_amdgcn_sqrtf(v);
        float th = fmaf(c * v, 1.0f / 24.0f, c);  // 2 asin(c/2) to third order
        t = est_log(EST) ? __builtin_amdgcn_logf(th) : th;
    } else {
        t = est_log(EST) ? __builtin_amdgcn_logf(v) : __builtin_amdgcn_sqrtf(v);
    }
    return (int)__builtin_amdgcn_fmed3f(fmaf(t, P.e1a, P.e1b), 0.0f, P.n1m1);
}

// clamp to [0, n-1] with one v_med3; a NaN estimate converts to bin 0 or is
// clamped, so the index always stays in range
__device__ __forceinline__ int guess_lin(float t, float a, float b, float nm1) {
    return (int)__builtin_amdgcn_fmed3f(fmaf(t, a, b), 0.0f, nm1);
}

// Canonical classification of a queued pair from the sorted FP64 copies.
template <int MODE, int EST>
__device__ uint32_t classify_pair64(const CountArgs& P, const double* T1, const double* T2,
                                    const P64& p, const P64& q) {
    double dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
    if (P.periodic) {
        const double L = P.L, h = 0.5 * P.L;
        dx = dx > h ? dx - L : (dx < -h ? dx + L : dx);
        dy = dy > h ? dy - L : (dy < -h ? dy + L : dy);
        dz = dz > h ? dz - L : (dz < -h ? dz + L : dz);
    }
    double lx = p.x + q.x, ly = p.y + q.y, lz = p.z + q.z;
    double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
    float v = (float)d2;
    int k1, k2 = 0;
    if (MODE == M_SIGMAPI) {
        double sl = fma(dz, lz, fma(dy, ly, dx * lx));
        double ll = fma(lz, lz, fma(ly, ly, lx * lx));
        float inv = ll > 0.0 ? (float)(1.0 / ll) : 0.0f;
        float pi2 = (float)(sl * sl) * inv;
        float sg2 = fmaxf(v - pi2, 0.0f);
        k1 = guess_lin(__builtin_amdgcn_sqrtf(sg2), P.e1a, P.e1b, P.n1m1);
        k2 = guess_lin(__builtin_amdgcn_sqrtf(pi2), P.e2a, P.e2b, P.n2m1);
    } else {
        k1 = guess1<MODE, EST>(P, v);
        if (MODE == M_RMU_Z) {
            float mu = d2 > 0.0 ? (float)(fabs(dz) / sqrt(d2)) : 0.0f;
            k2 = guess_lin(mu, P.e2a, P.e2b, P.n2m1);
        } else if (MODE == M_RMU_MID) {
            double sl = fma(dz, lz, fma(dy, ly, dx * lx));
            double ll = fma(lz, lz, fma(ly, ly, lx * lx));
            float mu = (d2 > 0.0 && ll > 0.0) ? (float)(fabs(sl) / sqrt(d2 * ll)) : 0.0f;
            k2 = guess_lin(mu, P.e2a, P.e2b, P.n2m1);
        }
    }
    return classify64<MODE>(P, T1, T2, dx, dy, dz, lx, ly, lz, k1, k2);
}

// ---------------------------------------------------------------------------
// FP32 classification with rounding bands.
//
// Bin estimates are kept as biased integers: the bits of the float 2^23 + k.
// The host shifts the estimated variable t by s = (b - 1/2) / a, so that
// fma(t + s, a, 2^23) rounds to 2^23 + floor(t a + b) (for |t a + b| < 2^22);
// the bits are then clamped as unsigned integers to [2^23, 2^23 + n - 1]
// (below 2^23 the float bits are smaller, a NaN or a negative float larger,
// so every estimate lands on a valid index). The low 24 bits are k itself,
// which v_mad_u32_u24 reads directly, and (bits << 3) plus a pre-biased table
// address is the table entry: no float-to-int conversion anywhere.
// Output: in   -> certainly in the estimated bin (same as the canonical decision)
//         out  -> certainly not counted
//         else -> ambiguous (to be re-tested)
// tent: the FP32-only decision (bin or kNoBin), used by FP32_ONLY and for
//       counting flips.
// ---------------------------------------------------------------------------
constexpr uint32_t kBias = 0x4B000000u;   // bits of 2^23

struct C32 {
    bool in, out;
    uint32_t kb, kmb;   // biased estimates of dimension 1 and 2 (kmb = kBias for 1-D kinds)
};

// wave-uniform constants the VALU needs in VGPRs (an fma or med3 can read
// only one SGPR): the bias (which is also the float 2^23) and the LDS
// addresses of the band tables minus the bias times 8
struct Tab32 {
    uint32_t vbias;      // VGPR copy of kBias
    uint32_t vbias1;     // and of kBias + 1 (the float 2^23 + 1)
    uint32_t tb1, tb2;   // LDS byte address of B1 (B2) - (kBias << 3), modulo 2^32
    float d0, d1;        // VGPR copies of the mu band's constant and linear terms
    float mt;            // sigma-pi: the tile's t
};

typedef float __attribute__((ext_vector_type(2))) f2v;
typedef const __attribute__((address_space(3))) f2v* lds_f2p;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}

template <int EST>
__device__ __forceinline__ Tab32 make_tab32(const CountArgs& P, const float2* B1, const float2* B2) {
    Tab32 t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t.vbias) : "s"(kBias));
    asm volatile("v_mov_b32 %0, %1" : "=v"(t.vbias1) : "s"(kBias + 1u));
    asm volatile("v_mov_b32 %0, %1" : "=v"(t.d0) : "s"(est_muf(EST) ? P.muB0 : P.dA0p));
    asm volatile("v_mov_b32 %0, %1" : "=v"(t.d1) : "s"(P.muB1));
    t.mt = 0.f;
    t.tb1 = lds_addr(B1) - (kBias << 3);
    t.tb2 = lds_addr(B2) - (kBias << 3);
    return t;
}

__device__ __forceinline__ uint32_t med3u(uint32_t x, uint32_t lo_v, uint32_t hi_s) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(lo_v), "s"(hi_s));
    return r;
}

// biased estimate from a shifted variable ts (see above)
__device__ __forceinline__ uint32_t est_bits(float ts, float a, const Tab32& T, uint32_t top) {
    return med3u(__float_as_uint(fmaf(ts, a, __uint_as_float(T.vbias))), T.vbias, top);
}

// The same estimate in two parts: the float e = fl(2^23 + x), x = ts a, is
// 2^23 + round(x) for x >= -1/4; its bits clamped to the bins (est_bits) are
// those of the float 2^23 + k, k the pair's bin along that dimension. The
// offset x - k is formed with one rounding (the fma adds 2^23 - (2^23 + k),
// exact, to the exact product ts a): the pair's distance from the centre of
// bin k in bin units, at least 1/2 in size for a pair outside bin k (past
// the first or the last bin included).
__device__ __forceinline__ float est_float(float ts, float a, const Tab32& T) {
    return fmaf(ts, a, __uint_as_float(T.vbias));
}
__device__ __forceinline__ float est_offset(float ts, float a, const Tab32& T, uint32_t kbits) {
    return fmaf(ts, a, __uint_as_float(T.vbias) - __uint_as_float(kbits));
}

// v inside the band [lo, hi'] of its bin (hi' the largest float below the
// upper threshold; an empty band is (inf, inf)): one med3 and one compare,
// whose result is the mask itself
__device__ __forceinline__ bool in_band(float v, float2 b) {
    return __builtin_amdgcn_fmed3f(v, b.x, b.y) == v;
}

__device__ __forceinline__ float2 band_at(uint32_t tb, uint32_t kb) {
    const f2v b = *(lds_f2p)(uintptr_t)((kb << 3) + tb);
    return make_float2(b.x, b.y);
}

// flattened bin of an estimate
__device__ __forceinline__ uint32_t c32_bin(const CountArgs& P, const C32& c) {
    return __umul24(c.kb, (uint32_t)P.n2p1) + (c.kmb - kBias);
}

// LO: the first threshold can be crossed (out_lo >= 0); without it a pair is
// never clean-out on the low side, so that compare is skipped.
template <int MODE, int EST, bool WANT_TENT, bool LO = true>
__device__ __forceinline__ C32 classify32(const CountArgs& P, const Tab32& T, float dx, float dy,
                                          float dz, float lx, float ly, float lz, uint32_t* tent) {
    C32 c;
    c.kmb = kBias;
    float v = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    if (MODE == M_MONO | MODE == M_THETA) {
        float ts;
        if (MODE == M_THETA) {
            float ch = __builtin_amdgcn_sqrtf(v);
            float th = fmaf(ch * v, 1.0f / 24.0f, ch);  // 2 asin(c/2) to third order
            ts = (est_log(EST) ? __builtin_amdgcn_logf(th) : th) + P.s1;
        } else if (est_log(EST)) {
            ts = __builtin_amdgcn_logf(v) + P.s1;
        } else {
            ts = fmaf(v, __builtin_amdgcn_rsqf(v), P.s1);
        }
        c.kb = est_bits(ts, P.e1a, T, P.top1);
        float2 b = band_at(T.tb1, c.kb);
        c.in = in_band(v, b);
        c.out = LO ? (v >= P.out_hi) | (v < P.out_lo) : (v >= P.out_hi);
        if (WANT_TENT) *tent = (v >= P.bot32 & v < P.top32) ? c.kb - kBias : kNoBin;
        return c;
    }
    if (MODE == M_RMU_Z) {
        float rinv = __builtin_amdgcn_rsqf(v);
        float ts = est_log(EST) ? __builtin_amdgcn_logf(v) + P.s1 : fmaf(v, rinv, P.s1);
        const float er = est_float(ts, P.e1a, T);
        c.kb = med3u(__float_as_uint(er), T.vbias, P.top1);
        float ts2 = fmaf(fabsf(dz), rinv, P.s2);
        const float em = est_float(ts2, P.e2a, T);
        c.kmb = med3u(__float_as_uint(em), T.vbias, P.top2);
        float dz2 = dz * dz;
        // linear r bins: r is decided in bin units as mu is, without the
        // band table; a pair certified there lies inside the v-space band of
        // its bin
        constexpr bool kRx = est_muf(EST) && !est_log(EST) && !WANT_TENT;
        bool rin;
        if constexpr (kRx) {
            rin = fabsf(est_offset(ts, P.e1a, T, c.kb)) <= P.rB0;
        } else {
            float2 b = band_at(T.tb1, c.kb);
            rin = in_band(v, b);
        }
        bool min_;
        if (est_muf(EST) && !WANT_TENT) {
            // in mu space: x = ts2 a = mu a + b - 1/2 is the pair's position
            // in bin units, inside its bin when the offset from the bin's
            // centre is at most 1/2 - beta(r), beta(r) = muB0' + |muB1| / r
            // (T.d0 = 1/2 - muB0', the band kept as a half-width)
            float half = fmaf(P.muB1, rinv, T.d0);
            min_ = fabsf(est_offset(ts2, P.e2a, T, c.kmb)) <= half;
        } else {
            float2 m = band_at(T.tb2, c.kmb);
            // band of the mu predicates, linear in r: dA1 r + dA0. With linear
            // r bins ts = r + s1 and the host folds -dA1 s1 into the constant.
            float delta = est_log(EST) ? fmaf(P.dA1, v * rinv, T.d0) : fmaf(P.dA1, ts, T.d0);
            float flo = fmaf(m.x, v, dz2);
            float fhi = fmaf(m.y, v, dz2);
            min_ = (flo >= delta) & (fhi <= -delta);
        }
        // only r decides a clean "out"; a pair outside a partial mu range is
        // re-tested instead (never the case for mu in [0, 1])
        c.out = LO ? (v >= P.out_hi) | (v < P.out_lo) : (v >= P.out_hi);
        c.in = rin & min_;
        if (WANT_TENT) {
            bool rr = v >= P.bot32 & v < P.top32;
            bool mm = true;
            if (P.d2_partial) mm = (fmaf(P.nlo2_first, v, dz2) >= 0.0f) & (fmaf(P.nhi2_last, v, dz2) < 0.0f);
            *tent = (rr & mm) ? c32_bin(P, c) : kNoBin;
        }
        return c;
    }
    if (MODE == M_RMU_MID) {
        float sl = fmaf(dz, lz, fmaf(dy, ly, dx * lx));
        float ll = fmaf(lz, lz, fmaf(ly, ly, lx * lx));
        float rinv = __builtin_amdgcn_rsqf(v);
        float r = v * rinv;
        float ts = est_log(EST) ? __builtin_amdgcn_logf(v) + P.s1 : r + P.s1;
        c.kb = est_bits(ts, P.e1a, T, P.top1);
        float w = v * ll;
        float sl2 = sl * sl;
        // 1/|l| once: |l| for the band and mu = |s.l| / (r |l|) for the estimate
        float rl = __builtin_amdgcn_rsqf(ll);
        float lnorm = ll * rl;
        c.kmb = est_bits(fmaf(fabsf(sl), rinv * rl, P.s2), P.e2a, T, P.top2);
        float2 b = band_at(T.tb1, c.kb);
        float2 m = band_at(T.tb2, c.kmb);
        float delta = fmaf(ll, fmaf(P.dA2, v, fmaf(P.dA1, r, P.dA0)),
                           fmaf(lnorm, fmaf(P.dB2, v, fmaf(P.dB1, r, P.dB0)),
                                fmaf(P.dC2, v, P.dC0)));
        float flo = fmaf(m.x, w, sl2);
        float fhi = fmaf(m.y, w, sl2);
        bool rin = in_band(v, b);
        bool min_ = (flo >= delta) & (fhi <= -delta);
        c.in = rin & min_ & (ll >= P.llg);
        c.out = LO ? (v >= P.out_hi) | (v < P.out_lo) : (v >= P.out_hi);
        if (WANT_TENT) {
            bool rr = v >= P.bot32 & v < P.top32;
            bool mm = true;
            if (P.d2_partial) mm = (fmaf(P.nlo2_first, w, sl2) >= 0.0f) & (fmaf(P.nhi2_last, w, sl2) < 0.0f);
            *tent = (rr & mm) ? c32_bin(P, c) : kNoBin;
        }
        return c;
    }
    // SIGMAPI (midpoint): sigma^2 ll = |s|^2 |l|^2 - (s.l)^2, pi^2 ll = (s.l)^2
    float sl = fmaf(dz, lz, fmaf(dy, ly, dx * lx));
    float ll = fmaf(lz, lz, fmaf(ly, ly, lx * lx));
    float sl2 = sl * sl;
    float c2 = fmaf(v, ll, -sl2);
    // sigma = sqrt(c2) / |l| and pi = |s.l| / |l| share one 1/|l|. A c2
    // rounded below zero (a pair all but along l) gives a NaN estimate,
    // which the clamp puts in the last sigma bin, whose band test (on c2
    // itself) then fails: the pair is re-tested. The FP32-only decision
    // takes sigma = 0 instead.
    float rl = __builtin_amdgcn_rsqf(ll);
    float sg = __builtin_amdgcn_sqrtf(WANT_TENT ? fmaxf(c2, 0.0f) : c2) * rl;
    float pp = fabsf(sl) * rl;
    c.kb = est_bits(sg + P.s1, P.e1a, T, P.top1);
    c.kmb = est_bits(pp + P.s2, P.e2a, T, P.top2);
    if (WANT_TENT) {
        // out of range: sigma >= sigma_max, pi >= pi_max, or below the first edges
        float fstop = fmaf(P.out_hi, ll, c2);       // out_hi holds -S2f[n1]
        float fptop = fmaf(P.nhi2_last, ll, sl2);   // -P2f[n2]
        float fsbot = fmaf(P.out_lo, ll, c2);       // out_lo holds -S2f[0] (or +BIG)
        float fpbot = fmaf(P.nlo2_first, ll, sl2);  // -P2f[0] (or +BIG)
        bool ok = (fsbot >= 0.0f) & (fstop < 0.0f) & (fpbot >= 0.0f) & (fptop < 0.0f);
        // (top1 and top2 may be one past the last bin, see decide)
        c.kb = min(c.kb, kBias + (uint32_t)(P.n1 - 1));
        c.kmb = min(c.kmb, kBias + (uint32_t)(P.n2 - 1));
        *tent = ok ? c32_bin(P, c) : kNoBin;
        c.in = c.out = false;
        return c;
    }
    // the per-edge parts of the bands are in the tables; the part from the
    // direction error of l is t, in units of F. A bin's entry is (m, H): the
    // pair is inside it along that dimension when |F + m ll| <= H ll - t
    // (F/ll within H - t/ll of the centre -m of the certified interval)
    float t = fmaf(P.spK1, ll * rl, P.spK0);
    float2 bs = band_at(T.tb1, c.kb);
    float2 bp = band_at(T.tb2, c.kmb);
    // |s| below the skip threshold bounds every error term; ll >= llg bounds
    // the direction error of l
    bool vin = v < P.skip32;
    bool lg = ll >= P.llg;
    bool ins = fabsf(fmaf(bs.x, ll, c2)) <= fmaf(bs.y, ll, -t);
    bool inp = fabsf(fmaf(bp.x, ll, sl2)) <= fmaf(bp.y, ll, -t);
    c.in = vin & lg & ins & inp;
    bool top = (fmaf(P.sp_wstop, ll, c2) >= t) | (fmaf(P.sp_wptop, ll, sl2) >= t);
    if (LO) top = top | (fmaf(P.sp_wsbot, ll, c2) <= -t) | (fmaf(P.sp_wpbot, ll, sl2) <= -t);
    c.out = !vin | (lg & top);
    return c;
}

// ---------------------------------------------------------------------------
// Per-wave working state.
// ---------------------------------------------------------------------------
// Periodic image of a neighbour point: (kx+1) | (ky+1) << 2 | (kz+1) << 4,
// k in {-1, 0, 1}; the image lies at q + k L in the home point's frame.
constexpr uint32_t kNoShift = 0x15u;
// Beside it in a chunk's codes: the j > i test applies.
constexpr uint32_t kSelfSpan = 0x80u;

__device__ __forceinline__ float shift32(uint32_t code, int axis, float Lf) {
    return (float)((int)((code >> (2 * axis)) & 3u) - 1) * Lf;
}
__device__ __forceinline__ double shift64(uint32_t code, int axis, double L) {
    return (double)((int)((code >> (2 * axis)) & 3u) - 1) * L;
}

// Per-wave state. The queue, the histogram and the re-test statistics live
// in LDS; the rare paths take the queue length by value and return it.
struct WaveState {
    unsigned char* hist; // the workgroup's shared histogram (hist_words counters, kH32)
    uint32_t* qi;        // re-test queue: home index
    uint32_t* qj;        // re-test queue: neighbour index
    uint8_t* qc;         // re-test queue: neighbour image code
    float4* stage;       // the tile's home points in its own frame (kMfma kernels)
    uint16_t* list;      // ambiguous pairs of the chunk at hand: home offset << 6 | lane (kMfma)
    uint32_t nlist;      // how many (wave-uniform)
    float* alpha;        // per home point: |p|^2 - |P0|^2, P0 the origin (midpoint kinds); its
                         // redshift in bins (radial)
    float ox, oy, oz;    // that frame's origin in the grid's FP32 frame (wave-uniform)
    float lx, ly, lz;    // midpoint kinds: L0 = 2 P0 from the observer (wave-uniform)
    float mt, mb0, mb1;  // sigma-pi: the tile's t; mu: its band's constant and linear terms;
                         // radial: mt the largest alpha in size
    unsigned long long* rstat;  // [0] retests, [1] flips (LDS)
    uint32_t tail;       // queued entries (wave-uniform)
    uint64_t evals, tiles;
    // 32-bit histograms: the workgroup's budget of pair evaluations since the
    // histogram was last moved to the global counts (LDS), and this wave's
    // evaluations not reported to it yet
    uint32_t* budget;
    uint32_t pend;
    uint32_t all64;      // radial: counting in FP64 for now (see do_tile)
};

// LDS of a count workgroup: [staged home points | tables | histogram |
// re-test statistics | queues | spans | ambiguous pairs | queue and span
// codes | control words]; stage and ambiguous pairs for kMfma kernels only.
struct WgLds {
    double *T1, *T2;
    float2 *B1, *B2;
    unsigned char* hist;
    size_t hbytes;       // hist_words counters of 4 (kH32) or 8 bytes, padded to 8
    unsigned long long* rstat;
    uint32_t *queue, *spans, *ctl;
    uint16_t* list;
    uint8_t *qcodes, *scodes;
    float4* stage;
    float* alpha;
};
template <bool H32, bool MFMA, bool ALPHA>
__device__ __forceinline__ WgLds wg_lds(unsigned char* smem, int nwaves, int n1, int n2, int hist_words) {
    const int n2p = n2 > 0 ? n2 : 0;
    WgLds l;
    l.stage = reinterpret_cast<float4*>(smem);
    l.alpha = reinterpret_cast<float*>(smem + (MFMA ? (size_t)nwaves * kStage : 0));
    l.T1 = reinterpret_cast<double*>(l.alpha + (MFMA && ALPHA ? (size_t)nwaves * (kStageMid / 4) : 0));
    l.T2 = l.T1 + (n1 + 1);
    l.B1 = reinterpret_cast<float2*>(l.T2 + (n2p + 1));
    l.B2 = l.B1 + n1 + (MFMA ? 1 : 0);   // (sigma-pi: an entry past the last bin)
    l.hist = reinterpret_cast<unsigned char*>(l.B2 + (n2p > 0 ? n2p : 1) + (MFMA ? 1 : 0));
    l.hbytes = ((size_t)hist_words * (H32 ? 4 : 8) + 7) & ~(size_t)7;
    l.rstat = reinterpret_cast<unsigned long long*>(l.hist + l.hbytes);
    l.queue = reinterpret_cast<uint32_t*>(l.rstat + 2 * nwaves);
    l.spans = l.queue + (size_t)nwaves * 2 * kQCap;
    l.list = reinterpret_cast<uint16_t*>(l.spans + (size_t)nwaves * 2 * kSpanCap);
    l.qcodes = reinterpret_cast<uint8_t*>(l.list + (MFMA ? (size_t)nwaves * kList : 0));
    l.scodes = l.qcodes + (size_t)nwaves * kQCap;
    l.ctl = reinterpret_cast<uint32_t*>(l.scodes + (size_t)nwaves * kSpanCap);
    return l;
}

// The workgroup's histogram: several interleaved copies so that lanes
// hitting the same bin use different banks, copies a power of two: counter =
// (bin << log2(copies)) | (lane & (copies - 1)). 64-bit counters never wrap;
// 32-bit ones (kH32) are moved to the global counts in time (h32_flush).
template <bool H32>
__device__ __forceinline__ void hist_add(unsigned char* hist, uint32_t bin, int copies, int lane,
                                         uint64_t w = 1u) {
    const uint32_t lc = (uint32_t)__builtin_ctz((unsigned)copies);
    const uint32_t k = (bin << lc) | (uint32_t)(lane & (copies - 1));
    if constexpr (H32)
        atomicAdd(reinterpret_cast<uint32_t*>(hist) + k, (uint32_t)w);
    else
        atomicAdd(reinterpret_cast<unsigned long long*>(hist) + k, (unsigned long long)w);
}

// One increment at an LDS byte address (the lane's copy already folded in).
template <bool H32>
__device__ __forceinline__ void lds_add(uint32_t byte_addr, uint64_t w) {
    if constexpr (H32)
        __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t*)(uintptr_t)byte_addr,
                               (uint32_t)w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        __hip_atomic_fetch_add((__attribute__((address_space(3))) unsigned long long*)(uintptr_t)byte_addr,
                               (unsigned long long)w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ WaveState wave_state(const WgLds& l, int wave) {
    WaveState W;
    W.hist = l.hist;
    W.budget = nullptr;
    W.pend = 0;
    W.all64 = 0;
    W.qi = l.queue + (size_t)wave * 2 * kQCap;
    W.qj = W.qi + kQCap;
    W.qc = l.qcodes + (size_t)wave * kQCap;
    W.stage = l.stage + (size_t)wave * (kStage / 16);
    W.list = l.list + (size_t)wave * kList;
    W.nlist = 0;
    W.alpha = l.alpha + (size_t)wave * (kStageMid / 4);
    W.ox = W.oy = W.oz = W.lx = W.ly = W.lz = W.mt = W.mb0 = W.mb1 = 0.f;
    W.rstat = l.rstat + 2 * wave;
    W.tail = 0;
    W.evals = W.tiles = 0;
    return W;
}

// Move a 32-bit histogram to the global counts (one wave): every counter is
// swapped with zero, so increments of the other waves land either in the
// value moved or in the emptied counter, and none is lost. Out of line: it
// runs about once per 2^30 increments, and inlined it measured no faster.
__device__ __attribute__((noinline)) void h32_flush(uint32_t* hist, int words, int copies,
                                                    unsigned long long* counts, int lane) {
    const uint32_t lc = (uint32_t)__builtin_ctz((unsigned)copies);
    for (int w = lane; w < words; w += 64) {
        const uint32_t v = atomicExch(&hist[w], 0u);
        if (v) atomicAdd(&counts[(uint32_t)w >> lc], (unsigned long long)v);
    }
}

// The same for 64-bit counters that hold two 32-bit ones (region passes: pairs
// with a neighbour in the home region in the low half, others in the high).
__device__ __attribute__((noinline)) void h64_flush(unsigned long long* hist, int words, int copies,
                                                    unsigned long long* lo, unsigned long long* hi, int lane) {
    const uint32_t lc = (uint32_t)__builtin_ctz((unsigned)copies);
    for (int w = lane; w < words; w += 64) {
        const unsigned long long v = atomicExch(&hist[w], 0ull);
        if ((uint32_t)v) atomicAdd(&lo[(uint32_t)w >> lc], v & 0xffffffffull);
        if (v >> 32) atomicAdd(&hi[(uint32_t)w >> lc], v >> 32);
    }
}

// Account the pair evaluations of a chunk to the workgroup's budget of a
// 32-bit histogram (every pair adds at most wmax to one counter; PAIR: one of
// two halves, at most 1). A wave
// reports its evaluations every h32_report of them; the wave that finds the
// budget at h32_flush or more resets it and moves the histogram. A counter
// then holds at most h32_flush plus what the waves have not reported or were
// adding during the move (a few h32_report), far below 2^32.
template <bool PAIR = false>
__device__ __forceinline__ void h32_account(const CountArgs& P, WaveState& W, int lane,
                                            uint32_t evals) {
    W.pend += evals;
    if (W.pend < P.h32_report) return;
    uint32_t old = 0;
    if (lane == 0) old = atomicAdd(W.budget, W.pend);
    old = uni(old);
    const uint32_t now = old + W.pend;
    W.pend = 0;
    if (now < P.h32_flush) return;
    if (lane == 0) atomicExch(W.budget, 0u);
    if constexpr (PAIR)
        h64_flush(reinterpret_cast<unsigned long long*>(W.hist), P.hist_words, P.copies, P.counts,
                  P.counts_hi, lane);
    else
        h32_flush(reinterpret_cast<uint32_t*>(W.hist), P.hist_words, P.copies, P.counts, lane);
}

// Weight of a pair in a region pass: wsame if the neighbour lies in the home
// region, wdiff otherwise (1 outside region passes).
__device__ __forceinline__ uint64_t pair_weight(const CountArgs& P, uint32_t j) {
    if (P.regs == nullptr) return 1u;
    return P.regs[j] == (uint16_t)P.region ? P.wsame : P.wdiff;
}

// Weight of the pair (home i, neighbour j): the product of the two point
// weights of pixel maps, else the region weight.
__device__ __forceinline__ uint64_t pair_weight2(const CountArgs& P, uint32_t i, uint32_t j) {
    if (P.wA != nullptr) return (uint64_t)P.wA[i] * (uint64_t)P.wB[j];
    return pair_weight(P, j);
}

// Radial pairs (Sec. 2.1, radial 2PCF; Sec. 3.4): inside the aperture when
// the chord^2 of the unit vectors is below ap2, then binned by the redshift
// difference |r_i - r_j| against the unsquared edges T1 (half-open).
__device__ __forceinline__ uint32_t classify_radial(const CountArgs& P, const double* T1, double d2,
                                                    double dr) {
    if (!(d2 < P.ap2)) return kNoBin;
    const int n = P.n1;
    if (!(T1[0] <= dr && dr < T1[n])) return kNoBin;
    int lo = 0, hi = n;  // T1[lo] <= dr < T1[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (T1[mid] <= dr) lo = mid; else hi = mid;
    }
    return (uint32_t)lo;
}

// Re-test up to 64 queued pairs per pass, one per lane, through the canonical
// FP64 predicates; count the pairs for which FP32_ONLY decides otherwise (flips).
// Returns the new queue length.
template <int MODE, int EST>
__device__ __forceinline__ uint32_t drain_queue(
    const CountArgs* __restrict__ Pg, unsigned char* hist, uint32_t* qi, uint32_t* qj, uint8_t* qc,
    unsigned long long* rstat, const float2* B1, const float2* B2, const double* T1,
    const double* T2, int lane, uint32_t tail, bool all) {
    const CountArgs& P = *Pg;
    tail = uni(tail);
    while (tail >= 64u || (all && tail > 0u)) {
        const uint32_t n = tail < 64u ? tail : 64u;
        const bool act = (uint32_t)lane < n;
        uint32_t k = kNoBin, t = kNoBin;
        if (act) {
            const uint32_t i = qi[lane], j = qj[lane], code = qc[lane];
            const P64 p = P.A.p64[i];
            const P64 q = P.B.p64[j];
            if constexpr (MODE == M_RADIAL) {
                const double dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
                k = classify_radial(P, T1, fma(dz, dz, fma(dy, dy, dx * dx)), fabs(P.rA[i] - P.rB[j]));
                t = k;   // (no FP32-only decision to differ from)
            } else {
                k = classify_pair64<MODE, EST>(P, T1, T2, p, q);
            }
            if (k != kNoBin) hist_add<kH32<MODE>>(hist, k, P.copies, lane, pair_weight2(P, i, j));
            if constexpr (MODE != M_RADIAL) {
                // the decision that FP32_ONLY makes for the same pair
                const float4 a = P.A.p32[i];
                const float4 b = P.B.p32[j];
                const float Lf = (float)P.L;
                const float qx = b.x - (P.offx - shift32(code, 0, Lf));
                const float qy = b.y - (P.offy - shift32(code, 1, Lf));
                const float qz = b.z - (P.offz - shift32(code, 2, Lf));
                const Tab32 tab = make_tab32<EST>(P, B1, B2);
                (void)classify32<MODE, EST, true>(P, tab, a.x - qx, a.y - qy, a.z - qz,
                                                  a.x + (qx + P.lcx), a.y + (qy + P.lcy),
                                                  a.z + (qz + P.lcz), &t);
            }
        }
        const uint64_t fl = __builtin_amdgcn_ballot_w64(act && k != t);
        if (lane == 0) {
            rstat[0] += n;
            rstat[1] += (unsigned long long)__popcll(fl);
        }
        const uint32_t rest = tail - n;
        if ((uint32_t)lane < rest) {
            const uint32_t a = qi[n + lane], b = qj[n + lane], c = qc[n + lane];
            qi[lane] = a;
            qj[lane] = b;
            qc[lane] = (uint8_t)c;
        }
        tail = rest;
    }
    return tail;
}

// Queue the ambiguous pairs of a chunk: for every home offset o set in hsum,
// the lanes whose bit o is set in ambh (pair: home ts + o, the lane's
// neighbour). Drains whenever 64 or more pairs are waiting. Both functions
// are inlined: most chunks of a clustered catalog queue a pair or two, and an
// out-of-line call costs its argument moves, the registers the call
// convention saves (the r-mu and sigma-pi kernels spilled around it) and a
// stack frame; inlined, the r-mu count takes 3 % less time, the others 1 %.
template <int MODE, int EST>
__device__ __forceinline__ uint32_t enqueue_chunk(
    const CountArgs* __restrict__ Pg, unsigned char* hist, uint32_t* qi, uint32_t* qj, uint8_t* qc,
    unsigned long long* rstat, const float2* B1, const float2* B2, const double* T1,
    const double* T2, int lane, uint32_t tail, uint32_t ts, uint32_t lj, uint32_t lcode,
    uint64_t ambh, uint64_t hsum) {
    tail = uni(tail);
    uint32_t hlo = uni((uint32_t)hsum), hhi = uni((uint32_t)(hsum >> 32));
    while (hlo | hhi) {
        const uint32_t o = hlo ? (uint32_t)__builtin_ctz(hlo) : 32u + (uint32_t)__builtin_ctz(hhi);
        if (o < 32u) hlo &= hlo - 1u; else hhi &= hhi - 1u;
        const bool mine = ((ambh >> o) & 1ull) != 0ull;
        const uint64_t m = __builtin_amdgcn_ballot_w64(mine);
        const uint32_t pre =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (mine) {
            const uint32_t pos = tail + pre;
            qi[pos] = ts + o;
            qj[pos] = lj;
            qc[pos] = (uint8_t)lcode;
        }
        tail += (uint32_t)__popcll(m);
        if (tail >= 64u)
            tail = drain_queue<MODE, EST>(Pg, hist, qi, qj, qc, rstat, B1, B2, T1, T2, lane, tail,
                                          false);
    }
    return tail;
}

// ---------------------------------------------------------------------------
// The hot loop. A chunk holds up to 64 neighbour points, one per lane, in
// VGPRs; the home points of the tile are taken U at a time, so that U
// independent pair evaluations per lane interleave. Every lane evaluates the
// pair (home h, its neighbour). In the matrix-core kernels the home points are
// rows of a product, staged in LDS (see step_mfma); in the others they are
// wave-uniform and arrive through scalar loads.
// ---------------------------------------------------------------------------
// Home points h .. h+U-1 not excluded by the point mask (wave-uniform).
template <bool PM, uint32_t U>
__device__ __forceinline__ void home_valid(const CountArgs& P, uint32_t h, bool* hv) {
#pragma unroll
    for (uint32_t u = 0; u < U; u++) hv[u] = true;
    if (PM && P.mbA != nullptr) {
        const cu32p mb = (cu32p)(const void*)P.mbA;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const uint32_t i = h + u;
            hv[u] = ((mb[i >> 5] >> (i & 31u)) & 1u) == 0u;
        }
    }
}

// Weights of home points h .. h+U-1 (wave-uniform, scalar loads).
template <bool WT, uint32_t U>
__device__ __forceinline__ void home_weights(const CountArgs& P, uint32_t h, uint32_t* hw) {
#pragma unroll
    for (uint32_t u = 0; u < U; u++) hw[u] = 1u;
    if (WT) {
        const cu32p wa = (cu32p)(const void*)P.wA;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) hw[u] = wa[h + u];
    }
}

template <int MODE, int PREC, int EST, bool PM, bool WT, bool MASKED, bool LO, uint32_t U>
__device__ __forceinline__ void step32(const CountArgs& P, WaveState& W, const Tab32& T,
                                       const float2* B1, const float2* B2, const double* T1,
                                       const double* T2, int lane, bool lvalid, bool lmask,
                                       uint32_t lj, uint32_t lcode, float qx, float qy, float qz,
                                       float qlx, float qly, float qlz, uint32_t lb, uint64_t lw,
                                       uint32_t ts, uint64_t& ambh, uint64_t& hsum, uint32_t h) {
    float hx[U], hy[U], hz[U];
    load_points32<U>(P.A.p32, h, hx, hy, hz);
    bool hv[U];
    home_valid<PM, U>(P, h, hv);
    uint32_t hw[U];
    home_weights<WT, U>(P, h, hw);
    {
        // Every mode has a separation past which no pair is counted: the top edge of r or of the
        // chord of theta, the aperture of radial pairs, and for sigma-pi sqrt(sigma_max^2 +
        // pi_max^2), since sigma^2 + pi^2 = r^2 for any line of sight. A step whose every pair
        // lies past it (skip32 in FP32, on the clean-out side of the rounding band; top64 in
        // FP64) is skipped after the separations alone. Points are sorted by cell and home tiles
        // are compact, so on clustered catalogs whole steps (four home points against a chunk of
        // nearby neighbours) often fall beyond r_max together; the separations are still formed
        // for every pair.
        float vmin = 0.f;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const float dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
            const float v = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            vmin = u == 0 ? v : fminf(vmin, v);
        }
        if (__builtin_amdgcn_ballot_w64(vmin < P.skip32) == 0ull) return;
    }
    uint32_t off[U];
    bool cnt[U], amb[U];
#pragma unroll
    for (uint32_t u = 0; u < U; u++) {
        const bool act = lvalid & hv[u] &
                         (!MASKED | !lmask | (lj > h + u) | ((P.selfx != 0) & (lj < h + u)));
        const float dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
        float lx = 0.f, ly = 0.f, lz = 0.f;
        if (MODE == M_RMU_MID || MODE == M_SIGMAPI) {
            lx = hx[u] + qlx;
            ly = hy[u] + qly;
            lz = hz[u] + qlz;
        }
        if (PREC == P_FP32O) {
            uint32_t tent;
            (void)classify32<MODE, EST, true>(P, T, dx, dy, dz, lx, ly, lz, &tent);
            cnt[u] = act & (tent != kNoBin);
            off[u] = __umul24(tent, (uint32_t)P.hs2) + lb;
            amb[u] = false;
        } else {
            const C32 c = classify32<MODE, EST, false, LO>(P, T, dx, dy, dz, lx, ly, lz, nullptr);
            cnt[u] = act & c.in;
            amb[u] = act & !(c.in | c.out);
            // LDS byte address of the bin in this lane's copy of the histogram
            if (MODE == M_MONO || MODE == M_THETA)
                off[u] = __umul24(c.kb, (uint32_t)P.hs1) + lb;
            else
                off[u] = __umul24(c.kb, (uint32_t)P.hs1) + (__umul24(c.kmb, (uint32_t)P.hs2) + lb);
        }
    }
    // one vote for the whole step; the per-pair votes only on the rare path
    uint64_t any_amb = 0;
    if (PREC == P_FP32E) {
        bool any = false;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) any = any | amb[u];
        any_amb = __builtin_amdgcn_ballot_w64(any);
    }
#pragma unroll
    for (uint32_t u = 0; u < U; u++)
        if (cnt[u]) lds_add<kH32<MODE>>(off[u], WT ? lw * hw[u] : lw);
    if (PREC == P_FP32E && any_amb) {
        // remember the pair for the end of the chunk: bit (home - ts) of this
        // lane's mask, and the home offset in the wave's mask
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const uint64_t bit = 1ull << (h + u - ts);
            if (__builtin_amdgcn_ballot_w64(amb[u])) hsum |= bit;
            if (amb[u]) ambh |= bit;
        }
    }
}

// ---------------------------------------------------------------------------
// Separations from the matrix cores (FP32_EDGE). With the home points and the neighbours in the frame of the home
// tile (a and b), |a - b|^2 = |b|^2 - 2 a.b + |a|^2 is one chain of four
// v_mfma_f32_4x4x1 (sixteen blocks of 4 x 4 pairs, K = 1 each): the columns of
// the blocks are the lanes' neighbours, the four rows of every block the same
// four home points, so a lane receives its neighbour's values against four
// home points in four registers, the layout of the VALU code that follows.
// An instruction takes 10.4 cycles (measured; it shares the FP32 pipe, so it
// does not overlap with VALU work) and does what four VALU fused
// multiply-adds do in 17.8: the separations of four pairs take 41.4 cycles
// instead of 107 for three subtractions and three multiply-adds per pair, and
// dz 10.4 instead of 17.8. Each step is a fused multiply-add rounded once
// (checked bit for bit against fmaf); the error of the expanded form is in
// d2_bound. A point that is not there (past the tile's end, masked, or an
// idle lane) has |a|^2 or |b|^2 = kFar and falls past the top edge.
// ---------------------------------------------------------------------------
typedef float __attribute__((ext_vector_type(4))) f4v;
constexpr float kFar = 1e33f;
template <int MODE>
constexpr bool kMid = MODE == M_SIGMAPI || MODE == M_RMU_MID;
template <int MODE>
constexpr bool kAlpha = alpha_mode(MODE);

// Origin of a tile's frame, in the grid's FP32 frame: the centre of its box
// of cells (an axis of one cell: the grid's centre), on the sphere the point
// in the middle of its run.
template <bool SPH>
__device__ __forceinline__ void tile_origin(const CountArgs& P, const Tile& tl, float* ox, float* oy,
                                            float* oz) {
    const GridView& A = P.A;
    float x, y, z;
    if constexpr (SPH) {
        const float4 p = A.p32[tl.start + ((tl.end - tl.start) >> 1)];
        x = p.x;
        y = p.y;
        z = p.z;
    } else {
        const int c0 = (int)(tl.c0c1 & 0xffffu), c1 = (int)(tl.c0c1 >> 16);
        const int cy = (int)(tl.row % (uint32_t)A.ny), cz = (int)(tl.row / (uint32_t)A.ny);
        x = A.nx == 1 ? 0.f : (float)(A.ox + 0.5 * (double)(c0 + c1 + 1) * A.ax - A.cx);
        y = A.ny == 1 ? 0.f : (float)(A.oy + ((double)cy + 0.5) * A.ay - A.cy);
        z = A.nz == 1 ? 0.f : (float)(A.oz + ((double)cz + 0.5) * A.az - A.cz);
    }
    *ox = __uint_as_float(uni(__float_as_uint(x)));
    *oy = __uint_as_float(uni(__float_as_uint(y)));
    *oz = __uint_as_float(uni(__float_as_uint(z)));
}

// The arguments' copy in device memory, out of the compiler's sight.
__device__ __forceinline__ const CountArgs& args_again(const CountArgs& P) {
    const uint64_t u = (uint64_t)(uintptr_t)P.self;
    uint64_t v = (uint64_t)uni((uint32_t)u) | ((uint64_t)uni((uint32_t)(u >> 32)) << 32);
    asm volatile("" : "+s"(v));
    return *(const CountArgs*)(cargp)v;
}

__device__ __forceinline__ double dot64(float ax, float ay, float az, float bx, float by, float bz) {
    return fma((double)az, (double)bz, fma((double)ay, (double)by, (double)ax * (double)bx));
}
__device__ __forceinline__ double sq64(float x, float y, float z) { return dot64(x, y, z, x, y, z); }
__device__ __forceinline__ float unif(float v) { return __uint_as_float(uni(__float_as_uint(v))); }

// Midpoint line of sight, l = p + q = L0 + a + b with L0 = 2 P0 (P0 the tile's
// origin from the observer): s.l = |p|^2 - |q|^2 = alpha - beta with alpha =
// L0.a + |a|^2 and beta = L0.b + |b|^2 (formed in FP64, rounded once), and
// |l|^2 = |L0|^2 + 2 alpha + 2 beta - |s|^2. So sl and |l|^2 + v are two more
// products of one step each and ll one subtraction, where the components took
// twelve operations. Errors (u = 2^-24, M >= |a| + |b|, Lx = |L0| + M >= |l|):
//   |sl32 - s.l| <= Esl + u |sl|,   Esl = u (Lx M + M^2)
//   |ll32 - |l|^2| <= Ell = 1.01 u (3 Lx^2 + 2 Lx M + 9.1 M^2)
// (u |alpha|, u |beta| <= u (|L0| |a| + a^2) each; 2 alpha, the rounding of 2
// beta + |L0|^2, of the sum, of ll, and the error of v). In units of F (c2 or
// sl^2, see midpoint_bands) they and the direction error of l are below
//   t = K1 Lx + K0 + (T_max + R^2) Ell + 2 R Lx Esl + Esl^2
// for every pair of the tile; mu: see midpoint_mu_band.
template <int MODE>
__device__ __forceinline__ void midpoint_tile(const CountArgs& P, WaveState& W) {
    const float u = 0x1p-24f;
    W.lx = unif((float)(2.0 * (P.A.cx + (double)W.ox)));
    W.ly = unif((float)(2.0 * (P.A.cy + (double)W.oy)));
    W.lz = unif((float)(2.0 * (P.A.cz + (double)W.oz)));
    const float l0 = __builtin_sqrtf((float)sq64(W.lx, W.ly, W.lz));
    const float M = P.mdM, Lx = fmaf(l0, 1.00001f, M);
    const float esl = 1.001f * u * (Lx * M + M * M);
    const float ell = 1.011f * u * (3.0f * Lx * Lx + 2.0f * Lx * M + 9.1f * M * M);
    if constexpr (MODE == M_SIGMAPI) {
        const float t = P.spK1 * Lx + P.spK0 + P.mdTR * ell + P.md2R * Lx * esl + esl * esl;
        W.mt = unif(fmaxf(1.1f * t, P.mdTmin));
    } else {
        // |l| >= lmin; a tile too close to the observer decides nothing in
        // FP32 (mt < 0) and is counted in FP64
        const float lmin = l0 * 0.99999f - M;
        const float i = 1.0f / lmin;
        const float d0 = P.mdN * (2.0f * P.mdFe * i + 0.5f * ell * i * i), d1 = P.mdN * esl * i;
        W.mt = unif(lmin > 0.05f * M && lmin > 16.0f * P.mdFe && d0 < 0.2f ? 1.0f : -1.0f);
        W.mb0 = unif(P.muB0 - 1.001f * d0);
        W.mb1 = unif(P.muB1 - 1.001f * d1);
    }
}

// The tile's home points as the rows of the products: (-2 a, |a|^2), and alpha.
template <int MODE, bool PM>
__device__ __forceinline__ void stage_home(const CountArgs& Pk, WaveState& W, const Tile& tl, int lane) {
    const CountArgs& P = args_again(Pk);   // see next_rows
    tile_origin<kSphere<MODE>>(P, tl, &W.ox, &W.oy, &W.oz);
    const uint32_t i = tl.start + (uint32_t)lane;
    bool ok = i < tl.end;
    if (PM && P.mbA != nullptr && ok) ok = ((P.mbA[i >> 5] >> (i & 31u)) & 1u) == 0u;
    float4 s = make_float4(0.f, 0.f, 0.f, kFar);
    float al = 0.f;
    if constexpr (kMid<MODE>) midpoint_tile<MODE>(P, W);
    if (ok) {
        const float4 p = P.A.p32[i];
        const float x = p.x - W.ox, y = p.y - W.oy, z = p.z - W.oz;
        const double a2 = sq64(x, y, z);
        s = make_float4(-2.0f * x, -2.0f * y, -2.0f * z, (float)a2);
        if constexpr (kMid<MODE>) al = (float)(dot64(W.lx, W.ly, W.lz, x, y, z) + a2);
        if constexpr (MODE == M_RADIAL) al = (float)(P.rA[i] * P.rdA);
    }
    if constexpr (MODE == M_RADIAL) {
        float m = fabsf(al);
        for (int k = 32; k > 0; k >>= 1) m = fmaxf(m, __shfl_xor(m, k));
        W.mt = unif(m);
    }
    wave_lds_fence();
    W.stage[lane] = s;
    if constexpr (kAlpha<MODE>) W.alpha[lane] = al;
    wave_lds_fence();
}

// A chunk's neighbour as a column: b, |b|^2 and -b_z in the four rows;
// midpoint kinds: -beta and 2 beta + |L0|^2; radial: nbeta its negated redshift
// in bins, beta2 the half-width of the band.
struct Column {
    float bx, by, bz;
    f4v b2, nbz, nbeta, beta2;
};

// The arguments that every step reads, in registers. The batched kernels read
// their arguments through a pointer, and the compiler took these up again from
// memory in every step (six loads, each a wait): PIN keeps it from doing so.
struct Hot {
    float s1, e1a, s2, e2a, skip32, muB2, rB0, out_lo, rdIn;
    uint32_t top1, top2, hs1, hs2, rdLow;
};
template <bool PIN>
__device__ __forceinline__ Hot hot_args(const CountArgs& P) {
    Hot h;
    auto f = [](float x) {
        if constexpr (PIN) asm volatile("" : "+s"(x));
        return x;
    };
    auto u = [](uint32_t x) {
        if constexpr (PIN) asm volatile("" : "+s"(x));
        return x;
    };
    h.s1 = f(P.s1);
    h.e1a = f(P.e1a);
    h.s2 = f(P.s2);
    h.e2a = f(P.e2a);
    h.skip32 = f(P.skip32);
    h.muB2 = f(P.muB2);
    h.rB0 = f(P.rB0);
    h.out_lo = f(P.out_lo);
    h.rdIn = P.rdIn;
    h.top1 = u(P.top1);
    h.top2 = u(P.top2);
    h.hs1 = u((uint32_t)P.hs1);
    h.hs2 = u((uint32_t)P.hs2);
    h.rdLow = (uint32_t)P.rdLow;
    return h;
}

// Decision of the lanes' pairs from v = |s|^2 and dz: the lanes whose pair is
// certainly in the bin at LDS address *off (lt: the lanes whose pair is not
// past the top edge). Lane masks throughout: the logic of a step is scalar
// work then.
// r-mu in bin units uses estimates biased by 2^23 + 1: x >= -1/2 then stays
// at or above 2^23, where floats are whole, so the estimate needs no clamp (a
// pair that is in has |x - k| < 1/2 and lies below the top edge, hence k is a
// bin; the offset of any other pair is not used). NaN decides nothing.
// d: dz, or sl for the midpoint kinds; ss: |l|^2 + v for those. Sigma-pi: the
// tables hold one entry past the last bin, for the pairs certainly past the top
// edge; *skip receives the lanes that are (not counted, not ambiguous).
// Radial: d the redshift difference in bins, ss the half-width; the bin counts
// from 2^23 + 1 as for r-mu, *skip receives the lanes certainly outside the bins.
template <int MODE, int EST>
__device__ __forceinline__ uint64_t decide(const Hot& P, const Tab32& T, float v, float d, float ss,
                                           uint64_t lt, uint32_t lb, uint32_t* off, uint64_t* skip) {
    if constexpr (MODE == M_SIGMAPI) {
        const float ll = ss - v;
        const float sl2 = d * d;
        const float c2 = fmaf(v, ll, -sl2);
        // (a c2 rounded below zero gives a NaN estimate, which the clamp puts
        // past the last sigma bin, where its band test fails: re-tested)
        const float rl = __builtin_amdgcn_rsqf(ll);
        const uint32_t ks = est_bits(fmaf(__builtin_amdgcn_sqrtf(c2), rl, P.s1), P.e1a, T, P.top1);
        const uint32_t kp = est_bits(fmaf(fabsf(d), rl, P.s2), P.e2a, T, P.top2);
        const float2 bs = band_at(T.tb1, ks);
        const float2 bp = band_at(T.tb2, kp);
        const uint64_t in =
            __builtin_amdgcn_ballot_w64(fabsf(fmaf(bs.x, ll, c2)) <= fmaf(bs.y, ll, -T.mt)) &
            __builtin_amdgcn_ballot_w64(fabsf(fmaf(bp.x, ll, sl2)) <= fmaf(bp.y, ll, -T.mt)) & lt;
        *off = __umul24(ks, (uint32_t)P.hs1) + (__umul24(kp, (uint32_t)P.hs2) + lb);
        *skip = in & (__builtin_amdgcn_ballot_w64(ks == P.top1) | __builtin_amdgcn_ballot_w64(kp == P.top2));
        return in & ~*skip;
    }
    if constexpr (MODE == M_RADIAL) {
        const float bias1 = __uint_as_float(T.vbias1);
        const float ts = fabsf(d) + P.s1;
        const float e = ts + bias1;
        const uint64_t sure = __builtin_amdgcn_ballot_w64(fabsf(ts + (bias1 - e)) <= ss) & lt;
        uint64_t bin = __builtin_amdgcn_ballot_w64(__float_as_uint(e) < P.top1);
        if (P.rdLow) bin &= __builtin_amdgcn_ballot_w64(__float_as_uint(e) > kBias);
        *off = __umul24(__float_as_uint(e), (uint32_t)P.hs1) + lb;
        *skip = sure & ~bin;
        return sure & bin & __builtin_amdgcn_ballot_w64(v <= P.rdIn);
    }
    float dz = d;
    if constexpr (MODE == M_RMU_MID) dz = d * __builtin_amdgcn_rsqf(ss - v);   // |s.l| / |l|
    if constexpr (MODE == M_MONO || MODE == M_THETA) {
        float e;
        if constexpr (MODE == M_THETA && est_log(EST)) {
            // 2 log2(theta) = log2(v) + v / (12 ln 2) to the order of the
            // table's guess: theta = c + c^3 / 24
            const float t = fmaf(v, 0.12022458674074695f, P.s1 + P.s1);
            e = fmaf(t + __builtin_amdgcn_logf(v), 0.5f * P.e1a, __uint_as_float(T.vbias));
        } else {
            float ts;
            if constexpr (MODE == M_THETA) {
                const float ch = __builtin_amdgcn_sqrtf(v);
                ts = fmaf(ch * v, 1.0f / 24.0f, ch) + P.s1;  // 2 asin(c/2) to third order
            } else if constexpr (est_log(EST)) {
                ts = __builtin_amdgcn_logf(v) + P.s1;
            } else {
                ts = fmaf(v, __builtin_amdgcn_rsqf(v), P.s1);
            }
            e = fmaf(ts, P.e1a, __uint_as_float(T.vbias));
        }
        const uint32_t kb = med3u(__float_as_uint(e), T.vbias, P.top1);
        *off = __umul24(kb, (uint32_t)P.hs1) + lb;
        return __builtin_amdgcn_ballot_w64(in_band(v, band_at(T.tb1, kb)));
    } else {
        const float rinv = __builtin_amdgcn_rsqf(v);
        const float ts = est_log(EST) ? __builtin_amdgcn_logf(v) + P.s1 : fmaf(v, rinv, P.s1);
        const float ts2 = fmaf(fabsf(dz), rinv, P.s2);
        static_assert(MODE == M_SIGMAPI || MODE == M_RADIAL || est_muf(EST),
                      "r-mu with band tables forms its separations component by component");
        const float bias1 = __uint_as_float(T.vbias1);
        const float em = fmaf(ts2, P.e2a, bias1);
        const float half = fmaf(fmaf(P.muB2, rinv, T.d1), rinv, T.d0);
        const uint64_t min_ = __builtin_amdgcn_ballot_w64(fabsf(fmaf(ts2, P.e2a, bias1 - em)) <= half);
        const uint32_t om = __umul24(__float_as_uint(em), (uint32_t)P.hs2) + lb;
        if constexpr (!est_log(EST)) {
            const float er = fmaf(ts, P.e1a, bias1);
            *off = __umul24(__float_as_uint(er), (uint32_t)P.hs1) + om;
            return __builtin_amdgcn_ballot_w64(fabsf(fmaf(ts, P.e1a, bias1 - er)) <= P.rB0) & min_ & lt;
        } else {
            const uint32_t kr = est_bits(ts, P.e1a, T, P.top1);
            *off = __umul24(kr, (uint32_t)P.hs1) + om;
            return __builtin_amdgcn_ballot_w64(in_band(v, band_at(T.tb1, kr))) & min_ & lt;
        }
    }
}

// The histogram address of a decision's estimates starts at the lane's copy
// minus the bias of each estimate that is one above the bin.
template <int MODE, int EST>
__device__ __forceinline__ uint32_t decide_base(const CountArgs& P, uint32_t lb) {
    if constexpr (MODE == M_RADIAL) return lb - (uint32_t)P.hs1;
    if constexpr (est_muf(EST))
        return lb - (uint32_t)P.hs2 - (est_log(EST) ? 0u : (uint32_t)P.hs1);
    return lb;
}

// |s|^2 of four home points against the chunk: the K-th four of the sixteen
// whose rows are in a (in every group of 16 lanes; the instruction broadcasts
// its K-th block to the group), or with K < 0 the four whose rows are in every
// four lanes of a.
template <int K>
__device__ __forceinline__ f4v sep_mfma(const float4& a, const Column& q) {
    constexpr int B = K < 0 ? 0 : 2, I = K < 0 ? 0 : K;
    f4v v = __builtin_amdgcn_mfma_f32_4x4x1f32(a.x, q.bx, q.b2, B, I, 0);
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(a.y, q.by, v, B, I, 0);
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(a.z, q.bz, v, B, I, 0);
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a.w, 1.0f, v, B, I, 0);
}

// Four home points (the K-th of the rows a, home offsets o .. o + 3,
// separations v) against the chunk. Ambiguous pairs go to the wave's list, which has room for all of
// a step's.
template <int MODE, int EST, bool WT, bool MASKED, int K>
__device__ __forceinline__ void step_mfma(const CountArgs& P, const Hot& H, WaveState& W, const Tab32& T, const float4& a,
                                          float al, const f4v& v, const Column& q, bool lmask, uint32_t lj,
                                          uint32_t lb, uint64_t lw, int lane, uint32_t ts,
                                          uint32_t te, uint32_t o) {
    // every pair past the top edge (the clean-out side of its rounding band):
    // nothing to count or re-test
    uint64_t lt[4];
#pragma unroll
    for (int u = 0; u < 4; u++) lt[u] = __builtin_amdgcn_ballot_w64(v[u] < H.skip32);
    if ((lt[0] | lt[1] | lt[2] | lt[3]) == 0ull) return;
    constexpr int B = K < 0 ? 0 : 2, I = K < 0 ? 0 : K;
    f4v d = {0.f, 0.f, 0.f, 0.f}, ss = d;
    if constexpr (kMid<MODE>) {
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(al, 1.0f, q.nbeta, B, I, 0);
        ss = __builtin_amdgcn_mfma_f32_4x4x1f32(al, 2.0f, q.beta2, B, I, 0);
    } else if constexpr (MODE == M_RADIAL) {
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(al, 1.0f, q.nbeta, B, I, 0);
        ss = q.beta2;
    } else if constexpr (MODE == M_RMU_Z) {
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(a.z, -0.5f, q.nbz, B, I, 0);
    }
    uint32_t off[4];
    uint64_t cnt[4], amb[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
        uint64_t skip = 0;
        cnt[u] = decide<MODE, EST>(H, T, v[u], d[u], ss[u], lt[u], lb, &off[u], &skip);
        amb[u] = lt[u] & ~(cnt[u] | skip);
        if constexpr (MASKED) {
            const uint32_t h = ts + o + (uint32_t)u;
            const uint64_t act = __builtin_amdgcn_ballot_w64(!lmask | (lj > h) | ((P.selfx != 0) & (lj < h)));
            cnt[u] &= act;
            amb[u] &= act;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; u++) {
        uint64_t w = lw;
        if constexpr (WT) {
            // (rows past the tile's end are never counted)
            const cu32p wa = (cu32p)(const void*)P.wA;
            const uint32_t i = ts + o + (uint32_t)u;
            w *= wa[i < te ? i : te - 1u];
        }
        if (in_mask(cnt[u])) lds_add<kH32<MODE>>(off[u], w);
    }
    if ((amb[0] | amb[1] | amb[2] | amb[3]) != 0ull) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            // pairs below the first edge are clean (out_lo < 0 without one)
            if (amb[u] == 0ull) continue;
            uint64_t m = amb[u];
            if constexpr (MODE != M_SIGMAPI) {
                m &= ~__builtin_amdgcn_ballot_w64(v[u] < H.out_lo);
            } else if (P.sp_low) {
                const float ll = ss[u] - v[u], sl2 = d[u] * d[u], c2 = fmaf(v[u], ll, -sl2);
                m &= ~(__builtin_amdgcn_ballot_w64(fmaf(P.sp_wsbot, ll, c2) <= -T.mt) |
                       __builtin_amdgcn_ballot_w64(fmaf(P.sp_wpbot, ll, sl2) <= -T.mt));
            }
            const uint32_t pos = lanes_below(m, W.nlist);
            if (in_mask(m)) W.list[pos] = (uint16_t)(((o + (uint32_t)u) << 6) | (uint32_t)lane);
            W.nlist += (uint32_t)__popcll(m);
        }
    }
}

// Move the listed pairs of the chunk at hand (neighbour lj, image lcode in
// each lane) to the re-test queue, draining it whenever 64 are waiting.
template <int MODE, int EST>
__device__ __forceinline__ void queue_list(const CountArgs& P, WaveState& W, const float2* B1,
                                           const float2* B2, const double* T1, const double* T2,
                                           int lane, uint32_t ts, uint32_t lj, uint32_t lcode) {
    wave_lds_fence();
    for (uint32_t i = 0; i < W.nlist; i += 64u) {
        const uint32_t n = W.nlist - i < 64u ? W.nlist - i : 64u;
        const uint32_t e = (uint32_t)lane < n ? (uint32_t)W.list[i + (uint32_t)lane] : 0u;
        const uint32_t j = (uint32_t)__shfl((int)lj, (int)(e & 63u));
        const uint32_t c = (uint32_t)__shfl((int)lcode, (int)(e & 63u));
        if ((uint32_t)lane < n) {
            const uint32_t pos = W.tail + (uint32_t)lane;
            W.qi[pos] = ts + (e >> 6);
            W.qj[pos] = j;
            W.qc[pos] = (uint8_t)c;
        }
        W.tail += n;
        wave_lds_fence();
        if (W.tail >= 64u)
            W.tail = drain_queue<MODE, EST>(P.self, W.hist, W.qi, W.qj, W.qc, W.rstat, B1, B2, T1, T2,
                                            lane, W.tail, false);
    }
    W.nlist = 0;
}

// The canonical FP64 bin of a pair when a guess from FP32 holds: the edges
// around the guessed bin are compared once, without a search. False when the
// guess is off by a bin, at zero separation and in the closed last mu edge: the
// pair then goes through classify64, so that a search costs a step nothing
// unless one of its pairs needs it. (The predicates are those of classify64:
// the products with the squared mu edges grow with the edge, so a pair between
// two of them has no larger edge below it.) With the search in every step, the
// 1.8e9 candidate pairs of an r-mu count of 4e5 points cost 50 VALU instructions
// each and 2.9 ms; they cost 24 and 1.6 ms. VALU bound (78 % busy), beside LDS
// reads of the edges (57 %).
struct EdgePair {
    double lo, hi;
};
__device__ __forceinline__ EdgePair edges_at(uint32_t base, uint32_t kb) {
    typedef const __attribute__((address_space(3))) double* lds_dp;
    const lds_dp p = (lds_dp)(uintptr_t)((kb << 3) + base);
    EdgePair e;
    e.lo = p[0];
    e.hi = p[1];
    return e;
}
template <int MODE, int EST>
__device__ __forceinline__ bool guessed64(const CountArgs& P, const Tab32& T, double dz, double d2, uint32_t* bin) {
    const float v = (float)d2;
    const float rinv = __builtin_amdgcn_rsqf(v);
    float ts;
    if constexpr (MODE == M_THETA) {
        const float c = v * rinv;
        const float th = fmaf(c * v, 1.0f / 24.0f, c);  // 2 asin(c/2) to third order
        ts = (est_log(EST) ? __builtin_amdgcn_logf(th) : th) + P.s1;
    } else {
        ts = est_log(EST) ? __builtin_amdgcn_logf(v) + P.s1 : fmaf(v, rinv, P.s1);
    }
    const uint32_t k1 = est_bits(ts, P.e1a, T, kBias + (uint32_t)(P.n1 - 1));
    const EdgePair e = edges_at(T.tb1, k1);
    bool ok = (e.lo <= d2) & (d2 < e.hi);
    if constexpr (MODE == M_RMU_Z) {
        const uint32_t k2 = est_bits(fmaf(fabsf((float)dz), rinv, P.s2), P.e2a, T, kBias + (uint32_t)(P.n2 - 1));
        const EdgePair m = edges_at(T.tb2, k2);
        const double num = dz * dz;
        ok = ok & (num >= m.lo * d2) & (num < m.hi * d2);
        *bin = __umul24(k1, (uint32_t)P.hs1) + __umul24(k2, (uint32_t)P.hs2);
    } else {
        *bin = __umul24(k1, (uint32_t)P.hs1);
    }
    return ok;
}

template <int MODE, int EST, bool PM, bool WT, bool MASKED, bool SHIFTED, uint32_t U>
__device__ __forceinline__ void step64(const CountArgs& P, WaveState& W, const double* T1,
                                       const double* T2, int lane, bool lvalid, bool lmask,
                                       uint32_t lj, double qx, double qy, double qz, double sx, double sy,
                                       double sz, uint64_t lw, uint32_t h, double qr,
                                       const Tab32& T, uint32_t lb) {
    double hx[U], hy[U], hz[U];
    load_points64<U>(P.A.p64, h, hx, hy, hz);
    bool hv[U];
    home_valid<PM, U>(P, h, hv);
    uint32_t hw[U];
    home_weights<WT, U>(P, h, hw);
    {
        // every pair of the step at or past the top threshold (exact FP64)
        double dmin = 0.0;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            double dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
            if (SHIFTED) {
                dx = dx - sx;
                dy = dy - sy;
                dz = dz - sz;
            }
            const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
            dmin = u == 0 ? d2 : fmin(dmin, d2);
        }
        if (__builtin_amdgcn_ballot_w64(dmin < P.top64) == 0ull) return;
    }
    if constexpr (MODE == M_MONO || MODE == M_THETA || MODE == M_RMU_Z) {
        uint32_t off[U];
        bool cnt[U], amb[U], any = false;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            double dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
            if (SHIFTED) {
                dx = dx - sx;
                dy = dy - sy;
                dz = dz - sz;
            }
            const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
            bool act = lvalid & hv[u] & (d2 < P.top64);
            if constexpr (MASKED) act = act & (!lmask | (lj > h + u) | ((P.selfx != 0) & (lj < h + u)));
            const bool ok = guessed64<MODE, EST>(P, T, dz, d2, &off[u]);
            cnt[u] = act & ok;
            amb[u] = act & !ok;
            any = any | amb[u];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; u++)
            if (cnt[u]) lds_add<kH32<MODE>>(off[u] + lb, WT ? lw * hw[u] : lw);
        if (__builtin_amdgcn_ballot_w64(any) == 0ull) return;
        // The misses. Edges that no guess fits miss in nearly every step, so the
        // one-variable kinds search unrolled (the loop below selects a pair's
        // home point among four: uneven angular bins 9.40 ms so, 8.24 unrolled;
        // the r-mu kernel, with twice the search, gains nothing from it).
        if constexpr (MODE != M_RMU_Z) {
#pragma unroll
            for (uint32_t u = 0; u < U; u++) {
                if (!amb[u]) continue;
                double dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
                if (SHIFTED) {
                    dx = dx - sx;
                    dy = dy - sy;
                    dz = dz - sz;
                }
                const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
                const int k1 = guess1<MODE == M_THETA ? M_THETA : M_MONO, EST>(P, (float)d2);
                const uint32_t bin = classify64<MODE>(P, T1, T2, dx, dy, dz, 0.0, 0.0, 0.0, k1, 0);
                if (bin != kNoBin)
                    hist_add<kH32<MODE>>(W.hist, bin, P.copies, lane, WT ? lw * hw[u] : lw);
            }
        } else {
#pragma unroll 1
            for (uint32_t u = 0; u < U; u++) {
                bool a = false;
                double x = 0.0, y = 0.0, z = 0.0;
                uint32_t w = 1u;
#pragma unroll
                for (uint32_t t = 0; t < U; t++)
                    if (t == u) {
                        a = amb[t];
                        x = hx[t];
                        y = hy[t];
                        z = hz[t];
                        w = hw[t];
                    }
                if (!a) continue;
                double dx = x - qx, dy = y - qy, dz = z - qz;
                if (SHIFTED) {
                    dx = dx - sx;
                    dy = dy - sy;
                    dz = dz - sz;
                }
                const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
                const float v = (float)d2;
                const int k1 = guess1<M_MONO, EST>(P, v);
                const int k2 =
                    guess_lin(fabsf((float)dz) * __builtin_amdgcn_rsqf(v), P.e2a, P.e2b, P.n2m1);
                const uint32_t bin = classify64<MODE>(P, T1, T2, dx, dy, dz, 0.0, 0.0, 0.0, k1, k2);
                if (bin != kNoBin)
                    hist_add<kH32<MODE>>(W.hist, bin, P.copies, lane, WT ? lw * w : lw);
            }
        }
        return;
    }
    double hr[U];
    if constexpr (MODE == M_RADIAL) {
        const cdp ra = (cdp)(const void*)P.rA;
#pragma unroll
        for (uint32_t u = 0; u < U; u++) hr[u] = ra[h + u];
    }
    uint32_t bin[U];
    bool cnt[U];
#pragma unroll
    for (uint32_t u = 0; u < U; u++) {
        const bool act = lvalid & hv[u] &
                         (!MASKED | !lmask | (lj > h + u) | ((P.selfx != 0) & (lj < h + u)));
        double dx = hx[u] - qx, dy = hy[u] - qy, dz = hz[u] - qz;
        if (SHIFTED) {
            // the neighbour's periodic image: equal to the minimum-image wrap
            // for every pair the stencil can form
            dx = dx - sx;
            dy = dy - sy;
            dz = dz - sz;
        }
        double lx = 0.0, ly = 0.0, lz = 0.0;
        if (MODE == M_RMU_MID || MODE == M_SIGMAPI) {
            lx = hx[u] + qx;
            ly = hy[u] + qy;
            lz = hz[u] + qz;
        }
        int k1 = 0, k2 = 0;
        const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
        if constexpr (MODE == M_RADIAL) {
            bin[u] = classify_radial(P, T1, d2, fabs(hr[u] - qr));
            cnt[u] = act & (bin[u] != kNoBin);
            continue;
        }
        const float v = (float)d2;
        if (MODE == M_RMU_MID) {
            k1 = guess1<M_MONO, EST>(P, v);
            const float sl = (float)fma(dz, lz, fma(dy, ly, dx * lx));
            const float ll = (float)fma(lz, lz, fma(ly, ly, lx * lx));
            k2 = guess_lin(fabsf(sl) * __builtin_amdgcn_rsqf(v * ll), P.e2a, P.e2b, P.n2m1);
        } else {
            const float sl = (float)fma(dz, lz, fma(dy, ly, dx * lx));
            const float ll = (float)fma(lz, lz, fma(ly, ly, lx * lx));
            const float pi2 = sl * sl * __builtin_amdgcn_rcpf(ll);
            k1 = guess_lin(__builtin_amdgcn_sqrtf(fmaxf(v - pi2, 0.0f)), P.e1a, P.e1b, P.n1m1);
            k2 = guess_lin(__builtin_amdgcn_sqrtf(pi2), P.e2a, P.e2b, P.n2m1);
        }
        bin[u] = classify64<MODE>(P, T1, T2, dx, dy, dz, lx, ly, lz, k1, k2);
        cnt[u] = act & (bin[u] != kNoBin);
    }
#pragma unroll
    for (uint32_t u = 0; u < U; u++)
        if (cnt[u]) hist_add<kH32<MODE>>(W.hist, bin[u], P.copies, lane, WT ? lw * hw[u] : lw);
}

// The chunk being assembled from neighbour spans (per-lane fields in VGPRs,
// the rest wave-uniform).
struct Chunk {
    uint32_t filled;   // lanes holding a neighbour
    bool masked;       // some lane needs the j > i test
    bool shifted;      // some lane holds a periodic image
    uint32_t lj;       // per lane: neighbour index
    uint32_t lcode;    // per lane: image code | kSelfSpan
};

// What a chunk's lanes load of their neighbours, a chunk ahead: the FP32 point,
// the redshift (radial), the point weight (pixel maps) or region (region
// passes), the word of the point mask. (Loaded where they are used, the
// regions alone cost the region pass the whole latency of every chunk's loads:
// loads return in order.)
struct Near {
    float4 p;
    double r;
    uint32_t w, mask;
};
template <int MODE, bool PM, bool WT>
__device__ __forceinline__ void load_near(const CountArgs& P, Near& n, uint32_t j) {
    n.p = P.B.p32[j];
    if constexpr (MODE == M_RADIAL) n.r = P.rB[j];
    if constexpr (WT) n.w = P.wB[j];
    else if (PM && P.regs != nullptr) n.w = P.regs[j];
    if (PM && P.mbB != nullptr) n.mask = P.mbB[j >> 5];
}

// A chunk against the tile's staged home points. p: the lanes' neighbours. The separations of a step are formed while the
// step before it is decided, so that their chain of dependent instructions
// does not wait in the open.
template <int MODE, int EST, bool PM, bool WT>
__device__ __forceinline__ void run_chunk_mfma(const CountArgs& P, const Hot& H, WaveState& W, const Tab32& T,
                                               const float2* B1, const float2* B2, const double* T1,
                                               const double* T2, int lane, const Chunk& C,
                                               const Near& p, uint32_t ts, uint32_t te) {
    if constexpr (kH32<MODE>) {
        // every pair of the chunk adds at most the largest region weight
        const uint32_t wmax = !PM || P.regs == nullptr ? 1u : (uint32_t)(P.wsame > P.wdiff ? P.wsame : P.wdiff);
        h32_account(P, W, lane, C.filled * (te - ts) * wmax);
    } else if (PM && P.counts_hi != nullptr) {
        h32_account<true>(P, W, lane, C.filled * (te - ts));
    }
    bool ok = (uint32_t)lane < C.filled;
    // a neighbour excluded by the point mask leaves its lane idle
    if (PM && P.mbB != nullptr) ok = ok && ((p.mask >> (C.lj & 31u)) & 1u) == 0u;
    uint64_t lw = 1u;
    if constexpr (WT) lw = p.w;
    else if (PM && P.regs != nullptr) lw = p.w == (uint32_t)P.region ? P.wsame : P.wdiff;
    const bool self = (C.lcode & kSelfSpan) != 0u;
    // the neighbour in the home grid's FP32 frame (q - (cA - cB) for two open
    // grids, or its periodic image q + k L: only one of the two is ever
    // non-zero), then in the tile's
    float kx = P.offx, ky = P.offy, kz = P.offz;
    if (C.shifted) {
        const float Lf = (float)P.L;
        kx -= shift32(C.lcode, 0, Lf);
        ky -= shift32(C.lcode, 1, Lf);
        kz -= shift32(C.lcode, 2, Lf);
    }
    Column q;
    q.bx = ok ? (p.p.x - kx) - W.ox : 0.f;
    q.by = ok ? (p.p.y - ky) - W.oy : 0.f;
    q.bz = ok ? (p.p.z - kz) - W.oz : 0.f;
    const double b2d = sq64(q.bx, q.by, q.bz);
    const float b2 = ok ? (float)b2d : kFar;
    q.b2 = f4v{b2, b2, b2, b2};
    if constexpr (kMid<MODE>) {
        const double beta = dot64(W.lx, W.ly, W.lz, q.bx, q.by, q.bz) + b2d;
        const float nb = (float)-beta, be = (float)fma(2.0, beta, sq64(W.lx, W.ly, W.lz));
        q.nbeta = f4v{nb, nb, nb, nb};
        q.beta2 = f4v{be, be, be, be};
    } else if constexpr (MODE == M_RADIAL) {
        const float w = ok ? (float)(p.r * P.rdA) : 0.f;
        const float half = fmaf(-3.5f * 0x1p-24f, W.mt + fabsf(w), P.rB0);
        q.nbeta = f4v{-w, -w, -w, -w};
        q.beta2 = f4v{half, half, half, half};
    } else {
        q.nbz = f4v{-q.bz, -q.bz, -q.bz, -q.bz};
    }
    // this lane's histogram copy
    const uint32_t lb = decide_base<MODE, EST>(
        P, lds_addr(W.hist) + ((uint32_t)lane & (uint32_t)(P.copies - 1)) * (kH32<MODE> ? 4u : 8u));
    const uint32_t n = te - ts;
    uint32_t o = 0;
#define CUTE_STEP(K)                                                                               \
    {                                                                                              \
        const f4v w = sep_mfma<(K + 1) & 3>(K == 3 ? an : a, q);                                   \
        step_mfma<MODE, EST, WT, false, K>(P, H, W, T, a, al, v, q, false, 0u, lb, lw, lane, ts, te, o); \
        v = w;                                                                                     \
        o += 4u;                                                                                   \
        if (o >= n || W.nlist > kList - 256u) break;                                               \
    }
    while (o < n) {
        if (!C.masked && (o & 15u) == 0u) {
            // Sixteen home points per read of the stage: the wait for a read
            // is also one for the histogram adds before it (one counter, in
            // order), and with a read per step it stood open in every step.
            const float4* row = W.stage + (lane & 15);
            const float* arow = W.alpha + (lane & 15);
            float4 a = row[o];
            float al = kAlpha<MODE> ? arow[o] : 0.f;
            f4v v = sep_mfma<0>(a, q);
            for (;;) {
                const float4 an = row[(o + 16u) & 48u];
                const float aln = kAlpha<MODE> ? arow[(o + 16u) & 48u] : 0.f;
                CUTE_STEP(0)
                CUTE_STEP(1)
                CUTE_STEP(2)
                CUTE_STEP(3)
                a = an;
                al = aln;
            }
        } else {
            // chunks with the index test, and what is left of sixteen home
            // points after the list was moved
            const float4* row = W.stage + (lane & 3);
            do {
                const float4 a = row[o];
                const float al = kAlpha<MODE> ? W.alpha[o + (uint32_t)(lane & 3)] : 0.f;
                step_mfma<MODE, EST, WT, true, -1>(P, H, W, T, a, al, sep_mfma<-1>(a, q), q, self,
                                                   C.lj, lb, lw, lane, ts, te, o);
                o += 4u;
            } while (o < n && W.nlist <= kList - 256u && (C.masked || (o & 15u) != 0u));
        }
        // a step adds at most 256 pairs to the list: it is moved to the queue
        // when it could not take another step's, and at the chunk's end
        if (W.nlist > kList - 256u || (o >= n && W.nlist != 0u))
            queue_list<MODE, EST>(P, W, B1, B2, T1, T2, lane, ts, C.lj, C.lcode);
    }
#undef CUTE_STEP
}

template <int MODE, int PREC, int EST, bool PM, bool WT>
__device__ void run_chunk(const CountArgs& P, WaveState& W, const float2* B1, const float2* B2,
                          const double* T1, const double* T2, int lane, const Chunk& C, uint32_t ts,
                          uint32_t te) {
    constexpr uint32_t U = 4;
    if constexpr (kH32<MODE>) {
        // every pair of the chunk adds at most the largest region weight
        const uint32_t wmax = !PM || P.regs == nullptr ? 1u : (uint32_t)(P.wsame > P.wdiff ? P.wsame : P.wdiff);
        h32_account(P, W, lane, C.filled * (te - ts) * wmax);
    } else if (PM && P.counts_hi != nullptr) {
        h32_account<true>(P, W, lane, C.filled * (te - ts));
    }
    bool lvalid = (uint32_t)lane < C.filled;
    // a neighbour excluded by the point mask leaves its lane idle
    if (PM && P.mbB != nullptr && lvalid) lvalid = ((P.mbB[C.lj >> 5] >> (C.lj & 31u)) & 1u) == 0u;
    const uint64_t lw = lvalid ? (WT ? P.wB[C.lj] : PM ? pair_weight(P, C.lj) : 1u) : 1u;
    const bool self = (C.lcode & kSelfSpan) != 0u;
    if constexpr (PREC == P_FP64) {
        double qx = 0.0, qy = 0.0, qz = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, qr = 0.0;
        // the tables here are the canonical edges, and this lane's histogram copy
        Tab32 tab = make_tab32<EST>(P, B1, B2);
        tab.tb1 = lds_addr(T1) - (kBias << 3);
        tab.tb2 = lds_addr(T2) - (kBias << 3);
        const uint32_t lb = lds_addr(W.hist) +
                            ((uint32_t)lane & (uint32_t)(P.copies - 1)) * (kH32<MODE> ? 4u : 8u);
        if (MODE == M_RADIAL && lvalid) qr = P.rB[C.lj];
        if (lvalid) {
            const P64 q = P.B.p64[C.lj];
            qx = q.x;
            qy = q.y;
            qz = q.z;
            sx = shift64(C.lcode, 0, P.L);
            sy = shift64(C.lcode, 1, P.L);
            sz = shift64(C.lcode, 2, P.L);
        }
#define CUTE_RUN64(MSK, SH)                                                                     \
    {                                                                                           \
        uint32_t h = ts;                                                                        \
        for (; h + U <= te; h += U)                                                             \
            step64<MODE, EST, PM, WT, MSK, SH, U>(P, W, T1, T2, lane, lvalid, self, C.lj, qx, qy, qz, \
                                          sx, sy, sz, lw, h, qr, tab, lb);                               \
        for (; h < te; h++)                                                                     \
            step64<MODE, EST, PM, WT, MSK, SH, 1>(P, W, T1, T2, lane, lvalid, self, C.lj, qx, qy, qz, \
                                          sx, sy, sz, lw, h, qr, tab, lb);                               \
    }
        if (C.masked) {
            if (C.shifted) CUTE_RUN64(true, true) else CUTE_RUN64(true, false)
        } else {
            if (C.shifted) CUTE_RUN64(false, true) else CUTE_RUN64(false, false)
        }
#undef CUTE_RUN64
    } else {
        // wave-uniform constants in VGPRs, and this lane's histogram copy
        const Tab32 tab = make_tab32<EST>(P, B1, B2);
        const uint32_t lb = lds_addr(W.hist) +
                            ((uint32_t)lane & (uint32_t)(P.copies - 1)) * (kH32<MODE> ? 4u : 8u);
        // the neighbour in the home grid's FP32 frame: q - (cA - cB) for two
        // open grids, or its periodic image q + k L (only one of the two is
        // ever non-zero), and q + 2 cA for the midpoint line of sight
        float qx = 0.f, qy = 0.f, qz = 0.f, qlx = 0.f, qly = 0.f, qlz = 0.f;
        if (lvalid) {
            const float4 q = P.B.p32[C.lj];
            const float Lf = (float)P.L;
            qx = q.x - (P.offx - shift32(C.lcode, 0, Lf));
            qy = q.y - (P.offy - shift32(C.lcode, 1, Lf));
            qz = q.z - (P.offz - shift32(C.lcode, 2, Lf));
            qlx = qx + P.lcx;
            qly = qy + P.lcy;
            qlz = qz + P.lcz;
        }
        // ambiguous pairs of this chunk: per lane, bit (home - ts); per wave,
        // the home offsets with any (queued once the home loop is done)
        uint64_t ambh = 0, hsum = 0;
        // bins starting at zero separation have no low-side clean "out"
        const bool low = MODE == M_SIGMAPI ? P.sp_low != 0 : !(P.out_lo < 0.0f);
#define CUTE_RUN32(MSK, LOW)                                                                     \
    {                                                                                              \
        uint32_t h = ts;                                                                           \
        for (; h + U <= te; h += U)                                                                \
            step32<MODE, PREC, EST, PM, WT, MSK, LOW, U>(P, W, tab, B1, B2, T1, T2, lane, lvalid,  \
                                                     self, C.lj, C.lcode, qx, qy, qz, qlx, qly, \
                                                     qlz, lb, lw, ts, ambh, hsum, h);              \
        for (; h < te; h++)                                                                        \
            step32<MODE, PREC, EST, PM, WT, MSK, LOW, 1>(P, W, tab, B1, B2, T1, T2, lane, lvalid,  \
                                                     self, C.lj, C.lcode, qx, qy, qz, qlx, qly, \
                                                     qlz, lb, lw, ts, ambh, hsum, h);              \
    }
        if (C.masked) {
            if (low) CUTE_RUN32(true, true) else CUTE_RUN32(true, false)
        } else {
            if (low) CUTE_RUN32(false, true) else CUTE_RUN32(false, false)
        }
        if (PREC == P_FP32E && hsum != 0ull)
            W.tail = enqueue_chunk<MODE, EST>(P.self, W.hist, W.qi, W.qj, W.qc, W.rstat, B1, B2, T1,
                                              T2, lane, W.tail, ts, C.lj, C.lcode, ambh, hsum);
#undef CUTE_RUN32
    }
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
__device__ __forceinline__ int imod(int a, int n) {
    int r = a % n;
    return r < 0 ? r + n : r;
}

// Span list of one batch of stencil rows (in LDS) and where the walk over a
// tile's neighbours stands (wave-uniform).
struct SpanBuf {
    uint2* e;      // position of the span's first neighbour in the concatenation of the
                   // batch's spans, and that neighbour's index minus this position
    uint8_t* f;    // image code | kSelfSpan
    int nrows, row0;   // rows of the stencil, first row not taken yet
    uint32_t n, k;     // spans of the batch, the one at hand
    uint32_t pos, end; // positions not taken yet
    uint32_t own;      // the j > i test applies to positions below it
};
__device__ __forceinline__ SpanBuf span_buf(const WgLds& l, int wave) {
    SpanBuf S;
    S.e = reinterpret_cast<uint2*>(l.spans + (size_t)wave * 2 * kSpanCap);
    S.f = l.scodes + (size_t)wave * kSpanCap;
    S.nrows = S.row0 = 0;
    S.n = S.k = S.pos = S.end = S.own = 0u;
    return S;
}

// The stencil of one tile (Sec. 3.3: the rows of cells within r_max of it),
// wave-uniform: how many rows to look at, and what the rows of each kind of
// grid need.
struct TileStencil {
    uint32_t ts, te;
    int c0, c1, cy, cz;
    int nrows;
    // SPHERE: first band, the phi range of every band, or the whole ring
    int b0, x0, x1;
    bool full;
    // 3-D boxes without a row table: the rows' rectangle and the tile's box
    int y0, z0, nyr;
    double xlo, xhi, ylo, yhi, zlo, zhi;
};

// SPH: spherical grids (their kernels hold no code of the boxes, and the
// other way round: the trigonometry alone set the registers of every kernel)
template <bool SPH>
__device__ __forceinline__ TileStencil tile_stencil(const CountArgs& P, const Tile& tl) {
    const GridView& A = P.A;
    const GridView& B = P.B;
    TileStencil t;
    t.ts = tl.start;
    t.te = tl.end;
    t.c0 = (int)(tl.c0c1 & 0xffffu);
    t.c1 = (int)(tl.c0c1 >> 16);
    t.cy = (int)(tl.row % (uint32_t)A.ny);
    t.cz = (int)(tl.row / (uint32_t)A.ny);
    t.nrows = t.b0 = t.x0 = t.x1 = t.y0 = t.z0 = t.nyr = 0;
    t.full = false;
    t.xlo = t.xhi = t.ylo = t.yhi = t.zlo = t.zhi = 0.0;
    if constexpr (SPH) {
        // tile pixel block: phi in [c0, c1+1) * ax, cos theta in one band; the
        // band's reach (first and last band, half-width in phi, negative for
        // whole rings) comes from the host's table
        const cu32p st = (cu32p)(const void*)P.stencil + 4 * (size_t)t.cy;
        const int b0 = (int)uni(st[0]), b1 = (int)uni(st[1]);
        const double hw = __hiloint2double((int)uni(st[3]), (int)uni(st[2]));
        // an autocorrelation takes its own band and the ones after it
        t.b0 = P.is_auto && b0 < t.cy ? t.cy : b0;
        const double phlo = t.c0 * A.ax - hw, phhi = (t.c1 + 1) * A.ax + hw;
        t.x0 = unii((int)floor(phlo / B.ax) - 1);
        t.x1 = unii((int)floor(phhi / B.ax) + 1);
        t.full = unii((hw < 0.0 || t.x1 - t.x0 + 1 >= B.nx) ? 1 : 0) != 0;
        t.nrows = b1 - t.b0 + 1;
    } else if (P.stencil != nullptr) {
        t.nrows = P.nst;
    } else {
        // the tile box, grown by R, selects rows of neighbour cells
        const double R = P.Rs;
        t.xlo = A.ox + t.c0 * A.ax;
        t.xhi = A.ox + (t.c1 + 1) * A.ax;
        t.ylo = A.oy + t.cy * A.ay;
        t.yhi = t.ylo + A.ay;
        t.zlo = A.oz + t.cz * A.az;
        t.zhi = t.zlo + A.az;
        int y0 = (int)floor((t.ylo - R - B.oy) / B.ay), y1 = (int)floor((t.yhi + R - B.oy) / B.ay);
        int z0 = (int)floor((t.zlo - R - B.oz) / B.az), z1 = (int)floor((t.zhi + R - B.oz) / B.az);
        if (!P.periodic) {
            y0 = clampi(y0, 0, B.ny - 1);
            y1 = clampi(y1, 0, B.ny - 1);
            z0 = clampi(z0, 0, B.nz - 1);
            z1 = clampi(z1, 0, B.nz - 1);
        }
        t.y0 = unii(y0);
        t.z0 = unii(z0);
        t.nyr = unii(y1) - t.y0 + 1;
        t.nrows = t.nyr * (unii(z1) - t.z0 + 1);
    }
    return t;
}

// One stencil row (per lane): at most two pieces of its x-range (a periodic
// or phi wrap cuts it once), as neighbour index ranges [a0, a1) and [b0, b1)
// with their image codes. home: the tile's own row, whose part inside the
// tile is a span of its own with the index test: m1 is the end of that span
// [ts, m1) (0 = none), and [h0, h1) the rest of the row past the tile where
// the pieces do not hold it (full stencils).
struct RowSpans {
    uint32_t a0, a1, b0, b1, ca, cb;
    uint32_t m1, h0, h1;
};

// Row e of the tile's stencil, e < t.nrows (any lane value).
template <bool SPH>
__device__ __forceinline__ RowSpans row_spans(const CountArgs& P, const TileStencil& t, int e) {
    const GridView& B = P.B;
    RowSpans r;
    r.a0 = r.a1 = r.b0 = r.b1 = 0u;
    r.ca = r.cb = kNoShift;
    r.m1 = r.h0 = r.h1 = 0u;
    // the row's cells [pa, pb] and, past a wrap, [qa, qb]; empty when pb < pa
    int pa = 0, pb = -1, qa = 0, qb = -1;
    uint32_t rb = 0u;
    bool same = false;   // the tile's own row of an autocorrelation
    bool home = false;   // the tile's own row of a full stencil over one catalog
    int kxa = 0, kxb = 0, ky = 0, kz = 0;
    if constexpr (SPH) {
        const int by = t.b0 + e;
        rb = (uint32_t)by * (uint32_t)B.nx;
        same = P.is_auto && by == t.cy;
        if (same) {
            // index rule inside the home band: partners with a larger index,
            // i.e. cells >= c0 up to the right reach, plus the left reach
            // that wraps past phi = 2 pi onto the band's last cells
            pa = t.c0;
            pb = B.nx - 1;
            if (!t.full) {
                const int r1 = t.x1 < B.nx - 1 ? t.x1 : B.nx - 1;
                const int s2 = t.x0 < 0 ? t.x0 + B.nx : B.nx;
                if (s2 > r1 + 1) {
                    pb = r1;
                    qa = s2;
                    qb = B.nx - 1;
                }
            }
        } else if (t.full) {
            pb = B.nx - 1;
        } else {
            // cyclic range [x0, x1] (length < nx) split at the phi wrap
            pa = imod(t.x0, B.nx);
            pb = pa + (t.x1 - t.x0);
            if (pb > B.nx - 1) {
                qb = pb - B.nx;
                pb = B.nx - 1;
            }
        }
    } else {
        int by, bz, x0, x1;
        bool ok = true;
        if (P.stencil != nullptr) {
            // 3-D boxes of one geometry: the rows are precomputed offsets
            const int4 o = P.stencil[e];
            by = t.cy + o.x;
            bz = t.cz + o.y;
            same = P.is_auto && o.x == 0 && o.y == 0;
            home = P.selfx && o.x == 0 && o.y == 0;
            x0 = same ? t.c0 : t.c0 - o.z;
            x1 = t.c1 + o.w;
            // never more than one full turn of the row
            if (P.periodic) x1 = x1 < x0 + B.nx - 1 ? x1 : x0 + B.nx - 1;
        } else {
            bz = t.z0 + e / t.nyr;
            by = t.y0 + e % t.nyr;
            if (P.is_auto) {
                const int oz_ = bz - t.cz, oy_ = by - t.cy;
                if (oz_ < 0 || (oz_ == 0 && oy_ < 0)) ok = false;
                same = (oz_ == 0 && oy_ == 0);
            }
            // distance in y and z between the tile box and this row of cells
            const double R2 = P.Rs * P.Rs;
            const double rylo = B.oy + by * B.ay, ryhi = rylo + B.ay;
            const double rzlo = B.oz + bz * B.az, rzhi = rzlo + B.az;
            const double dy = fmax(0.0, fmax(rylo - t.yhi, t.ylo - ryhi));
            const double dz = fmax(0.0, fmax(rzlo - t.zhi, t.zlo - rzhi));
            const double rem = R2 - dy * dy - dz * dz;
            if (rem <= 0.0) ok = false;
            const double w = sqrt(fmax(rem, 0.0));
            x0 = (int)floor((t.xlo - w - B.ox) / B.ax);
            x1 = (int)floor((t.xhi + w - B.ox) / B.ax);
            if (same && x0 < t.c0) x0 = t.c0;
        }
        int ry = by, rz = bz;
        if (P.periodic) {
            ky = floordiv(by, B.ny);
            kz = floordiv(bz, B.nz);
            ry = by - ky * B.ny;
            rz = bz - kz * B.nz;
        } else {
            if (by < 0 || by >= B.ny || bz < 0 || bz >= B.nz) ok = false;
            x0 = x0 < 0 ? 0 : x0;
            x1 = x1 > B.nx - 1 ? B.nx - 1 : x1;
        }
        if (!ok || x0 > x1) return r;
        rb = (uint32_t)B.nx * ((uint32_t)ry + (uint32_t)B.ny * (uint32_t)rz);
        // [x0, x1], cut at a periodic wrap (at most two pieces)
        if (P.periodic) {
            kxa = floordiv(x0, B.nx);
            kxb = kxa + 1;
            const int lim = kxb * B.nx - 1;
            pa = x0 - kxa * B.nx;
            pb = (x1 < lim ? x1 : lim) - kxa * B.nx;
            qb = x1 - kxb * B.nx;
        } else {
            pa = x0;
            pb = x1;
        }
    }
    const uint32_t* cs = B.cstart;
    if (pb >= pa) {
        r.a0 = cs[rb + (uint32_t)pa];
        r.a1 = cs[rb + (uint32_t)pb + 1u];
    }
    if (qb >= qa) {
        r.b0 = cs[rb + (uint32_t)qa];
        r.b1 = cs[rb + (uint32_t)qb + 1u];
    }
    // (no images on the sphere: kx, ky and kz are 0)
    r.ca = (uint32_t)(kxa + 1) | ((uint32_t)(ky + 1) << 2) | ((uint32_t)(kz + 1) << 4);
    r.cb = (uint32_t)(kxb + 1) | ((uint32_t)(ky + 1) << 2) | ((uint32_t)(kz + 1) << 4);
    if (same) {
        // points of the first cell before the tile pair with it from their
        // own tile; the tile's points pair among themselves (j > i) and with
        // the rest of the row
        r.m1 = t.te < r.a1 ? t.te : r.a1;
        r.a0 = t.te;
    } else if (home) {
        // the tile's points pair with all of their row but themselves: the
        // piece that holds the tile ends before it, the rest follows it
        if (kxa == 0 && pa <= t.c0 && t.c1 <= pb) {
            r.m1 = t.te;
            r.h0 = t.te;
            r.h1 = r.a1;
            r.a1 = t.ts;
        } else if (kxb == 0 && qa <= t.c0 && t.c1 <= qb) {
            r.m1 = t.te;
            r.h0 = t.te;
            r.h1 = r.b1;
            r.b1 = t.ts;
        }
    }
    return r;
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)v, o);
        v += lane >= o ? u : 0u;
    }
    return v;
}

// The spans of the next kRowBatch stencil rows of a tile, one row per lane (a serial
// walk of the rows spent more time on dependent loads than the pairs of a
// small tile take), compacted to LDS in row order. Of their concatenated
// neighbours a part takes a run of whole chunks, so that the parts of a tile
// share out its chunks evenly.
template <bool SPH>
__device__ __forceinline__ void next_rows(const CountArgs& Pk, WaveState& W, SpanBuf& S, const Tile& tl,
                                          int lane, uint32_t part, uint32_t plog) {
    // the stencil again for every batch of rows, from the arguments' copy in
    // memory: nothing of it is live while pairs are evaluated (the asm keeps
    // the compiler from loading or deriving it ahead of the walk, where it
    // would fill the registers of the pair loop)
    const CountArgs& P = args_again(Pk);
    Tile tb = tl;
    tb.row = uni(tb.row);
    asm volatile("" : "+s"(tb.row));
    const TileStencil t = tile_stencil<SPH>(P, tb);
    S.nrows = t.nrows;
    RowSpans r;
    r.a0 = r.a1 = r.b0 = r.b1 = r.m1 = r.h0 = r.h1 = 0u;
    r.ca = r.cb = kNoShift;
    if (lane < kRowBatch && S.row0 + lane < t.nrows) r = row_spans<SPH>(P, t, S.row0 + lane);
    S.row0 += kRowBatch;
    S.pos = S.end = S.own = 0u;
    const uint32_t na = r.a1 > r.a0 ? r.a1 - r.a0 : 0u, nb = r.b1 > r.b0 ? r.b1 - r.b0 : 0u;
    // the tile's own spans, from the lane that holds its row
    const uint64_t mh = __builtin_amdgcn_ballot_w64(r.m1 != 0u);
    uint32_t m1 = 0u, h0 = 0u, h1 = 0u;
    if (mh != 0ull) {
        const int l = __builtin_ctzll(mh);
        m1 = lane_u32(r.m1, l);
        h0 = lane_u32(r.h0, l);
        h1 = lane_u32(r.h1, l);
    }
    const uint32_t nm = m1 > t.ts ? m1 - t.ts : 0u, nh = h1 > h0 ? h1 - h0 : 0u;
    const uint32_t own = nm + nh, nown = (nm ? 1u : 0u) + (nh ? 1u : 0u);
    const uint32_t end = own + wave_incl_scan(na + nb, lane);
    const uint32_t total = lane_u32(end, 63);
    // this part's chunks
    const uint32_t nc = (total + 63u) >> 6;
    const uint32_t c0 = (uint32_t)(((uint64_t)nc * part) >> plog);
    const uint32_t c1 = (uint32_t)(((uint64_t)nc * (part + 1u)) >> plog);
    if (c0 >= c1) return;
    const uint32_t v0 = c0 << 6, v1 = (c1 << 6) < total ? c1 << 6 : total;
    S.pos = v0;
    S.end = v1;
    S.own = nm;
    // the pairs of these neighbours: with the tile's own points j > i (or j !=
    // i), so neighbour ts + p pairs with p home points
    const uint32_t q = v1 < nm ? v1 : nm, nq = q > v0 ? q - v0 : 0u, nhome = t.te - t.ts;
    W.evals += (uint64_t)nhome * (v1 - v0 - nq);
    W.evals += P.selfx ? (uint64_t)(nhome - 1u) * nq : (uint64_t)(v0 + q - 1u) * nq / 2u;
    const uint64_t ma = __builtin_amdgcn_ballot_w64(na != 0u);
    const uint64_t mb = __builtin_amdgcn_ballot_w64(nb != 0u);
    const uint32_t pos = nown + lanes_below(ma) + lanes_below(mb);
    S.n = nown + (uint32_t)(__popcll(ma) + __popcll(mb));
    // (starts clipped to v0, so that no lane below it takes a span)
    auto put = [&](uint32_t k, uint32_t start, uint32_t first, uint32_t code) {
        S.e[k] = make_uint2(start > v0 ? start : v0, first - start);
        S.f[k] = (uint8_t)code;
    };
    wave_lds_fence();
    if (lane == 0) {
        if (nm) put(0u, 0u, t.ts, kNoShift | kSelfSpan);
        if (nh) put(nown - 1u, nm, h0, kNoShift);
    }
    const uint32_t sa = end - na - nb;
    if (na) put(pos, sa, r.a0, r.ca);
    if (nb) put(pos + (na ? 1u : 0u), sa + na, r.b0, r.cb);
    // the span that holds position v0, or the one before it in its row
    S.k = 0u;
    if (v0 >= own) S.k = lane_u32(pos, (int)__popcll(__builtin_amdgcn_ballot_w64(end <= v0)));
    wave_lds_fence();
}

// Assemble the next chunk of the walk over a tile's neighbours (filled = 0 at
// its end): every lane takes the last span that starts at or before its
// position. A span costs four VALU instructions and no scalar bookkeeping but
// its number. (Copying span by span took about 100 scalar instructions each and
// as much time as the pairs of a tile of 16 points: the r-mu count of 1e6
// points takes 2.60 ms with this, 2.73 with that; of 2.5e5, 1.28 and 1.42.)
template <bool SPH>
__device__ __forceinline__ void next_chunk(const CountArgs& P, WaveState& W, SpanBuf& S, Chunk& C,
                                           const Tile& tl, int lane, uint32_t part, uint32_t plog) {
    C.filled = 0;
    C.masked = false;
    C.shifted = false;
    for (;;) {
        if (S.pos < S.end) {
            // (lanes filled from the batch before have positions below S.pos,
            // perhaps negative ones; positions stay below 2^31)
            const int v = (int)(S.pos - C.filled) + lane;
            uint2 e = S.e[S.k];
            uint32_t f = S.f[S.k];
            for (;;) {
                const uint32_t kn = S.k + 1u < S.n ? S.k + 1u : S.k;
                const uint2 en = S.e[kn];
                const uint32_t fn = S.f[kn];
                const bool in = v >= (int)e.x;
                C.lj = in ? (uint32_t)v + e.y : C.lj;
                C.lcode = in ? f : C.lcode;
                if (kn == S.k || __builtin_amdgcn_ballot_w64(v >= (int)en.x) == 0ull) break;
                S.k = kn;
                e = en;
                f = fn;
            }
            const uint32_t room = 64u - C.filled, left = S.end - S.pos;
            const uint32_t take = left < room ? left : room;
            C.masked = C.masked | (S.pos < S.own);
            C.filled += take;
            S.pos += take;
            if (C.filled == 64u) break;
        } else if (S.row0 < S.nrows) {
            next_rows<SPH>(P, W, S, tl, lane, part, plog);
        } else {
            break;
        }
    }
    if (!SPH && P.periodic)
        C.shifted = __builtin_amdgcn_ballot_w64((uint32_t)lane < C.filled && (C.lcode & ~kSelfSpan) != kNoShift) != 0ull;
}

// Count the pairs of one home tile, or one of its 2^plog parts.
template <int MODE, int PREC, int EST, bool PM, bool WT>
__device__ void do_tile(const CountArgs& P, WaveState& W, SpanBuf& S, const float2* B1,
                        const float2* B2, const double* T1, const double* T2, int lane,
                        const Tile& tl, uint32_t part, uint32_t plog) {
    if (part == 0u) W.tiles++;
    if (PM && P.mbA != nullptr) {
        // a tile whose home points are all masked out has no pair to count
        const uint32_t i = tl.start + (uint32_t)lane;
        const bool live = i < tl.end && ((P.mbA[i >> 5] >> (i & 31u)) & 1u) == 0u;
        if (__builtin_amdgcn_ballot_w64(live) == 0ull) return;
    }
    S.row0 = 0;
    S.nrows = 1;
    S.n = S.k = S.pos = S.end = S.own = 0u;
    Chunk C;
    C.lj = 0;
    C.lcode = kNoShift;
    if constexpr (kMfma<MODE, PREC, EST>) {
        stage_home<MODE, PM>(P, W, tl, lane);
        Tab32 tab = make_tab32<EST>(P, B1, B2);
        const Hot hot = hot_args<PM>(P);
        if constexpr (MODE == M_SIGMAPI) tab.mt = W.mt;
        if constexpr (MODE == M_RMU_MID) {
            tab.d0 = W.mb0;
            tab.d1 = W.mb1;
        }
        // the neighbours of a chunk are loaded while the one before it is
        // counted
        Chunk N = C;
        N.filled = 0u;
        Near pn;
        pn.p = make_float4(0.f, 0.f, 0.f, 0.f);
        pn.r = 0.0;
        pn.w = 1u;
        pn.mask = 0u;
        do {
            C = N;
            const Near p = pn;
            next_chunk<kSphere<MODE>>(P, W, S, N, tl, lane, part, plog);
            if ((uint32_t)lane < N.filled) load_near<MODE, PM, WT>(P, pn, N.lj);
            if (C.filled == 0u) continue;
            // Radial: redshifts rounded to the bin width leave most pairs on an
            // edge, where re-tests take longer than FP64 throughout: a wave
            // that re-tested more than 1/24 of its pairs so far (pend, in units
            // of 64; looked at every 512 of them) counts so. Data and randoms
            // of 3e5 rounded to the width: 8.1 ms without, 5.5 with this as in
            // FP64 throughout; rounded to a tenth of it, 2 % re-tested: 2.6.
            bool all64 = MODE == M_RMU_MID && W.mt < 0.f;
            if constexpr (MODE == M_RADIAL) {
                const uint32_t seen = W.pend + ((C.filled * (tl.end - tl.start) + 63u) >> 6);
                if (((seen ^ W.pend) & ~511u) != 0u)
                    W.all64 = uni(W.rstat[0] * 24ull > (unsigned long long)seen * 64ull ? 1u : 0u);
                W.pend = seen;
                all64 = W.all64 != 0u;
            }
            if ((MODE == M_RMU_MID || MODE == M_RADIAL) && all64)
                run_chunk<MODE, P_FP64, EST & E_LOG, PM, WT>(P, W, B1, B2, T1, T2, lane, C, tl.start, tl.end);
            else
                run_chunk_mfma<MODE, EST, PM, WT>(P, hot, W, tab, B1, B2, T1, T2, lane, C, p, tl.start, tl.end);
        } while (N.filled != 0u);
    } else {
        for (;;) {
            next_chunk<kSphere<MODE>>(P, W, S, C, tl, lane, part, plog);
            if (C.filled == 0u) break;
            run_chunk<MODE, PREC, EST, PM, WT>(P, W, B1, B2, T1, T2, lane, C, tl.start, tl.end);
        }
    }
}


}  // namespace
}  // namespace cute
