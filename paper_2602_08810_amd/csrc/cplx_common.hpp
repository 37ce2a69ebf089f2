// Complex-arithmetic building blocks shared by the forward and backward selective-scan kernels with a complex
// diagonal state matrix: the complex word of the I/O type, exp(dt A) through the hardware exp2 / sin / cos, the four
// discretisations of Sec. 3 of the paper in complex arithmetic, and one Hillis-Steele step on a complex affine pair.
#pragma once
#include "scan_common.hpp"

namespace lrnnx {

template <typename IO> struct cword;                   // one complex number in the I/O type, as stored in LDS
template <> struct cword<bf16_t> {
    using type = uint32_t;
    static __device__ __forceinline__ float2 unpack(uint32_t w) { return make_float2(i2f((int)(w << 16)), i2f((int)(w & 0xFFFF0000u))); }
};
template <> struct cword<float> {
    using type = float2;
    static __device__ __forceinline__ float2 unpack(float2 w) { return w; }
};

// NK consecutive complex words, 16 bytes at a time where they fill whole 16-byte chunks (the caller's base pointer
// is 16-byte aligned and the row pitch N * sizeof(CW) is then a multiple of 16 too)
template <typename CW, int NK>
__device__ __forceinline__ void load_cwords(const CW *p, CW *out) {
    constexpr int BYTES = NK * (int)sizeof(CW);
    if constexpr (BYTES % 16 == 0) {
        uint4 r[BYTES / 16];
#pragma unroll
        for (int c = 0; c < BYTES / 16; ++c) r[c] = reinterpret_cast<const uint4 *>(p)[c];
        __builtin_memcpy(out, r, BYTES);
    } else {
#pragma unroll
        for (int k = 0; k < NK; ++k) out[k] = p[k];
    }
}

constexpr float kInv2Pi = 0.15915494309189535f;

// a = exp(dt A) for complex A = (Ar, Ai): e^{dt Ar} (cos(dt Ai), sin(dt Ai)).  v_sin/v_cos take revolutions and are
// only valid within +-256 of them, so the whole revolutions are dropped first (v_fract_f32): any dt Im(A) is
// accepted; the phase keeps the absolute accuracy of the fp32 product, |dt Im(A) / 2 pi| * 2^-24 revolutions.
__device__ __forceinline__ float2 cexp_dt(float dt, float A2r, float Arev) {
    const float e = exp2_fast(dt * A2r);
    const float rev = __builtin_amdgcn_fractf(dt * Arev);
    return make_float2(e * __builtin_amdgcn_cosf(rev), e * __builtin_amdgcn_sinf(rev));
}

struct CCoef {
    float Ar, Ai;       // A
    float A2r, Arev;    // Ar * log2(e), Ai / (2 pi): arguments of the hardware exp2 / sin / cos
    float iAr, iAi;     // 1 / A
};
__device__ __forceinline__ CCoef make_ccoef(float Ar, float Ai) {
    CCoef c;
    c.Ar = Ar; c.Ai = Ai; c.A2r = Ar * kLog2e; c.Arev = Ai * kInv2Pi;
    const float den = Ar * Ar + Ai * Ai;
    const float r = den > 0.0f ? rcp_fast(den) : 0.0f;
    c.iAr = Ar * r; c.iAi = -Ai * r;
    return c;
}

// Bilinear scheme: q = 1 / (1 - dt A / 2), from which the multiplier (1 + dt A / 2) q = 2 q - 1, the gain dt q and all partials
// follow.  Not the other way round: for |dt A| >> 1 the multiplier is close to -1, and q = (a + 1) / 2 taken from the rounded
// a has a relative error of up to |dt A| 2^-27 (7e-6 at 10^3).
__device__ __forceinline__ float2 cbilinear_q(float dt, const CCoef &c) {
    const float hr = 0.5f * dt * c.Ar, hi = 0.5f * dt * c.Ai;               // dt A / 2
    const float wr = 1.0f - hr, wi = -hi;                                   // 1 - dt A / 2
    const float r = rcp_fast(wr * wr + wi * wi);
    return make_float2(wr * r, -wi * r);
}
__device__ __forceinline__ float2 cbilinear_a(float2 q) { return make_float2(__builtin_fmaf(2.0f, q.x, -1.0f), 2.0f * q.y); }

// c0 + c1 z + .. + c4 z^4 with real coefficients, z = (zr, zi), s = |z|^2: by z^2 = 2 zr z - s, nine instructions; Horner's rule in complex
// arithmetic took twelve to fourteen for one power less.  In the exact zero-order hold this and sums without intermediate results are 5 % of the
// whole training step (8 x 768 rows of 2048 steps, N = 16, bf16 1185 -> 1121 us), and the largest relative error of the two series up to
// |z| = 1/8 is 1.5e-7 where it was 3.6e-6.
__device__ __forceinline__ float2 creal_quartic(float zr, float zi, float s, float c0, float c1, float c2, float c3, float c4) {
    const float r = zr + zr, b3 = __builtin_fmaf(r, c4, c3), b2 = __builtin_fmaf(r, b3, __builtin_fmaf(-s, c4, c2)),
                b1 = __builtin_fmaf(r, b2, __builtin_fmaf(-s, b3, c1));
    return make_float2(__builtin_fmaf(zr, b1, __builtin_fmaf(-s, b2, c0)), zi * b1);
}

// multiplier a and input gain g of one step (schemes of Sec. 3, complex arithmetic)
template <int DISC>
__device__ __forceinline__ void cdisc_ag(float dt, const CCoef &c, float2 &a, float2 &g) {
    if constexpr (DISC == DISC_BILINEAR) {
        const float2 q = cbilinear_q(dt, c);
        a = cbilinear_a(q);
        g = make_float2(dt * q.x, dt * q.y);
    } else {
        a = cexp_dt(dt, c.A2r, c.Arev);
        if constexpr (DISC == DISC_ZOH_S6) g = make_float2(dt, 0.0f);
        else if constexpr (DISC == DISC_DIRAC) g = make_float2(1.0f, 0.0f);
        else {                                                              // exact ZOH: (a - 1) / A
            const float zr = dt * c.Ar, zi = dt * c.Ai;
            // small |z|: dt (1 + z/2 + z^2/6 + z^3/24 + z^4/120)
            const float s2 = __builtin_fmaf(zr, zr, zi * zi);
            const float2 ser = creal_quartic(zr, zi, s2, 1.0f, 0.5f, 0.16666667f, 0.041666668f, 0.0083333338f);
            const float sr = dt * ser.x, si = dt * ser.y;
            const float mr = a.x - 1.0f, mi = a.y;
            const float dr = mr * c.iAr - mi * c.iAi, di = mr * c.iAi + mi * c.iAr;
            const bool small = s2 < 0.015625f;
            g = make_float2(small ? sr : dr, small ? si : di);
        }
    }
}

// One Hillis-Steele step on a complex affine pair.  Lanes without a source lane (or in a masked row) read the
// identity pair, which leaves them unchanged.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void cpair_step(float2 &P, float2 &S) {
    const float qr = dpp<CTRL, ROW_MASK>(1.0f, P.x), qi = dpp<CTRL, ROW_MASK>(0.0f, P.y);
    const float tr = dpp<CTRL, ROW_MASK>(0.0f, S.x), ti = dpp<CTRL, ROW_MASK>(0.0f, S.y);
    S = make_float2(__builtin_fmaf(P.x, tr, __builtin_fmaf(-P.y, ti, S.x)),
                    __builtin_fmaf(P.x, ti, __builtin_fmaf(P.y, tr, S.y)));
    P = make_float2(P.x * qr - P.y * qi, P.x * qi + P.y * qr);
}
__device__ __forceinline__ void cwave_scan_fwd(float2 &P, float2 &S) {
    cpair_step<0x111, 0xF>(P, S);
    cpair_step<0x112, 0xF>(P, S);
    cpair_step<0x114, 0xF>(P, S);
    cpair_step<0x118, 0xF>(P, S);
    cpair_step<DPP_ROW_BCAST15, 0xA>(P, S);
    cpair_step<DPP_ROW_BCAST31, 0xC>(P, S);
}


// ---------------------------------------------------------------- complex arithmetic on float2
__device__ __forceinline__ float2 cxmul(float2 a, float2 b) {
    return make_float2(__builtin_fmaf(a.x, b.x, -a.y * b.y), __builtin_fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 cxmulc(float2 a, float2 b) {        // a * conj(b)
    return make_float2(__builtin_fmaf(a.x, b.x, a.y * b.y), __builtin_fmaf(a.y, b.x, -a.x * b.y));
}
__device__ __forceinline__ float2 cxfma(float2 a, float2 b, float2 c) {   // a * b + c
    return make_float2(__builtin_fmaf(a.x, b.x, __builtin_fmaf(-a.y, b.y, c.x)),
                       __builtin_fmaf(a.x, b.y, __builtin_fmaf(a.y, b.x, c.y)));
}

// dg/dA of one step of the exact zero-order hold, given its a and g (holomorphic in A; the other partials are written out where they
// are used): (dt A a - (a - 1)) / A^2 = (dt a - g) / A; for small z = dt A: dt^2 (1/2 + z/3 + z^2/8 + z^3/30 + z^4/144)
__device__ __forceinline__ float2 czoh_gain_dA(float dt, const CCoef &c, float2 a, float2 g) {
    const float zr = dt * c.Ar, zi = dt * c.Ai, s2 = __builtin_fmaf(zr, zr, zi * zi);
    const float2 s = creal_quartic(zr, zi, s2, 0.5f, 0.33333334f, 0.125f, 0.033333335f, 0.0069444445f);
    const float d2 = dt * dt;
    const float2 big = cxmul(make_float2(__builtin_fmaf(dt, a.x, -g.x), __builtin_fmaf(dt, a.y, -g.y)),
                             make_float2(c.iAr, c.iAi));
    const bool small = s2 < 0.015625f;
    return make_float2(small ? d2 * s.x : big.x, small ? d2 * s.y : big.y);
}

}  // namespace lrnnx
