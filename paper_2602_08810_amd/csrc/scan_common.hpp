// Device-side building blocks shared by the gfx950 scan kernels: I/O element access,
// transcendental helpers, the fused discretisations (schemes named in Sec. 3 of the
// paper) and the wavefront scans over affine pairs.
//
// The recurrence x_k = a_k x_{k-1} + b_k (Eq. 2, line 1, diagonal A) is the
// composition of affine maps (a, b): x -> a x + b.  Two maps compose as
//     (a2, b2) o (a1, b1) = (a2 a1, a2 b1 + b2),
// which is associative, so a wavefront can take an inclusive prefix over its 64
// lanes in six cross-lane steps.  Out-of-range lanes hold the identity (1, 0).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "kernels.hpp"

namespace lrnnx {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct bf16_t { unsigned short v; };

// ---------------------------------------------------------------- bit casts and cross-lane moves
__device__ __forceinline__ int f2i(float x) { return __builtin_bit_cast(int, x); }
__device__ __forceinline__ float i2f(int x) { return __builtin_bit_cast(float, x); }

// DPP move: lanes whose source lane does not exist (or whose row is masked off) keep `old`.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp(float old, float src) {
    return i2f(__builtin_amdgcn_update_dpp(f2i(old), f2i(src), CTRL, ROW_MASK, 0xF, false));
}
constexpr int DPP_WAVE_SHR1 = 0x138;
constexpr int DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143;

__device__ __forceinline__ float readlane(float x, int lane) { return i2f(__builtin_amdgcn_readlane(f2i(x), lane)); }
// copy of `old` with lane `lane` replaced by the wave-uniform value v: one v_writelane_b32.  This compiler has no
// builtin for it, so the LLVM intrinsic is declared by its name (the compiler still sees an ordinary instruction
// and handles its hazards).
extern "C" __device__ int lrnnx_llvm_writelane_i32(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ float writelane(float old, float v, int lane) {
    return i2f(lrnnx_llvm_writelane_i32(f2i(v), lane, f2i(old)));
}
// Rows of two registers: on return a holds the even rows of both (a's first), b the odd rows; its own inverse.  All in the vector ALU (a
// swizzle through the LDS crossbar would cost a round trip of a hundred cycles).
__device__ __forceinline__ void swap_rows(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)f2i(a), (unsigned)f2i(b), false, false);
    a = i2f((int)r[0]); b = i2f((int)r[1]);
}
// The sequence of a packed batch that a workgroup takes: batch entry b is the steps cu[b] .. cu[b+1]-1 of ONE packed time axis of Lp
// steps.  The bounds are clamped to the axis, so no content of cu can send an access out of the buffers.  Workgroups start in launch
// order; RANKED (at most 64 sequences), blockIdx.y counts from the longest sequence down (ties by index), so that the short ones fill the end of the launch instead of
// a long one running on alone: lane i holds sequence i, and each counts the longer ones, three instructions a sequence (24 sequences of
// 16384 steps in all, 1536 channels, N = 16, bf16: forward pass 124 -> 106 us, and the launch that formed the order for
// the backward pass, 4.7 us, is gone).
// `order`: the sequences in an order formed before, or null.  One result for the wavefront, in scalar registers.
struct SeqSpan { int b; int64_t toff, L; };
__device__ __forceinline__ SeqSpan seq_span(const int64_t *cu, int B, int64_t Lp, int index, bool ranked, const int *order = nullptr) {
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    if (order) index = order[index];
    const int i = ranked ? (lane < B ? lane : B - 1) : index;  // (not ranked: every lane the same sequence)
    int64_t o = cu[i], e = cu[i + 1];
    o = o < 0 ? 0 : (o > Lp ? Lp : o);
    e = e < o ? o : (e > Lp ? Lp : e);
    const int64_t n = e - o;
    int rank = 0, at = 0;
    if (ranked) {
        const int nlo = (int)n, nhi = (int)(n >> 32);
        if (Lp < (1 << 25)) {                                  // the index below the length, in one word
            const int key = nlo << 6 | (63 - lane);
            for (int k = 0; k < B; ++k) rank += __builtin_amdgcn_readlane(key, k) > key ? 1 : 0;
        } else {
            for (int k = 0; k < B; ++k) {
                const int64_t m = (int64_t)__builtin_amdgcn_readlane(nhi, k) << 32 | (unsigned)__builtin_amdgcn_readlane(nlo, k);
                rank += m > n || (m == n && k < lane) ? 1 : 0;
            }
        }
        at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < B && rank == index));    // (the ranks of the sequences are 0 .. B-1)
    }
    auto pick = [&](int64_t v) {
        return (int64_t)__builtin_amdgcn_readlane((int)(v >> 32), at) << 32 | (unsigned)__builtin_amdgcn_readlane((int)v, at);
    };
    return {ranked ? at : index, pick(o), pick(n)};
}
// The same for the forward kernels, most of whose launches are not ranked: those read their bounds into scalar registers at once.  Ranked launches are
// kernels of their own, since the mere code of the ranking costs the others time: batches [B,D,L] with 16 lanes a channel (8 x 1536 rows of 2048
// steps, N = 16, bf16: 95.6 -> 96.4 us, dirac 94.7 -> 95.5), packed ones with 64 lanes 2.5 %.
template <bool RANKED> __device__ __forceinline__ SeqSpan seq_span_fwd(const int64_t *cu, int B, int64_t Lp, int index) {
    if constexpr (RANKED) return seq_span(cu, B, Lp, index, true);
    int64_t o = cu[index], e = cu[index + 1];
    o = o < 0 ? 0 : (o > Lp ? Lp : o);
    e = e < o ? o : (e > Lp ? Lp : e);
    return {index, o, e - o};
}
// LDS accumulate without a returned value: the wavefront does not wait for it
__device__ __forceinline__ void lds_add(float *p, float v) {
    (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------- transcendentals (fp32, ~1 ulp hardware ops)
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }   // v_exp_f32
__device__ __forceinline__ float log2_fast(float x) { return __builtin_amdgcn_logf(x); }    // v_log_f32
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }     // v_rcp_f32

// softplus(s) = log(1 + e^s) and its derivative sigmoid(s) = e^s / (1 + e^s).
// The logarithm of 1 + w rounds its argument, which leaves an
// ABSOLUTE error of 2^-24 in the step size: for float32 I/O (PRECISE) small w take the series of log(1 + w) instead,
// which keeps full relative accuracy; with bfloat16 I/O, whose inputs and outputs carry relative errors of 2^-9, the
// absolute 6e-8 is far below anything the step size is multiplied into, and the series is left out.
template <bool PRECISE = true>
__device__ __forceinline__ void softplus_sigmoid(float s, float &sp, float &sg) {
    // w stays finite for any s; past the clamp (and within its rounding before it) softplus is s itself
    const float w = exp2_fast(fminf(s, 64.0f) * kLog2e);
    float v = log2_fast(1.0f + w) * kLn2;
    if constexpr (PRECISE) {
        const float series = w * (1.0f - w * (0.5f - w * (0.33333334f - w * 0.25f)));
        v = w < 0.015625f ? series : v;
    }
    sp = fmaxf(v, s);
    sg = w * rcp_fast(1.0f + w);
}
// softplus alone, as max(s, 0) + log(1 + e^-|s|)
template <bool PRECISE = true>
__device__ __forceinline__ float softplus(float s) {
    const float w = exp2_fast(__builtin_fabsf(s) * -kLog2e);
    const float v = log2_fast(1.0f + w);
    float r;                                     // (fmaxf would first spend an instruction on quieting s)
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(s));
    if constexpr (PRECISE) {
        const float series = w * (1.0f - w * (0.5f - w * (0.33333334f - w * 0.25f)));
        return r + (w < 0.015625f ? series : v * kLn2);
    }
    return __builtin_fmaf(v, kLn2, r);
}
__device__ __forceinline__ float sigmoid_fast(float zz) { return rcp_fast(1.0f + exp2_fast(-zz * kLog2e)); }

// Input gain of the exact zero-order hold, g = (e^{dt A} - 1) / A, given a = e^{dt A} and rA = 1/A (0 for A = 0).
// For |dt A| >= 1/64 the difference a - 1 loses at most 6 bits (relative error <= 64 eps = 4e-6); below, and for
// A = 0, g = dt (1 + x/2 + x^2/6) with x = dt A, whose first omitted term x^3/24 is below 2e-7.
__device__ __forceinline__ float zoh_gain(float dt, float A, float rA, float a) {
    const float x = dt * A;
    float small = dt * __builtin_fmaf(x, __builtin_fmaf(x, 0.16666667f, 0.5f), 1.0f), closed = (a - 1.0f) * rA;
    asm("" : "+v"(small), "+v"(closed));             // a select of two values: the compiler makes branches around the four
    return fabsf(x) < 0.015625f ? small : closed;    // instructions otherwise, which cost more than both sides together
}

// ---------------------------------------------------------------- fused discretisation (Sec. 3 schemes)
enum : int { DISC_ZOH_S6 = 0, DISC_ZOH = 1, DISC_BILINEAR = 2, DISC_DIRAC = 3 };

// Per-(d,n) constants derived once from A[d,n].
struct ACoef {
    float A;      // A[d,n]
    float A2;     // A * log2(e), so that exp(dt*A) = exp2(dt*A2)
    float rA;     // 1/A (exact ZOH only; 0 for A == 0, where the series branch of the gain applies)
    float hA;     // A/2 (bilinear only)
};
template <int DISC>
__device__ __forceinline__ ACoef make_acoef(float A) {
    ACoef c; c.A = A; c.A2 = A * kLog2e;
    if constexpr (DISC == 1) c.rA = (A != 0.0f) ? rcp_fast(A) : 0.0f; else c.rA = 0.0f;
    c.hA = 0.5f * A;
    return c;
}

// Bilinear scheme: q = 1 / (1 - dt A / 2), from which the multiplier a = (1 + dt A / 2) q = 2 q - 1, the gain dt q and all partials
// follow; v_rcp_f32 is accurate to 1 ulp, like the exponential of the other schemes.  Not the other way round: for |dt A| >> 1
// a is close to -1, and q = (a + 1) / 2 taken from the rounded a has a relative error of up to |dt A| 2^-27 (7e-6 at 10^3).
__device__ __forceinline__ float bilinear_q(float dt, const ACoef &c) { return rcp_fast(__builtin_fmaf(-dt, c.hA, 1.0f)); }
__device__ __forceinline__ float bilinear_a(float q) { return __builtin_fmaf(2.0f, q, -1.0f); }

// State multiplier a and input gain g of one step.
template <int DISC>
__device__ __forceinline__ void disc_ag(float dt, const ACoef &c, float &a, float &g) {
    if constexpr (DISC == DISC_BILINEAR) {
        const float q = bilinear_q(dt, c);
        a = bilinear_a(q);
        g = dt * q;
    } else {
        a = exp2_fast(dt * c.A2);
        if constexpr (DISC == DISC_ZOH_S6) g = dt;
        else if constexpr (DISC == DISC_DIRAC) g = 1.0f;
        else g = zoh_gain(dt, c.A, c.rA, a);
    }
}

// dg/dA of one step of the exact zero-order hold, given its a and g.  (The other partials of this scheme, da/ddt = A a, da/dA = dt a and
// dg/ddt = a, and all of the other schemes' are written out where they are used.)
// (dt A a - (a - 1)) / A^2 = (dt a - g) / A = dt^2 (1/2 + x/3 + x^2/8 + x^3/30 + ...), x = dt A.  A rounding error e in a reaches
// the difference dt a - g as e / A, i.e. 2 eps / x^2 relative to it: the closed form is used from |x| = 1/8 on (1e-5), the series
// below (first omitted term x^4/144 < 4e-6).
__device__ __forceinline__ float zoh_gain_dA(float dt, const ACoef &c, float a, float g) {
    const float x = dt * c.A;
    float small = dt * dt * __builtin_fmaf(x, __builtin_fmaf(x, __builtin_fmaf(x, 0.033333335f, 0.125f), 0.33333334f), 0.5f);
    float closed = __builtin_fmaf(dt, a, -g) * c.rA;
    asm("" : "+v"(small), "+v"(closed));         // (no branches, as in zoh_gain)
    return fabsf(x) < 0.125f ? small : closed;
}

// ---------------------------------------------------------------- per-step inputs of the backward pass
// gate y = ypre z sigmoid(z): dy becomes the gradient reaching ypre, zf the factor that turns ypre into dz
__device__ __forceinline__ void gate_bwd(float z, float &dy, float &zf) {
    const float sz = sigmoid_fast(z);
    const float dsz = dy * sz;
    dy = dsz * z;
    zf = dsz * __builtin_fmaf(z, 1.0f - sz, 1.0f);
}
// From the raw step input s = delta + bias, the upstream gradient dy and the gate input z of one time step:
// Delta and d Delta / d s, the gradient reaching ypre (y = ypre z sigmoid(z)) and the factor that turns ypre into dz
// (dz = dy ypre sigmoid(z) (1 + z (1 - sigmoid(z)))).
template <bool PRECISE = true>
__device__ __forceinline__ void bwd_step_inputs(float s, float dy, float z, bool softplus, bool has_z,
                                                float &sp, float &sg, float &dyp, float &zf) {
    if (softplus) softplus_sigmoid<PRECISE>(s, sp, sg); else { sp = s; sg = 1.0f; }
    dyp = dy; zf = 0.0f;
    if (has_z) gate_bwd(z, dyp, zf);
}

// ---------------------------------------------------------------- issue priority
// Two wavefronts of a SIMD issue plain fp32 instructions side by side (2.8 to 3 cycles of 2.4 GHz an instruction), and one wavefront issues
// them beside a transcendental, a row swap or a DPP operand of the other, which take the ALU 4.5 to 8.5 cycles.  But this lasts
// only while the wavefront with the slow instruction goes first, and only where slow instructions are dense: one exponential in
// 64 multiply-adds 3.0 cycles an instruction, one in eight 5.5, one DPP operand in eight 4.9, whatever the priorities.  So a kernel
// keeps such instructions together and raises its priority over them (slow_part), lowers it for plain arithmetic (fast_part), and raises
// it further where a workgroup is about to meet at a barrier (edge_part).  A loop like the backward pass's (18 exponentials and 46 DPP
// operands, then 244 plain): 4.0 cycles an instruction with two wavefronts a SIMD at equal priorities, 4.25 with the priorities the wrong
// way round, 3.1 with these; 3.8, 4.4 and 3.05 with three (valu_probe.hip).  The whole kernels keep part of that: see there.
template <int P>
__device__ __forceinline__ void issue_priority() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(P);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void slow_part() { issue_priority<1>(); }
__device__ __forceinline__ void fast_part() { issue_priority<0>(); }
__device__ __forceinline__ void edge_part() { issue_priority<2>(); }

// ---------------------------------------------------------------- wavefront scans over affine pairs
// One Hillis-Steele step on the pair held in (P,S): the pair of the lane named by the DPP
// control is composed in from the earlier side.  Both updates are single VALU instructions
// with a DPP source operand; a lane whose source lane does not exist, or whose row is
// masked off, is left unchanged (= composed with the identity).  The leading s_nop covers
// the two wait states a DPP read needs after a VALU write of the same register.
#define LRNNX_PAIR_STEP(P, S, CTRL)                                                   \
    asm("s_nop 1\n\t"                                                                 \
        "v_fmac_f32_dpp %0, %0, %1 " CTRL "\n\t"                                      \
        "v_mul_f32_dpp %1, %1, %1 " CTRL                                              \
        : "+v"(S), "+v"(P))

// Inclusive prefix over the 64 lanes, lane 0 first:  (P,S)_i <- (P,S)_i o ... o (P,S)_0.
__device__ __forceinline__ void wave_scan_fwd(float &P, float &S) {
    LRNNX_PAIR_STEP(P, S, "row_shr:1 row_mask:0xf bank_mask:0xf");
    LRNNX_PAIR_STEP(P, S, "row_shr:2 row_mask:0xf bank_mask:0xf");
    LRNNX_PAIR_STEP(P, S, "row_shr:4 row_mask:0xf bank_mask:0xf");
    LRNNX_PAIR_STEP(P, S, "row_shr:8 row_mask:0xf bank_mask:0xf");
    LRNNX_PAIR_STEP(P, S, "row_bcast:15 row_mask:0xa bank_mask:0xf");   // lane 15 of rows 0,2 -> rows 1,3
    LRNNX_PAIR_STEP(P, S, "row_bcast:31 row_mask:0xc bank_mask:0xf");   // lane 31 -> rows 2,3
}

// Parts of a kernel's own blocks: one Hillis-Steele step of a prefix pair (s, p), and of a prefix pair together with a suffix
// pair (r, q).  The numbers are operands of the block.  Whoever strings them together keeps two instructions between a
// register's write and its next DPP read, and begins the block with s_nop 1, in case the compiler placed a copy right before.
#define LRNNX_F_STATE(s, p, CF)                                                        \
    "v_fmac_f32_dpp %" #s ", %" #s ", %" #p " " CF "\n\t"                               \
    "v_mul_f32_dpp %" #p ", %" #p ", %" #p " " CF "\n\t"
#define LRNNX_FR_STATE(s, p, r, q, CF, CR) LRNNX_F_STATE(s, p, CF) LRNNX_F_STATE(r, q, CR)
#define LRNNX_ALLROWS " row_mask:0xf bank_mask:0xf"

// ---------------------------------------------------------------- words cleared on the stream
// thread i of `stride` threads
__device__ __forceinline__ void fill_words(const FillList &z, int64_t i, int64_t stride) {
#pragma unroll
    for (int k = 0; k < FillList::kMax; ++k) {
        uint32_t *ptr = reinterpret_cast<uint32_t *>(z.ptr[k]);
        if (!ptr) continue;
        const uint32_t word = z.bits[k];
        for (int64_t j = i; j < z.count[k]; j += stride) ptr[j] = word;
    }
}

// ---------------------------------------------------------------- I/O element access
template <typename IO> struct io_traits;
template <> struct io_traits<float> {
    static constexpr int EPC = 4;                                  // elements per 16-byte chunk
    __device__ static __forceinline__ float get(const float *p, int64_t i) { return p[i]; }
    __device__ static __forceinline__ void put(float *p, int64_t i, float v) { p[i] = v; }
    __device__ static __forceinline__ void unpack(const uint4 &r, float *o) {
        o[0] = i2f(r.x); o[1] = i2f(r.y); o[2] = i2f(r.z); o[3] = i2f(r.w);
    }
    __device__ static __forceinline__ uint4 pack(const float *v) {
        return make_uint4(f2i(v[0]), f2i(v[1]), f2i(v[2]), f2i(v[3]));
    }
};
typedef __bf16 bf16x2_native __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {   // round to nearest even
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_native));
}
template <> struct io_traits<bf16_t> {
    static constexpr int EPC = 8;
    __device__ static __forceinline__ float get(const bf16_t *p, int64_t i) { return i2f((int)p[i].v << 16); }
    __device__ static __forceinline__ void put(bf16_t *p, int64_t i, float v) {
        p[i].v = (unsigned short)(pack_bf16x2(v, 0.0f) & 0xFFFFu);
    }
    __device__ static __forceinline__ void unpack(const uint4 &r, float *o) {
        o[0] = i2f(r.x << 16); o[1] = i2f(r.x & 0xFFFF0000u);
        o[2] = i2f(r.y << 16); o[3] = i2f(r.y & 0xFFFF0000u);
        o[4] = i2f(r.z << 16); o[5] = i2f(r.z & 0xFFFF0000u);
        o[6] = i2f(r.w << 16); o[7] = i2f(r.w & 0xFFFF0000u);
    }
    __device__ static __forceinline__ uint4 pack(const float *v) {
        return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                          pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
};

// 16-, 8- and 4-byte accesses to the time axis of a [B,D,L] tensor are made at ELEMENT alignment: rows of packed
// variable-length batches start anywhere, and global memory takes unaligned vector accesses (the compiler is told
// the true alignment and still emits one instruction).  IO selects the alignment (2 or 4 bytes).
template <typename IO> struct ua;
template <> struct ua<float> {
    typedef uint4 __attribute__((aligned(4))) v4;
    typedef uint2 __attribute__((aligned(4))) v2;
    typedef uint32_t __attribute__((aligned(4))) v1;
};
template <> struct ua<bf16_t> {
    typedef uint4 __attribute__((aligned(2))) v4;
    typedef uint2 __attribute__((aligned(2))) v2;
    typedef uint32_t __attribute__((aligned(2))) v1;
};

// A lane's CNT consecutive elements row[l .. l+CNT), zero where l+i >= L.  `vec` allows vector accesses (the host
// sets it when every row pointer is element-aligned).
template <typename IO, int CNT>
__device__ __forceinline__ void load_seg(const IO *row, int64_t l, int64_t L, bool vec, float *out) {
    constexpr int EPC = io_traits<IO>::EPC;
    static_assert(CNT % EPC == 0, "segment must be whole 16-byte chunks");
#pragma unroll
    for (int c = 0; c < CNT / EPC; ++c) {
        int64_t lc = l + c * EPC;
        if (vec && lc + EPC <= L) {
            uint4 r = *reinterpret_cast<const typename ua<IO>::v4 *>(row + lc);
            io_traits<IO>::unpack(r, out + c * EPC);
        } else {
#pragma unroll
            for (int i = 0; i < EPC; ++i) out[c * EPC + i] = (lc + i < L) ? io_traits<IO>::get(row, lc + i) : 0.0f;
        }
    }
}
template <typename IO, int CNT>
__device__ __forceinline__ void store_seg(IO *row, int64_t l, int64_t L, bool vec, const float *v) {
    constexpr int EPC = io_traits<IO>::EPC;
#pragma unroll
    for (int c = 0; c < CNT / EPC; ++c) {
        int64_t lc = l + c * EPC;
        if (vec && lc + EPC <= L) {
            *reinterpret_cast<typename ua<IO>::v4 *>(row + lc) = io_traits<IO>::pack(v + c * EPC);
        } else {
#pragma unroll
            for (int i = 0; i < EPC; ++i) if (lc + i < L) io_traits<IO>::put(row, lc + i, v[c * EPC + i]);
        }
    }
}

// CNT contiguous elements starting at p, as floats.  p must be aligned to min(16, CNT*sizeof(IO)) bytes
// (CNT*sizeof(IO) is a power of two in every use).
template <typename IO, int CNT>
__device__ __forceinline__ void load_row(const IO *p, float *out) {
    constexpr int EPC = io_traits<IO>::EPC;
    constexpr int BYTES = CNT * (16 / EPC);
    if constexpr (BYTES % 16 == 0) {
#pragma unroll
        for (int c = 0; c < CNT / EPC; ++c) {
            uint4 r = reinterpret_cast<const uint4 *>(p)[c];
            io_traits<IO>::unpack(r, out + c * EPC);
        }
    } else if constexpr (BYTES == 8) {
        uint2 r = *reinterpret_cast<const uint2 *>(p);
        float tmp[EPC];
        io_traits<IO>::unpack(make_uint4(r.x, r.y, 0u, 0u), tmp);
#pragma unroll
        for (int i = 0; i < CNT; ++i) out[i] = tmp[i];
    } else if constexpr (BYTES == 4) {
        uint32_t r = *reinterpret_cast<const uint32_t *>(p);
        float tmp[EPC];
        io_traits<IO>::unpack(make_uint4(r, 0u, 0u, 0u), tmp);
#pragma unroll
        for (int i = 0; i < CNT; ++i) out[i] = tmp[i];
    } else {
#pragma unroll
        for (int i = 0; i < CNT; ++i) out[i] = io_traits<IO>::get(p, i);
    }
}

template <typename IO, int CNT, typename IDX>
__device__ __forceinline__ void store_few(IO *row, IDX l, IDX L, bool vec, const float *v) {
    constexpr int EPC = io_traits<IO>::EPC;
    constexpr int BYTES = CNT * (16 / EPC);
    if constexpr (CNT == 1) {                                   // one element: a single predicated access either way
        if (l < L) io_traits<IO>::put(row, l, v[0]);
    } else if (vec && l + CNT <= L && BYTES % 16 == 0) {
#pragma unroll
        for (int c = 0; c < BYTES / 16; ++c)
            reinterpret_cast<typename ua<IO>::v4 *>(row + l)[c] = io_traits<IO>::pack(v + c * EPC);
    } else if (vec && l + CNT <= L && (BYTES == 8 || BYTES == 4)) {
        float tmp[EPC];
#pragma unroll
        for (int i = 0; i < EPC; ++i) tmp[i] = i < CNT ? v[i] : 0.0f;
        uint4 r = io_traits<IO>::pack(tmp);
        if constexpr (BYTES == 8) *reinterpret_cast<typename ua<IO>::v2 *>(row + l) = make_uint2(r.x, r.y);
        else *reinterpret_cast<typename ua<IO>::v1 *>(row + l) = r.x;
    } else {
#pragma unroll
        for (int i = 0; i < CNT; ++i) if (l + i < L) io_traits<IO>::put(row, l + i, v[i]);
    }
}

// The same few elements as untouched 32-bit words, so that a load can be issued long before its
// data is needed (unpacking is a separate step and nothing waits on the load until then).
template <typename IO, int CNT>
struct RawFew {
    static constexpr int COUNT = CNT;
    static constexpr int WORDS = (CNT * (16 / io_traits<IO>::EPC) + 3) / 4;
    uint32_t w[WORDS];
};
template <typename IO, int CNT, typename IDX>
__device__ __forceinline__ void load_few_raw(const IO *row, IDX l, IDX L, bool vec, RawFew<IO, CNT> &r) {
    constexpr int BYTES = CNT * (16 / io_traits<IO>::EPC);
    constexpr int WORDS = RawFew<IO, CNT>::WORDS;
    if constexpr (CNT == 1) {
        // one element, read without a branch: past the end the last element is read again and dropped (L >= 1)
        const IDX lc = l < L ? l : L - 1;
        uint32_t v;
        if constexpr (sizeof(IO) == 4) v = *reinterpret_cast<const uint32_t *>(row + lc);
        else v = *reinterpret_cast<const unsigned short *>(row + lc);
        r.w[0] = l < L ? v : 0u;
    } else if (vec && l + CNT <= L) {
        if constexpr (BYTES % 16 == 0) {
#pragma unroll
            for (int c = 0; c < BYTES / 16; ++c) {
                const uint4 v = reinterpret_cast<const typename ua<IO>::v4 *>(row + l)[c];
                r.w[4 * c] = v.x; r.w[4 * c + 1] = v.y; r.w[4 * c + 2] = v.z; r.w[4 * c + 3] = v.w;
            }
        } else if constexpr (BYTES == 8) {
            const uint2 v = *reinterpret_cast<const typename ua<IO>::v2 *>(row + l);
            r.w[0] = v.x; r.w[1] = v.y;
        } else if constexpr (BYTES == 4) {
            r.w[0] = *reinterpret_cast<const typename ua<IO>::v1 *>(row + l);
        } else {
            r.w[0] = *reinterpret_cast<const unsigned short *>(row + l);
        }
    } else {
        // all of them without a branch, so that they are under way together (one after the other, each waited for, the end
        // of a sequence cost a wavefront ten microseconds); past the end the last element, dropped (L >= 1)
        uint32_t v[CNT];
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            const IDX lc = l + i < L ? l + i : L - 1;
            if constexpr (sizeof(IO) == 4) v[i] = *reinterpret_cast<const uint32_t *>(row + lc);
            else v[i] = *reinterpret_cast<const unsigned short *>(row + lc);
        }
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            v[i] = l + i < L ? v[i] : 0u;
            if constexpr (sizeof(IO) == 4) r.w[i] = v[i];
            else r.w[i / 2] = i % 2 ? r.w[i / 2] | v[i] << 16 : v[i];
        }
    }
}
template <typename IO, int CNT>
__device__ __forceinline__ void unpack_few(const RawFew<IO, CNT> &r, float *out) {
#pragma unroll
    for (int i = 0; i < CNT; ++i) {
        if constexpr (sizeof(IO) == 4) out[i] = i2f((int)r.w[i]);
        else out[i] = (i % 2) ? i2f((int)(r.w[i / 2] & 0xFFFF0000u)) : i2f((int)(r.w[i / 2] << 16));
    }
}

// The end of a sequence, without a branch: a lane whose CNT elements row[l .. l+CNT) reach past the last valid one, row[n-1],
// reads the last CNT valid ones instead (tail_window; they must exist, n may be less than CNT if the row has steps before
// row[0]) and moves them down once they are needed (tail_shift).  What then stands for elements past the end is some valid
// element: the CALLER discards it.  Element by element, a lane at the end sent its wavefront through CNT loads more, and in a
// packed batch every sequence has such a tile (24 sequences of 8192 steps in all, 2560 channels, N = 4, bf16: backward
// 306 us, so 235; 24 of 16384 steps, 1536 channels, N = 16: forward and backward 683 us, so 634).
template <int CNT>
__device__ __forceinline__ int tail_window(int l, int n) { return l + CNT <= n ? l : n - CNT; }
template <typename IO, int CNT>
__device__ __forceinline__ void tail_shift(RawFew<IO, CNT> &r, int by) {         // by = l - tail_window(l, n)
    constexpr int W = RawFew<IO, CNT>::WORDS, PER = sizeof(IO) == 2 ? 2 : 1;
    if constexpr (PER == 2 && CNT > 1) {
        const unsigned s = (by & 1) * 16;
#pragma unroll
        for (int i = 0; i < W; ++i) r.w[i] = __builtin_amdgcn_alignbit(i + 1 < W ? r.w[i + 1] : 0u, r.w[i], s);
    }
#pragma unroll
    for (int b = 1; b < W; b <<= 1) {
        const uint32_t move = by & (b * PER) ? ~0u : 0u;     // (a select of the two would become one of their addresses)
#pragma unroll
        for (int i = 0; i + b < W; ++i) r.w[i] = (move & r.w[i + b]) | (~move & r.w[i]);
    }
}

}  // namespace lrnnx
