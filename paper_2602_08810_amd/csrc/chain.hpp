// Helpers shared by the scans that cut the time axis into groups chained through global memory
// (the LTI scan, its adjoint, and the scan with caller-supplied coefficients): complex arithmetic on float2,
// uniform-row addressing, and the publish/poll protocol of the chain.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace lrnnx {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a^e by repeated squaring, carried in double precision and rounded once.  The powers lambda^len multiply the states
// carried between wavefronts and workgroups; a relative error eps in lambda^len acts like an error eps/len in lambda
// itself, to which a state with memory 1/(1-|lambda|) steps is 1/(1-|lambda|) times as sensitive: squaring in fp32
// (eps of about len * 2^-24) cost an order of magnitude in the accuracy of x and of the gradient with respect to lambda.
__device__ __forceinline__ float2 cpow(float2 a, int64_t e) {
    double ar = a.x, ai = a.y, rr = 1.0, ri = 0.0;
    while (e > 0) {
        if (e & 1) { const double t = rr * ar - ri * ai; ri = rr * ai + ri * ar; rr = t; }
        const double t = ar * ar - ai * ai; ai = 2.0 * ar * ai; ar = t;
        e >>= 1;
    }
    return make_float2((float)rr, (float)ri);
}
__device__ __forceinline__ float2 cfma(float2 a, float2 b, float2 c) {   // a*b + c
    return make_float2(__builtin_fmaf(a.x, b.x, __builtin_fmaf(-a.y, b.y, c.x)),
                       __builtin_fmaf(a.x, b.y, __builtin_fmaf(a.y, b.x, c.y)));
}

constexpr int kSpinLimit = 1 << 22;          // polls before a waiting wavefront gives up
constexpr int kAnchor = 16;                  // every 16th group publishes its true end state

// Elements of a wave-uniform row at a lane's 32-bit byte offset (scalar base + vector offset addressing), for the
// tensors that are streamed through once.  NT: a non-temporal access, which leaves the caches to others.
typedef float stream_f2 __attribute__((ext_vector_type(2)));
template <bool NT>
__device__ __forceinline__ float2 load_at(const float2 *row, unsigned byte_off) {
    const stream_f2 *q = reinterpret_cast<const stream_f2 *>(reinterpret_cast<const char *>(row) + byte_off);
    const stream_f2 t = NT ? __builtin_nontemporal_load(q) : *q;
    return make_float2(t.x, t.y);
}
template <bool NT>
__device__ __forceinline__ float load_at(const float *row, unsigned byte_off) {
    const float *q = reinterpret_cast<const float *>(reinterpret_cast<const char *>(row) + byte_off);
    return NT ? __builtin_nontemporal_load(q) : *q;
}
template <bool NT>
__device__ __forceinline__ void store_at(float2 *row, unsigned byte_off, float2 v) {
    stream_f2 *q = reinterpret_cast<stream_f2 *>(reinterpret_cast<char *>(row) + byte_off);
    const stream_f2 t = {v.x, v.y};
    if (NT) __builtin_nontemporal_store(t, q); else *q = t;
}
template <bool NT>
__device__ __forceinline__ void store_at(float *row, unsigned byte_off, float v) {
    float *q = reinterpret_cast<float *>(reinterpret_cast<char *>(row) + byte_off);
    if (NT) __builtin_nontemporal_store(v, q); else *q = v;
}

// Where the streams go past the caches (a forward call and its adjoint, us, before and after):
// - What an adjoint writes is not read again in the call: its stores are non-temporal.  LTI, P = 1024, 8 x 8192 steps
//   498 -> 485; 4 x 4096 steps, P = 256 43.2 -> 41.2; real coefficients, P = 1024, 8 x 2048 steps 127.5 -> 118.5.  Rows of real
//   values that are not whole lines share too many of them between workgroups (P = 129, 16 x 8001 steps 158 -> 170, P = 777 254 -> 270): ordinary
//   there; 8-byte values gain all the same (P = 1237, 3 x 4000 235 -> 226).  The forward's
//   states are read next by the adjoint, and its stores stay ordinary (non-temporal: 127 -> 133).
// - What an adjoint reads is read once, if the rows of P values are whole cache lines: then its loads are
//   non-temporal too (485 -> 458, 118.5 -> 116).  Rows that are not share their lines with the neighbouring
//   workgroup's (P = 1000 real, 8 x 4096 steps: 234 and 242 with such loads; P = 777, 1 x 13476 84 and 98); 8-byte values share fewer and
//   gain from 256 MiB of loads on, the size of the Infinity Cache (LTI, P = 600, 16 x 2000 steps 154 -> 147; with less P = 333, 2 x 9000 63 and 70).
// - The forward's loads likewise, but only from 384 MiB of traffic on, one and a half times the 256 MiB of Infinity Cache: there
//   458 -> 440 (complex coefficients, P = 1024, 8 x 4096: 397 -> 378); with less the inputs are often still in it (real
//   coefficients, 8 x 2048 steps: 116 and 120).  Rows of 8-byte values that are not whole lines, both rules together: LTI, P = 1001,
//   8 x 8192 568 -> 545; complex coefficients, P = 1000, 8 x 4096 401 -> 386, P = 1237, 3 x 4000 206 -> 199.
constexpr int64_t kCacheLine = 128;
constexpr int64_t kStreamPastCaches = 384ll << 20, kPastInfinityCache = 256ll << 20;
inline bool whole_lines(int64_t row_bytes, const void *a, const void *b, const void *c) {
    return ((row_bytes | (int64_t)(intptr_t)a | (int64_t)(intptr_t)b | (int64_t)(intptr_t)c) & (kCacheLine - 1)) == 0;
}

// The slab a workgroup takes: workgroup j of the n of one group of steps.  Consecutive workgroups run on the 8 dies in turn, each with an L2
// of its own; with `deal` the slabs go out so that each die gets a run of neighbours, which share the cache lines at their borders: read
// from memory once then, and the two parts of a line written meet in one L2.
__device__ __forceinline__ int slab_of(unsigned j, unsigned n, int deal) {
    const unsigned c = j & 7;
    return (int)(deal ? c * (n >> 3) + (c < (n & 7) ? c : (n & 7)) + (j >> 3) : j);
}
// Where dealing pays (a forward call and its adjoint, us, in turn and dealt): rows that are not whole lines (LTI, P = 1001, 8 x 8192 steps 632
// and 568, P = 207, 20 x 1265 56 and 50; real coefficients, P = 129, 16 x 8001 158 and 130, P = 1000, 8 x 4096 257 and 234; complex, P = 1001,
// 8 x 2048 254 and 233), and many slabs also where they share nothing (P = 1024: real, 8 x 2048 110.0 and 109.5, 8 x 8192 403 and 376; complex, 8 x 2048
// 207 and 201; LTI, 8 x 8192 439.5 and 433).  Few
// slabs of whole lines are as fast or faster in turn (LTI, P = 1024, 1 x 16384: 124 and 127; P = 256, 4 x 4096 40.0 and 40.5).
inline int deal_slabs(bool whole, unsigned n) { return !whole || n >= 64; }

// A published slot is an 8-byte complex value written by one relaxed atomic store at agent scope; kNotReady
// (all ones, a NaN pattern that arithmetic does not produce from other inputs) marks an empty slot, and a
// value that happens to equal it is stored as the canonical NaN instead.
constexpr unsigned long long kNotReady = ~0ull;
__device__ __forceinline__ void publish(float2 *slot, float2 val) {
    unsigned long long bits = ((unsigned long long)__float_as_uint(val.y) << 32) | __float_as_uint(val.x);
    if (bits == kNotReady) bits = 0x7fc000007fc00000ull;
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(slot), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const float2 *slot) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(slot), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 from_bits(unsigned long long bits) {
    return make_float2(__uint_as_float((unsigned)bits), __uint_as_float((unsigned)(bits >> 32)));
}

}  // namespace lrnnx
