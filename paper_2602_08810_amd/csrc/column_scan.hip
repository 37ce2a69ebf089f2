// Scans over time with one workgroup to a block of columns, for gfx950: the LTI recurrence x_k = lambda x_{k-1} + v_k and the real
// recurrence with caller-supplied coefficients x_k = a_k x_{k-1} + b_k (Eq. 2 of the paper, Sec. 2.2.1 and 2.2.2).
//
// The arrays are [B,L,P] with P contiguous.  A workgroup takes COLS neighbouring columns of one batch entry and walks the
// whole time axis in tiles, the next tile's loads under way during this one's steps.  Nothing is exchanged between
// workgroups: no workspace, no launch that arms one (4.7 us), no waiting on a chain.  Of a wavefront's 64 lanes COLS lie along the
// columns and J = 64 / COLS along time; a lane owns T consecutive steps, a wavefront J T and a tile W J T.  Lanes fold their steps
// to affine pairs, a prefix over the J pieces stays in the wavefront, and the wavefronts' pairs meet in LDS, where every lane chains
// them onto the carry that it keeps.
//
// What bounds it: memory, or with few tiles' work a workgroup the latency of a tile (1 to 3 us) and the fetching of the kernel's code.  Against the
// chained scans with the launch that arms their slots (us): 2 x 102 columns of 280 steps, LTI 8.5 -> 4.9, 7 x 455 of 1966 27.6 -> 25.8, 4 x 256 of
// 4096 18.5 -> 16.5; real coefficients 16 x 30 of 467 7.0 -> 4.6, 8 x 1024 of 2048 35.7 -> 33.9.  Since then: row addresses of a lane's steps added up
// in one vector register, where eight in scalar registers had up to 97 of these spilled, and one form of the loads for all tiles: 5.5 to 6 KB of
// code for 11 to 12, from a graph 5.5 -> 4.5 (the first of these calls), 5.3 -> 4.2 and 35.4 -> 33.7 (the real ones), none slower.  16 steps
// a lane spill (56 us on the 8 x 1024 columns), and with one set of registers refilled during the replay less is under way (36).
#include "kernels.hpp"
#include "chain.hpp"
#include "elem.hpp"
#include <cmath>
#include <type_traits>

namespace lrnnx {

template <bool LTI, int COLS, int T, int W>
__global__ __launch_bounds__(W * 64, 4) void k_column_scan(const ColumnParams p) {
    using EL = Elem<LTI>;                                      // complex poles, real coefficients
    using E = typename EL::T;
    constexpr int J = 64 / COLS, SPAN = J * T, TILE = W * SPAN;
    // The pairs of caller-supplied coefficients are formed and chained in double precision: 8 steps a lane pass through more of them than the
    // chained scan's 32, and in single precision the states' error (2-norm, against 64 bits) was 4.3e-8 where that scan's is 4.0e-8.
    // Products of many coefficients can leave the range of the states, which may be zero or tiny where they do (a lane's pieces begin
    // up to 120 steps after the wavefront's first).  Powers of lambda beyond single precision are taken in double as well, and what is beyond
    // that (any state but zero is infinite then) never meets a zero, a state's or a coefficient's that ends what came before: a power is kept finite,
    // a product of coefficients not applied to it.
    using ED = Elem<LTI, double>;
    using D = typename ED::T;
    using ES = std::conditional_t<LTI, EL, ED>;                // end states of pieces
    using End = typename ES::T;
    __shared__ End sS[2][W][COLS];
    __shared__ D sA[2][LTI ? 1 : W][COLS];

    const int lane = threadIdx.x & 63, c = lane % COLS, j = lane / COLS;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // blocks that share cache lines go to one XCD (workgroup i runs on XCD i % 8)
    const int nblk = (p.P + COLS - 1) / COLS;
    const unsigned id = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (id >= (unsigned)nblk * (unsigned)p.B) return;          // (the whole workgroup)
    const int b = id / nblk, col = (id % nblk) * COLS + c;
    const bool okp = col < p.P;
    const int64_t P = p.P, pc = okp ? col : p.P - 1;           // (lanes past the last column repeat it and store nothing)
    // An element's address: a row that all lanes share (in scalar registers) and the lane's offset in bytes, 32 bits: see column_shape
    const unsigned off = ((unsigned)(j * T) * (unsigned)p.P + (unsigned)pc) * (unsigned)sizeof(E);
    const int64_t row0 = ((int64_t)b * p.L + w * SPAN) * P;    // of the wavefront's first step
    const int first = (w * J + j) * T;                         // the lane's first position within a tile

    E lam = EL::one(), x0 = EL::zero();
    if constexpr (LTI) lam = reinterpret_cast<const E *>(p.a)[pc];
    if (p.x0) x0 = reinterpret_cast<const E *>(p.x0)[(int64_t)b * P + pc];

    struct Steps { E v[T], a[LTI ? 1 : T]; };
    // Steps past the end of the sequence are read from its last row and become the identity map in `run`.
    // (offsets are formed where they are used: kept through the loop, eight of each, they would be spilled)
    auto fresh = [](unsigned v) { asm volatile("" : "+v"(v)); return v; };
    const unsigned pitch = (unsigned)p.P * (unsigned)sizeof(E);
    auto fetch = [&](int64_t tile, Steps &s) {
        const int64_t k0 = tile * TILE + w * SPAN, left = p.L - 1 - k0;        // the wavefront's first step, the steps after it
        const int64_t at = ((int64_t)b * p.L + (left < 0 ? p.L - 1 : k0)) * P;
        const E *vr = reinterpret_cast<const E *>(p.b) + at, *ar = LTI ? nullptr : reinterpret_cast<const E *>(p.a) + at;
        const unsigned end = (left < 0 ? 0u : left < SPAN ? (unsigned)left : (unsigned)SPAN) * pitch + (unsigned)pc * (unsigned)sizeof(E);
        unsigned o = fresh(off);
#pragma unroll
        for (int i = 0; i < T; ++i, o += pitch) {
            const unsigned oi = o < end ? o : end;
            s.v[i] = load_at<false>(vr, oi);
            if constexpr (!LTI) s.a[i] = load_at<false>(ar, oi);
        }
    };
    Steps s0;
    fetch(0, s0);

    // Powers of lambda: T 2^i steps, the lane's pieces before it, a wavefront (the first tile's loads are under way)
    D pow_w = ED::one(), pow_j = ED::one(), pow_d[7] = {};
    bool wide = !LTI;
    if constexpr (LTI) {
        auto finite = [](D x) { return ED::pick(__builtin_isfinite(x.x) && __builtin_isfinite(x.y), x, ED::make(__DBL_MAX__, 0.0)); };
        D q = ED::from(lam), r = ED::one();
#pragma unroll
        for (int e = 1; e < T; e *= 2) q = ED::mul(q, q);
#pragma unroll
        for (int d = 1, i = 0; d < J; d *= 2, ++i) {
            pow_d[i] = finite(q);
            const D t = ED::mul(r, q);
            if (j & d) r = t;
            q = ED::mul(q, q);
        }
        pow_w = finite(q); pow_j = finite(r);
        // (of the powers the largest, if any is large; a wavefront has all columns of the workgroup: one answer for all of it)
        wide = __builtin_amdgcn_ballot_w64(__builtin_fabs(q.x) <= __FLT_MAX__ && __builtin_fabs(q.y) <= __FLT_MAX__) != ~0ull;
    }

    // The walk over the tiles.  WIDE: the carry and what is applied to it and to the lanes' ends in double precision: real coefficients always, LTI
    // where a power needs it (always would cost 0.9 us on 4 x 256 columns of 4096 steps).
    auto walk = [&](auto WIDE) {
        using EC = std::conditional_t<WIDE, ED, EL>;
        using C = typename EC::T;
        const C lam_w = EC::from(pow_w), lam_j = EC::from(pow_j);
        C lam_d[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) lam_d[i] = EC::from(pow_d[i]);
        C carry = EC::from(x0);
        // a pair applied to a state, or with S = 0 to an earlier product
        auto apply = [](C A, C x, C S) {
            if constexpr (!LTI) {
                const int lo = __double2loint(A), hi = __double2hiint(A);
                A = __hiloint2double(x == 0 ? 0 : hi, lo);         // (finite)
            }
            return EC::fma(A, x, S);
        };
        auto run = [&](int64_t tile, Steps &s, const int buf) {
            const int64_t rem = p.L - tile * TILE;
            if (rem < TILE) {
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    s.v[i] = EL::pick(first + i < rem, s.v[i], EL::zero());
                    if constexpr (!LTI) s.a[i] = EL::pick(first + i < rem, s.a[i], EL::one());
                }
            }
            auto coef = [&](int i) { if constexpr (LTI) return lam; else return s.a[i]; };
            // ---- fold of the lane's steps, prefix over the wavefront's pieces
            D A = ED::one();
            End S = ES::zero();
#pragma unroll
            for (int i = 0; i < T; ++i) {
                S = ES::fma(ES::from(coef(i)), S, ES::from(s.v[i]));
                if constexpr (!LTI) A = ED::mul(ED::from(s.a[i]), A);
            }
#pragma unroll
            for (int d = 1, n = 0; d < J; d *= 2, ++n) {
                const End Sp = ES::up(S, d * COLS);
                if constexpr (LTI) { if (j >= d) S = ES::from(apply(lam_d[n], EC::from(Sp), EC::from(S))); }
                else {
                    const D Ap = ED::up(A, d * COLS);
                    if (j >= d) { S = apply(A, Sp, S); A = apply(A, Ap, ED::zero()); }
                }
            }
            if (j == J - 1) { sS[buf][w][c] = S; if constexpr (!LTI) sA[buf][w][c] = A; }
            End Se = ES::zero();
            D Ae = ED::one();                                      // of the pieces before this lane's
            if constexpr (J > 1) {
                Se = ES::pick(j > 0, ES::up(S, COLS), Se);
                if constexpr (!LTI) Ae = ED::pick(j > 0, ED::up(A, COLS), Ae);
            }
            __syncthreads();                                       // (two buffers: the one of the tile before may still be read)
            // ---- the wavefronts' pairs onto the carry
            C enter = carry;
#pragma unroll
            for (int ww = 0; ww < W; ++ww) {
                if (ww == w) enter = carry;
                if constexpr (LTI) carry = apply(lam_w, carry, EC::from(sS[buf][ww][c]));
                else carry = apply(sA[buf][ww][c], carry, sS[buf][ww][c]);
            }
            E x;
            if constexpr (LTI) x = EL::from(apply(lam_j, enter, EC::from(Se)));
            else x = EL::from(apply(Ae, enter, Se));
            // ---- replay
            E *xr = reinterpret_cast<E *>(p.x) + row0 + tile * TILE * P;
            E xl = x;                                              // the state after the sequence's last step, in the lane that has it
            unsigned o = fresh(off);
            if (rem >= TILE) {
#pragma unroll
                for (int i = 0; i < T; ++i, o += pitch) {
                    x = EL::fma(coef(i), x, s.v[i]);
                    if (okp) store_at<false>(xr, o, x);
                }
                xl = x;
            } else {
#pragma unroll
                for (int i = 0; i < T; ++i, o += pitch) {
                    x = EL::fma(coef(i), x, s.v[i]);
                    if (okp && first + i < rem) store_at<false>(xr, o, x);
                    xl = EL::pick(first + i < rem, x, xl);
                }
            }
            if (p.x_last && okp && first < rem && first + T >= rem) reinterpret_cast<E *>(p.x_last)[(int64_t)b * P + pc] = xl;
        };

        const int64_t ntiles = (p.L + TILE - 1) / TILE;
        [[maybe_unused]] Steps s1;
        if constexpr (LTI && WIDE) {                           // (no registers for a second tile)
            for (int64_t tile = 0; tile < ntiles; ++tile) {
                if (tile > 0) fetch(tile, s0);
                run(tile, s0, (int)tile & 1);
            }
            return;
        }
        for (int64_t tile = 0; tile < ntiles; tile += 2) {
            if (tile + 1 < ntiles) fetch(tile + 1, s1);
            run(tile, s0, 0);
            if (tile + 1 >= ntiles) break;
            if (tile + 2 < ntiles) fetch(tile + 2, s0);
            run(tile + 1, s1, 1);
        }
    };
    if (wide) walk(std::true_type{});
    else if constexpr (LTI) walk(std::false_type{});
}

// ---------------------------------------------------------------- which scan, which shape
// The estimated time of a call (us): a start, and of the rest a part for its steps one after the other and one for its bytes, which overlap:
// c0 + hypot(c1 * steps, c2 * MB), c2 for rows that are whole cache lines or not.  `steps` counts tiles, times the rounds in which the workgroups
// fit the chip, or for the chained scans thousands of time steps; the bytes of a column scan take longer, by the root of what a last round of one
// workgroup a compute unit lacks.  Rows that are not whole lines vary more with their length, and a column scan is taken there from an
// estimate a tenth below the other's.  Fitted over 240 shapes of 16 to 2048 columns, 64 to 16384 steps, 1 to 32 batch entries and 0.1 to 1100 MB: the
// choice is 1.33 (LTI) and 1.10 times (real) as fast as the chained scans alone (geometric mean), at worst 1.07 and 1.11 times as long.  (The costs are those of
// the kernel with twice the code, see above; the calls that take a column scan are now 0.83 (LTI, 40 calls) and 0.79 (real, 28) of that, from a graph.)
struct ColumnCost { int cols, waves; double c0, c1, c2[2]; };           // c2: whole lines, others
constexpr int kColumnT = 8;
constexpr double kChainedCost[2][4] = {{7.5, 1.39, 0.151, 0.21}, {6.2, 0.9, 0.163, 0.229}};
// LTI, real: 32-byte pieces of a row for few columns, 16 columns in half as large a workgroup for short sequences, whole lines of real values
// for many columns
constexpr ColumnCost kColumnCost[2][3] = {{{4, 8, 3.5, 1.45, {0.182, 0.209}}, {16, 4, 3.0, 0.9, {0.16, 0.185}}, {0, 0, 0, 0, {0, 0}}},
                                          {{8, 8, 3.1, 1.55, {0.194, 0.223}}, {16, 4, 2.75, 1.18, {0.167, 0.165}}, {32, 8, 3.27, 1.32, {0.138, 0.15}}}};

int column_shape(bool lti, int B, int P, int64_t L) {
    const int64_t es = lti ? 8 : 4, arrays = lti ? 2 : 3;
    const int part = P * es % kCacheLine == 0 ? 0 : 1;
    const double mb = (double)arrays * es * B * P * (double)L * 1e-6;
    const double *k = kChainedCost[lti ? 0 : 1];
    double least = k[0] + std::hypot(k[1] * (double)L * 1e-3, k[2 + part] * mb);
    int shape = 0;
    for (int i = 0; i < 3; ++i) {
        const ColumnCost &c = kColumnCost[lti ? 0 : 1][i];
        if (!c.cols) continue;
        const int64_t wgs = (int64_t)B * ((P + c.cols - 1) / c.cols), tile = (int64_t)c.waves * kColumnT * 64 / c.cols;
        // a lane's offset in 32 bits, and a grid's threads in 32 bits
        if (64 / c.cols * kColumnT * (int64_t)P * es >= (1ll << 31) || wgs > (1ll << 22)) continue;
        const int64_t places = (c.waves == 8 ? 2 : 4) * kNumCU, rounds = (wgs + places - 1) / places;
        const double full = std::sqrt((double)((wgs + kNumCU - 1) / kNumCU * kNumCU) / (double)wgs);
        const double t = (c.c0 + std::hypot(c.c1 * (double)((L + tile - 1) / tile * rounds), c.c2[part] * mb * full)) / (part ? 0.9 : 1.0);
        if (t < least) { least = t; shape = i + 1; }
    }
    return shape;
}

template <bool LTI, int COLS, int W> static void launch(const ColumnParams &p, hipStream_t s) {
    const unsigned wgs = (unsigned)p.B * ((p.P + COLS - 1) / COLS);
    hipLaunchKernelGGL((k_column_scan<LTI, COLS, kColumnT, W>), dim3((wgs + 7) / 8 * 8), dim3(W * 64), 0, s, p);
}

hipError_t launch_column_scan(bool lti, int shape, const ColumnParams &p, hipStream_t s) {
    if (lti) { if (shape == 1) launch<true, 4, 8>(p, s); else launch<true, 16, 4>(p, s); }
    else if (shape == 1) launch<false, 8, 8>(p, s);
    else if (shape == 2) launch<false, 16, 4>(p, s);
    else launch<false, 32, 8>(p, s);
    return hipGetLastError();
}

}  // namespace lrnnx
