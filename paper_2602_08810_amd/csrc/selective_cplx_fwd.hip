// Selective scan, forward, with a COMPLEX diagonal state matrix for gfx950:
//     x_{l,n} = a(Delta_l, A[d,n]) x_{l-1,n} + g(Delta_l, A[d,n]) Bm[b,l,n] u[b,d,l]        (complex)
//     y[b,d,l] = Re( sum_n Cm[b,l,n] x_{l,n} ) + Dskip[d] u[b,d,l],  then the optional gate
// (Eq. 2 of the paper with the output taken as Re(C x): the complex-diagonal layers of Sec. 2.2.1 with an
// input-dependent step size and input-dependent maps).
//
// Mapping: that of the real forward kernel (selective_fwd.hip).  A channel takes LPC lanes (16 or 64) of T consecutive steps
// each (4, 8 or 16); the W wavefronts of a workgroup walk the same tile of LPC T steps, whose maps are staged once per workgroup
// in LDS as fp32 pairs, eight states at a time, in an order that makes every access conflict-free.  Per state the lane folds its
// steps into one affine pair, the channel's lanes take the prefix over the pairs with DPP operands, and the lane replays its
// steps from the state that enters it, accumulating y.  The state after the tile waits in LDS.
//
// What bounds it: vector-ALU issue.  Multipliers, folds, scan and replay run at the priorities of scan_common.hpp: B=8, D=1536,
// N=16, L=2048, bf16 315 -> 258 us (multipliers, folds and scan as one part: 278).
//
// The same kernel serves the three launches of the chunk-carry path for few long rows (blockIdx.z = chunk), as in the real
// forward: MODE_AGG returns each chunk's pair, k_ss_ccarry chains them, MODE_APPLY reruns each chunk from its true carry-in.
#include "kernels.hpp"
#include "scan_common.hpp"
#include "cplx_common.hpp"
#include <type_traits>

namespace lrnnx {

// Inclusive prefix over the LPC lanes of each channel, first lane first: on return S holds it, X the prefix of the lane before (a
// channel's first lane keeps what it came with) and, in the channel's last lane with 16 lanes, P the product over all of them.
// Lanes without a source are left unchanged.  With 64 lanes the products have to be complete in every lane of a row, with 16
// an incomplete one is not used.  A DPP read comes two wait states or more after the write of its register.
template <int LPC>
__device__ __forceinline__ void cchannel_scan(float2 &P, float2 &S, float2 &X) {
    static_assert(LPC == 16 || LPC == 64, "lanes of a channel");
    float t, nx, ny;
#define LRNNX_ROW " row_mask:0xf bank_mask:0xf\n\t"
    // S += src(S) P, and (NX, NY) = P src(P); KEEP: what lanes without a source have as (NX, NY)
#define LRNNX_CS(CTRL, PX, PY, M1, M2, M3)                                                                                 \
    "v_mov_b32 %2, %0\n\t" M1 "v_fmac_f32_dpp %0, %0, " PX " " CTRL M2 "v_fmac_f32_dpp %0, -%1, " PY " " CTRL M3            \
    "v_fmac_f32_dpp %1, %1, " PX " " CTRL "v_fmac_f32_dpp %1, %2, " PY " " CTRL
#define LRNNX_CSP(CTRL, KEEP, PX, PY, NX, NY)                                                                              \
    LRNNX_CS(CTRL, PX, PY, KEEP "v_mul_f32_dpp " NX ", " PX ", " PX " " CTRL,                                              \
             "v_fmac_f32_dpp " NX ", -" PY ", " PY " " CTRL "v_mul_f32_dpp " NY ", " PX ", " PY " " CTRL,                   \
             "v_fmac_f32_dpp " NY ", " PY ", " PX " " CTRL)
#define LRNNX_CK(PX, PY, NX, NY) "v_mov_b32 " NX ", " PX "\n\tv_mov_b32 " NY ", " PY "\n\t"
    if constexpr (LPC == 16) {
        asm("s_nop 1\n\t"
            LRNNX_CSP("row_shr:1" LRNNX_ROW, "", "%3", "%4", "%5", "%6")
            LRNNX_CSP("row_shr:2" LRNNX_ROW, "", "%5", "%6", "%3", "%4")
            LRNNX_CSP("row_shr:4" LRNNX_ROW, "", "%3", "%4", "%5", "%6")
            LRNNX_CSP("row_shr:8" LRNNX_ROW, "", "%5", "%6", "%3", "%4")
            "v_mov_b32_dpp %7, %0 row_shr:1" LRNNX_ROW "s_nop 0\n\tv_mov_b32_dpp %8, %1 row_shr:1 row_mask:0xf bank_mask:0xf"
            : "+v"(S.x), "+v"(S.y), "=&v"(t), "+v"(P.x), "+v"(P.y), "=&v"(nx), "=&v"(ny), "+v"(X.x), "+v"(X.y));
    } else {
        asm("s_nop 1\n\t"
            LRNNX_CSP("row_shr:1" LRNNX_ROW, LRNNX_CK("%3", "%4", "%5", "%6"), "%3", "%4", "%5", "%6")
            LRNNX_CSP("row_shr:2" LRNNX_ROW, LRNNX_CK("%5", "%6", "%3", "%4"), "%5", "%6", "%3", "%4")
            LRNNX_CSP("row_shr:4" LRNNX_ROW, LRNNX_CK("%3", "%4", "%5", "%6"), "%3", "%4", "%5", "%6")
            LRNNX_CSP("row_shr:8" LRNNX_ROW, LRNNX_CK("%5", "%6", "%3", "%4"), "%5", "%6", "%3", "%4")
            // lane 15 of rows 0, 2 -> rows 1, 3, then lane 31 -> rows 2, 3
            LRNNX_CSP("row_bcast:15 row_mask:0xa bank_mask:0xf\n\t", LRNNX_CK("%3", "%4", "%5", "%6"), "%3", "%4", "%5", "%6")
            LRNNX_CS("row_bcast:31 row_mask:0xc bank_mask:0xf\n\t", "%5", "%6", "", "", "")
            "v_mov_b32_dpp %7, %0 wave_shr:1" LRNNX_ROW "s_nop 0\n\tv_mov_b32_dpp %8, %1 wave_shr:1 row_mask:0xf bank_mask:0xf"
            : "+v"(S.x), "+v"(S.y), "=&v"(t), "+v"(P.x), "+v"(P.y), "=&v"(nx), "=&v"(ny), "+v"(X.x), "+v"(X.y));
    }
#undef LRNNX_CK
#undef LRNNX_CSP
#undef LRNNX_CS
#undef LRNNX_ROW
}

template <int LPC, int T> struct CFwdGeom {
    static constexpr int W = LPC * T / 64 < 8 ? LPC * T / 64 : 8;      // wavefronts of a workgroup
    static constexpr int CPW = 64 / LPC;             // channels of a wavefront
    static constexpr int CH = W * CPW;               // channels of a workgroup
    static constexpr int TILE = LPC * T;
    static constexpr int Q = 4 * LPC + 128 / T;      // two steps of every lane, see below
    static constexpr int ROW = Q * (T / 2);          // a state of a staged map
};

// Wavefronts that share a SIMD: three with 16 lanes per channel (168 registers), four with 64.
// RANKED: a packed batch whose workgroups rank the sequences (ranked_sequences)
template <typename IO, int N, int DISC, bool WANT_Y, int LPC, int T, bool RANKED>
__global__ __launch_bounds__((CFwdGeom<LPC, T>::W * 64), (LPC == 16 ? 3 : 4)) void k_ss_cfwd(const CFwdParams p) {
    using CW = typename cword<IO>::type;
    using GE = CFwdGeom<LPC, T>;
    constexpr int W = GE::W, CPW = GE::CPW, CH = GE::CH, TILE = GE::TILE, NT = W * 64;
    constexpr int NS = N > 8 ? 8 : N, NH = N / NS;   // states staged at a time, and how often
    // registers enough to fetch what is staged next ahead of the state loop
    constexpr bool EARLY = LPC == 64 && (sizeof(IO) == 2 || T == 4 || N <= 4);
    static_assert(TILE == NT && TILE % kCkptInterval == 0, "a thread stages one step");
    __shared__ __attribute__((aligned(16))) float sBC[WANT_Y ? 2 * NS : NS][GE::ROW];      // Bm, Cm
    __shared__ __attribute__((aligned(16))) float2 sA[CH + 1][N], sX[CH + 2][N];   // A; the state entering the next tile, and zeros
    __shared__ float2 sP[WANT_Y ? 1 : CH][N];        // aggregate: product of the multipliers so far

    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane % LPC;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.y;
    // a workgroup takes CH consecutive channels of ONE Bm/Cm group (it stages that group's maps in LDS)
    const int blk_per_grp = (p.dpg + CH - 1) / CH;
    const int grp = blockIdx.x / blk_per_grp;
    const int din0 = (blockIdx.x % blk_per_grp) * CH;
    const int ch = w * CPW + lane / LPC;             // this lane's channel of the workgroup
    // lanes past the last channel of the group repeat it and store nothing.  (A wavefront that skips the work instead makes the
    // compiler keep what its lanes start from beside what they sum up: 16 registers.)
    const bool live = din0 + ch < p.dpg;
    const int d0 = grp * p.dpg + din0;
    const int d = grp * p.dpg + (live ? din0 + ch : p.dpg - 1);
    const int chunk = blockIdx.z;
    // packed variable-length mode (p.cu != nullptr, see seq_span): I/O rows have no batch stride, the maps are [G, p.L, N]
    int64_t L = p.L, toff = 0;
    constexpr bool BRIEF = LPC == 64 && T == 4;      // see row()
    std::conditional_t<BRIEF, unsigned, int64_t> bs = b;
    if (p.cu) {
        const SeqSpan q = seq_span_fwd<RANKED>(p.cu, p.B, p.L, b);
        b = q.b; toff = q.toff; L = q.L; bs = 0;
    }
    const int64_t ntiles = (L + TILE - 1) / TILE;
    const int64_t tile0 = (int64_t)chunk * p.tiles_per_chunk;
    const int64_t tile1 = (tile0 + p.tiles_per_chunk < ntiles) ? tile0 + p.tiles_per_chunk : ntiles;
    const bool vec = p.vec != 0;
    const int mode = p.mode;

    // Rows and lanes are worked out again where they are used: an opaque copy of the thread's number keeps the compiler
    // from holding a register for each address throughout.  Calls of many short rows are bound by scalar instructions, which the
    // SIMDs of a compute unit share: the shape for them (64 lanes of 4 steps, whose rows are the wavefront's) forms the addresses of a
    // tile that is not whole where they are used, and multiplies the strides unsigned (N = 1, float32: 4 x 1024 rows of 64 steps 7.0 ->
    // 6.7 us, 8 x 1536 of 256 13.3 -> 12.5; whole tiles of long rows, their addresses formed anew, and the longer tiles take up to
    // 6 % longer with it).
    auto fresh = [&]() { unsigned t = tid; asm volatile("" : "+v"(t)); return t; };
    using channel_t = std::conditional_t<BRIEF, unsigned, int>;
    auto row = [&](const void *base, int64_t sb, int64_t sd, int64_t l, auto FULL) {
        int wv = w;
        if constexpr (BRIEF && !FULL) asm volatile("" : "+s"(wv));
        int c = din0 + wv * CPW + (fresh() & 63) / LPC;
        c = c < p.dpg ? c : p.dpg - 1;
        return reinterpret_cast<const IO *>(base) + ((int64_t)bs * sb + (int64_t)(channel_t)(grp * p.dpg + c) * sd + toff + l);
    };
    const int64_t bc0 = (((int64_t)bs * p.bcg + grp) * p.L + toff) * N;       // first complex element of the maps of this sequence
    const CW *Bm = reinterpret_cast<const CW *>(p.Bm) + bc0;
    const CW *Cm = reinterpret_cast<const CW *>(p.Cm) + bc0;
    const float Dsk = p.Dskip ? p.Dskip[d] : 0.0f;
    const float bias = p.bias ? p.bias[d] : 0.0f;
    // checkpoints: [B,D,nck,N], or packed [D,nslots,N] with sequence b starting at slot toff/interval + b
    const int64_t nck = p.cu ? p.nslots : (L + kCkptInterval - 1) / kCkptInterval;
    const int64_t ck_first = p.cu ? toff / kCkptInterval + b : 0;

    for (int i = lane; i < CPW * N; i += 64) {       // a wavefront's channels are its own: no barrier between it and these
        const int c = w * CPW + i / N, n = i % N;
        const int dc = d0 + (din0 + c < p.dpg ? c : 0);
        const int64_t r = (int64_t)b * p.D + dc;
        sA[c][n] = p.A[(int64_t)dc * N + n];
        float2 x = make_float2(0.0f, 0.0f);
        if (mode == MODE_APPLY) x = p.ws_S[(r * p.nchunks + chunk) * N + n];
        else if (mode != MODE_AGG && p.x0) x = p.x0[r * N + n];
        sX[c][n] = x;
        if constexpr (!WANT_Y) sP[c][n] = make_float2(1.0f, 0.0f);
    }
    if (lane < N) sX[CH][lane] = make_float2(0.0f, 0.0f);            // (every wavefront: the same value)

    // A staged state of Bm or Cm: step 2 k + i of lane l (of T) at k Q + 4 l + 2 i.  The reads, 16 bytes from each lane, are
    // contiguous over the lanes and share one address; Q leaves a gap of 128 / T so that the 32 consecutive steps which half a
    // wavefront stages at once fall into 64 banks.
    // ---- the inputs of a tile, raw.  Those of a whole tile (FULL: nothing to check per element) are fetched ahead.
    const bool window = vec && L >= T;               // the last steps of the sequence: see tail_window
    RawFew<IO, T> r_u, r_dl;
    CW r_B[NS], r_C[WANT_Y ? NS : 1];
    auto fetch_rows = [&](int64_t tile, auto FULL) {
        const int64_t l0 = tile * TILE;
        const IO *u = row(p.u, p.u_sb, p.u_sd, l0, FULL), *dl = row(p.delta, p.dl_sb, p.dl_sd, l0, FULL);
        const int r = (fresh() % LPC) * T;
        if constexpr (FULL) {
            load_few_raw<IO, T>(u + r, 0, T, true, r_u);
            load_few_raw<IO, T>(dl + r, 0, T, true, r_dl);
        } else {
            const int n = L - l0 < TILE ? (int)(L - l0) : TILE;
            if (window) {
                const int o = tail_window<T>(r, n);
                load_few_raw<IO, T>(u + o, 0, T, true, r_u);
                load_few_raw<IO, T>(dl + o, 0, T, true, r_dl);
            } else {
                load_few_raw<IO, T>(u, r, n, vec, r_u);
                load_few_raw<IO, T>(dl, r, n, vec, r_dl);
            }
        }
    };
    auto fetch_maps = [&](int64_t tile, int h, auto FULL) {
        int64_t l = tile * TILE + (int)fresh();
        if constexpr (!FULL) l = l < L ? l : L - 1;  // rows past the sequence: the last one again, discarded below
        load_cwords<CW, NS>(Bm + (l * N + h * NS), r_B);
        if constexpr (WANT_Y) load_cwords<CW, NS>(Cm + (l * N + h * NS), r_C);
    };
    // after the last tile: these registers hold nothing any more (without it they would stay occupied throughout)
    auto forget = [](auto &r) {
        uint32_t *q = reinterpret_cast<uint32_t *>(&r);
#pragma unroll
        for (unsigned i = 0; i < sizeof(r) / 4; ++i) asm volatile("" : "=v"(q[i]));
    };
    auto do_tile = [&](int64_t tile, auto FULL, bool ahead) {
        const int64_t l0 = tile * TILE;
        const int rem = FULL ? TILE : (L - l0 < TILE ? (int)(L - l0) : TILE);
        float dl[T], du[T], yv[T], sum_dl = 0.0f;    // du: Delta*u for S6, u for the other schemes
        RawFew<IO, T> r_z;
        auto fetch_z = [&]() {
            if constexpr (WANT_Y) {
                if (!p.z) return;
                const IO *z = row(p.z, p.z_sb, p.z_sd, l0, FULL);
                const int r = (fresh() % LPC) * T;
                if constexpr (FULL) load_few_raw<IO, T>(z + r, 0, T, true, r_z);
                else if (window) load_few_raw<IO, T>(z + tail_window<T>(r, rem), 0, T, true, r_z);
                else load_few_raw<IO, T>(z, r, rem, vec, r_z);
            }
        };
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            // ---- stage the maps of NS states (all wavefronts) as fp32 pairs
            __syncthreads();
            {
                const unsigned r = fresh();
                float *at = &sBC[0][(r % T) / 2 * GE::Q + (r / T) * 4 + (r % 2) * 2];
                const bool ok = FULL || (int)r < rem;
#pragma unroll
                for (int n = 0; n < NS; ++n) {
                    const float2 v = cword<IO>::unpack(r_B[n]);
                    *reinterpret_cast<float2 *>(at + n * GE::ROW) = make_float2(ok ? v.x : 0.0f, ok ? v.y : 0.0f);
                }
                if constexpr (WANT_Y) {
#pragma unroll
                    for (int n = 0; n < NS; ++n) {
                        const float2 v = cword<IO>::unpack(r_C[n]);
                        *reinterpret_cast<float2 *>(at + (NS + n) * GE::ROW) = make_float2(ok ? v.x : 0.0f, ok ? v.y : 0.0f);
                    }
                }
            }
            if (TILE == kCkptInterval && p.ckpt && h == 0) {     // the state entering the tile is the carried one
                for (int i = fresh() & 63; i < CPW * N; i += 64) {
                    const int c = w * CPW + i / N;
                    const int64_t r = p.cu ? (int64_t)(d0 + c) : (int64_t)b * p.D + d0 + c;
                    if (din0 + c < p.dpg) p.ckpt[(r * nck + ck_first + tile) * N + i % N] = sX[c][i % N];
                }
            }
            __syncthreads();
            if (h == 0) {
                // ---- this lane's steps of Delta, Delta u and D u
                if (!FULL && window) {
                    const int r = (fresh() % LPC) * T, by = r - tail_window<T>(r, rem);
                    tail_shift<IO, T>(r_u, by);
                    tail_shift<IO, T>(r_dl, by);
                }
                unpack_few<IO, T>(r_u, du);
                unpack_few<IO, T>(r_dl, dl);
#pragma unroll
                for (int t = 0; t < T; ++t) asm volatile("" : "+v"(du[t]), "+v"(dl[t]));
                if constexpr (EARLY) fetch_z();
#pragma unroll
                for (int t = 0; t < T; ++t) { dl[t] += bias; asm volatile("" : "+v"(dl[t])); }
                if (p.softplus) {
#pragma unroll
                    for (int t = 0; t < T; ++t) dl[t] = softplus<sizeof(IO) == 4>(dl[t]);
                }
                if constexpr (!FULL) {                   // steps past the end are the identity map (a = 1, b = 0)
                    const int r0 = (fresh() % LPC) * T;
#pragma unroll
                    for (int t = 0; t < T; ++t) { dl[t] = (r0 + t < rem) ? dl[t] : 0.0f; du[t] = (r0 + t < rem) ? du[t] : 0.0f; }
                }
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    sum_dl += dl[t];
                    if constexpr (WANT_Y) yv[t] = Dsk * du[t];
                    if constexpr (DISC == DISC_ZOH_S6) du[t] *= dl[t];
                }
            }
            auto fetch_next = [&]() {
                if (h + 1 < NH) { fetch_maps(tile, h + 1, FULL); return; }
                if (FULL && ahead) {
                    fetch_maps(tile + 1, 0, FULL);
                    fetch_rows(tile + 1, FULL);
                } else { forget(r_B); forget(r_C); forget(r_u); forget(r_dl); }
            };
            {
                if constexpr (EARLY) fetch_next();
                auto read = [&](const float *m, auto COUNT, float2 *v) {       // COUNT steps
#pragma unroll
                    for (int k = 0; k < COUNT / 2; ++k) {
                        const float4 f = *reinterpret_cast<const float4 *>(m + k * GE::Q);
                        v[2 * k] = make_float2(f.x, f.y); v[2 * k + 1] = make_float2(f.z, f.w);
                    }
                };
                constexpr std::integral_constant<int, 4> kFew;
                const float *lB = &sBC[0][li * 4];
                const float2 *lA = &sA[ch][h * NS];
                const float2 *lX = &sX[li == 0 ? ch : CH][h * NS];   // the carried state enters through the channel's first lane
                float2 An = lA[0], xn = lX[0];
#pragma unroll 1
                for (int n = 0; n < NS; ++n) {
                    // Bm's reads are under way while the multipliers are formed, Cm's during the scan
                    const CCoef cc = make_ccoef(An.x, An.y);
                    float2 xin = xn, a[T], x[T], P, S;
                    An = lA[n + 1]; xn = lX[n + 1];      // (after the last n: not used)
                    read(lB + n * GE::ROW, std::integral_constant<int, T>{}, x);
                    slow_part();
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        float2 g;
                        cdisc_ag<DISC>(dl[t], cc, a[t], g);
                        if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) x[t] = make_float2(du[t] * x[t].x, du[t] * x[t].y);
                        else x[t] = cxmul(make_float2(g.x * du[t], g.y * du[t]), x[t]);
                        // (four steps at a time: all at once, the parts of the multipliers would take four registers a step)
                        if (T > 8 && t % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (DISC != DISC_BILINEAR) P = cexp_dt(sum_dl, cc.A2r, cc.Arev);     // product of the T multipliers
                    fast_part();
                    S = cxfma(a[0], xin, x[0]);
#pragma unroll
                    for (int t = 1; t < T; ++t) S = cxfma(a[t], S, x[t]);
                    if constexpr (DISC == DISC_BILINEAR) {
                        P = a[0];
#pragma unroll
                        for (int t = 1; t < T; ++t) P = cxmul(P, a[t]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    float2 Ct[2][4];                     // Cm four steps at a time, one such ahead
                    const float *lC = lB + (NS + n) * GE::ROW;
                    if constexpr (WANT_Y) read(lC, kFew, Ct[0]);
                    slow_part();
                    cchannel_scan<LPC>(P, S, xin);
                    fast_part();
                    if constexpr (TILE != kCkptInterval) {
                        const int64_t ll = l0 + li * T;
                        if (p.ckpt && li % ((int)kCkptInterval / T) == 0 && live && ll < L) {
                            const int64_t r = p.cu ? (int64_t)d : (int64_t)b * p.D + d;
                            p.ckpt[(r * nck + ck_first + ll / kCkptInterval) * N + h * NS + n] = xin;
                        }
                    }
                    if constexpr (WANT_Y) {
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            if (t % 4 == 0 && t + 4 < T) {
                                read(lC + (t / 2 + 2) * GE::Q, kFew, Ct[(t / 4 + 1) % 2]);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            const float2 c = Ct[t / 4 % 2][t % 4];
                            xin = cxfma(a[t], xin, x[t]);
                            yv[t] = __builtin_fmaf(c.x, xin.x, __builtin_fmaf(-c.y, xin.y, yv[t]));     // Re(C x)
                            if (t % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    if (li == LPC - 1) {                 // the channel's last lane ends on the tile's last step
                        sX[ch][h * NS + n] = WANT_Y ? xin : S;
                        if constexpr (!WANT_Y && LPC == 16) sP[ch][h * NS + n] = cxmul(sP[ch][h * NS + n], P);
                    }
                }
                edge_part();
                if constexpr (!EARLY) {
                    if (h + 1 == NH) fetch_z();
                    fetch_next();
                }
            }
        }
        if constexpr (WANT_Y) {
            {
                if (p.z) {
                    float zv[T];
                    if (!FULL && window) {
                        const int r = (fresh() % LPC) * T;
                        tail_shift<IO, T>(r_z, r - tail_window<T>(r, rem));
                    }
                    unpack_few<IO, T>(r_z, zv);
#pragma unroll
                    for (int t = 0; t < T; ++t) yv[t] *= zv[t] * sigmoid_fast(zv[t]);
                }
                if (live) {
                    IO *y = const_cast<IO *>(row(p.y, p.y_sb, p.y_sd, l0, FULL));
                    const int r = (fresh() % LPC) * T;
                    if constexpr (T == 4) store_few<IO, T>(y, r, rem, FULL || vec, yv);
                    else if constexpr (FULL) store_seg<IO, T>(y + r, 0, T, true, yv);
                    else store_seg<IO, T>(y, r, rem, vec, yv);
                }
            }
        }
    };
    const int64_t whole = vec ? L / TILE : 0, tilef = whole < tile0 ? tile0 : (whole < tile1 ? whole : tile1);
    int64_t tile = tile0;
    if (tile < tilef) {
        fetch_maps(tile, 0, std::true_type{});
        fetch_rows(tile, std::true_type{});
        for (; tile < tilef; ++tile) do_tile(tile, std::true_type{}, tile + 1 < tilef);
    }
    for (; tile < tile1; ++tile) {                   // the rest of the sequence (all of it without vector access)
        fetch_maps(tile, 0, std::false_type{});
        fetch_rows(tile, std::false_type{});
        do_tile(tile, std::false_type{}, false);
    }

    // every wavefront wrote the end states of its own channels
    for (int i = lane; i < CPW * N; i += 64) {
            const int c = w * CPW + i / N, n = i % N;
            if (din0 + c >= p.dpg) continue;
            const int64_t r = (int64_t)b * p.D + d0 + c;
            if (!WANT_Y && mode == MODE_AGG) {
                p.ws_P[(r * p.nchunks + chunk) * N + n] = sP[c][n];
                p.ws_S[(r * p.nchunks + chunk) * N + n] = sX[c][n];
            } else if (p.x_last && tile1 == ntiles) {
                p.x_last[r * N + n] = sX[c][n];
            }
        }
}

// ---------------------------------------------------------------- launchers
// The shape of a single pass, by the time each would take, as in the real forward pass (see fwd_shape in selective_fwd.hip): a
// tile costs its fixed part and a part for each state, and the same for each workgroup that shares the compute unit.  The
// costs (in 10 ns) are fitted to 850 calls of each type: 16 to 40960 rows, 64 to 32768 steps, N = 1 to 16, all schemes.
//   16 lanes: the fewest instructions; needs about 8000 rows (8 x 1536, L = 2048, N = 16, bf16: 250 us; 64 x 8: 296, 64 x 4: 389)
//   64 x 4:   the shortest tile and the quickest, for few rows (256 rows, L = 512, N = 16, bf16: 17.6 us, 16 lanes 34)
//   64 x 8:   in between (2 x 771 rows, L = 8192, N = 16, bf16: 247 us; 64 x 4: 333, 16 lanes 509)
// Over them the choice (with the chunk-carry path) is 0.3 % slower than the best, at most 1.18 times; with costs of an earlier form of the
// kernels, before their issue priorities, it was 1.3 % in float32 and 0.8 % in bfloat16, at most 1.6 times (3 x 1000 rows of 32768
// steps, N = 1, float32: 532 us in chunks, 327 in a single pass).
// A packed batch, whose lengths only the device knows, is priced by their mean, with half a tile more for the end of each sequence
// and fractions of a round, since its workgroups differ; its long sequences run on alone, hence costs of their own.  Over 250 batches
// of 2 to 96 sequences for each type 1.4 %, at most 1.28 times (with the batch's costs 6 %, at most 2.2: 6 sequences of 32768 steps in
// all, D = 1068, N = 1, bf16 207 us and 120).
enum class CFwdShape { l16, l64x4, l64x8 };
struct CFwdCost { int tile, state, wg, wg_state; };
static constexpr CFwdCost kCFwdCost[2][3] = {{{64, 45, 239, 38}, {32, 12, 44, 24}, {48, 14, 219, 67}},         // float32
                                             {{4, 99, 167, 12}, {42, 26, 32, 22}, {32, 35, 152, 67}}};         // bfloat16
static constexpr CFwdCost kCFwdPackedCost[2][3] = {{{233, 117, 241, 50}, {97, 58, 54, 22}, {90, 96, 246, 67}},
                                                   {{373, 109, 138, 54}, {130, 58, 40, 22}, {47, 131, 249, 57}}};
// share: workgroups of a compute unit
static double cfwd_cost(const CFwdCost &c, int64_t N, double tiles, double share) {
    return tiles * ((double)(c.tile + c.state * N) + share * (double)(c.wg + c.wg_state * N));
}
static double cfwd_time(int64_t maps, int64_t dpg, int64_t N, int64_t L, bool f32, CFwdShape shape, int64_t packed = 0) {
    static constexpr int steps[3] = {256, 256, 512}, channels[3] = {16, 4, 8};
    const int i = (int)shape;
    const int64_t wgs = maps * ((dpg + channels[i] - 1) / channels[i]);
    if (!packed) return cfwd_cost(kCFwdCost[f32 ? 0 : 1][i], N, (double)((L + steps[i] - 1) / steps[i]), (double)((wgs + kNumCU - 1) / kNumCU));
    const double tiles = (double)L / (double)(packed * steps[i]) + 0.5, share = (double)wgs / kNumCU;
    return cfwd_cost(kCFwdPackedCost[f32 ? 0 : 1][i], N, tiles < 1.0 ? 1.0 : tiles, share < 1.0 ? 1.0 : share);
}
static CFwdShape cfwd_shape(const CFwdParams &p, bool f32) {
    CFwdShape best = CFwdShape::l16;
    double least = 0.0;
    for (const CFwdShape shape : {CFwdShape::l16, CFwdShape::l64x4, CFwdShape::l64x8}) {
        const double t = cfwd_time((int64_t)p.B * p.bcg, p.dpg, p.N, p.L, f32, shape, p.cu ? p.B : 0);
        if (shape == CFwdShape::l16 || t < least) { least = t; best = shape; }
    }
    return best;
}

template <typename IO, int N, int DISC, int LPC, int T>
static hipError_t launch_cfwd_lanes(CFwdParams p, hipStream_t s) {
    using GE = CFwdGeom<LPC, T>;
    // tiles_per_chunk counts tiles of 256 steps; a single pass is one chunk whatever the tile
    if (p.nchunks == 1) p.tiles_per_chunk = (p.L + GE::TILE - 1) / GE::TILE;
    // the aggregate launch skips the last chunk: nobody needs its pair
    const dim3 grid(p.bcg * ((p.dpg + GE::CH - 1) / GE::CH), p.B, p.mode == MODE_AGG ? p.nchunks - 1 : p.nchunks), block(GE::W * 64);
    auto launch = [&](auto RANKED) {
        if (p.mode != MODE_AGG && p.y) hipLaunchKernelGGL((k_ss_cfwd<IO, N, DISC, true, LPC, T, RANKED>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((k_ss_cfwd<IO, N, DISC, false, LPC, T, RANKED>), grid, block, 0, s, p);
        return hipGetLastError();
    };
    // packed batches of more workgroups than the chip holds: longest sequences first
    if constexpr (LPC == 16 && N >= 8)
        if (ranked_sequences(p.cu, p.B, N, (int64_t)grid.x * grid.y)) return launch(std::true_type{});
    return launch(std::false_type{});
}
template <typename IO, int N, int DISC>
static hipError_t launch_cfwd_n(const CFwdParams &p, hipStream_t s) {
    if (p.mode == MODE_AGG && p.nchunks < 2) return hipSuccess;
    switch (p.nchunks == 1 ? cfwd_shape(p, sizeof(IO) == 4) : CFwdShape::l16) {      // (the chunk-carry path takes 16 lanes per channel)
        case CFwdShape::l64x4: return launch_cfwd_lanes<IO, N, DISC, 64, 4>(p, s);
        case CFwdShape::l64x8: return launch_cfwd_lanes<IO, N, DISC, 64, 8>(p, s);
        default: break;
    }
    return launch_cfwd_lanes<IO, N, DISC, 16, 16>(p, s);
}
template <typename IO, int DISC>
static hipError_t launch_cfwd_disc(const CFwdParams &p, hipStream_t s) {
    switch (p.N) {
        case 1: return launch_cfwd_n<IO, 1, DISC>(p, s);
        case 2: return launch_cfwd_n<IO, 2, DISC>(p, s);
        case 4: return launch_cfwd_n<IO, 4, DISC>(p, s);
        case 8: return launch_cfwd_n<IO, 8, DISC>(p, s);
        case 16: return launch_cfwd_n<IO, 16, DISC>(p, s);
    }
    return hipErrorInvalidValue;
}
template <typename IO>
static hipError_t launch_cfwd_io(const CFwdParams &p, int disc, hipStream_t s) {
    switch (disc) {
        case DISC_ZOH_S6: return launch_cfwd_disc<IO, DISC_ZOH_S6>(p, s);
        case DISC_ZOH: return launch_cfwd_disc<IO, DISC_ZOH>(p, s);
        case DISC_BILINEAR: return launch_cfwd_disc<IO, DISC_BILINEAR>(p, s);
        case DISC_DIRAC: return launch_cfwd_disc<IO, DISC_DIRAC>(p, s);
    }
    return hipErrorInvalidValue;
}
// float32 and bfloat16 are compiled side by side: selective_cplx_fwd_f32.hip includes this file for the former.
hipError_t launch_ss_cfwd_f32(const CFwdParams &p, int disc, hipStream_t s);
#ifdef LRNNX_CFWD_F32
hipError_t launch_ss_cfwd_f32(const CFwdParams &p, int disc, hipStream_t s) { return launch_cfwd_io<float>(p, disc, s); }
#else
hipError_t launch_ss_cfwd(const CFwdParams &p, int io_dtype, int disc, hipStream_t s) {
    return io_dtype == 1 ? launch_cfwd_io<bf16_t>(p, disc, s) : launch_ss_cfwd_f32(p, disc, s);
}

int cfwd_channels_per_workgroup() { return CFwdGeom<16, 16>::CH; }
int cfwd_tile_steps() { return CFwdGeom<16, 16>::TILE; }

// Whether the chunk-carry path is faster than the best single pass, by 3 % at least since it takes scratch (costs fitted as above,
// with bfloat16 I/O for both types: the query of the number of chunks does not know the type; the first two are those of
// the three launches).  N = 16, bf16: 16 rows of 8192 steps 36 us, 227 in a single pass; 768 rows of 32768 steps 460 and 919.
bool cfwd_chunks_pay(int64_t B, int64_t bcg, int64_t dpg, int64_t N, int64_t L) {
    static constexpr CFwdCost cost = {859, 105, 350, 104};
    const int64_t tiles = (L + cfwd_tile_steps() - 1) / cfwd_tile_steps();
    if (tiles < 2) return false;
    const int64_t channels = cfwd_channels_per_workgroup(), wgs = B * bcg * ((dpg + channels - 1) / channels) * tiles;
    const double chunked = cfwd_cost(cost, N, 1.0, (double)((wgs + kNumCU - 1) / kNumCU));
    constexpr double launch = 220;
    for (const CFwdShape shape : {CFwdShape::l16, CFwdShape::l64x4, CFwdShape::l64x8})
        if (cfwd_time(B * bcg, dpg, N, L, false, shape) + launch <= 1.03 * chunked) return false;
    return true;
}

// Chains the chunk aggregates of one (b,d,n): carry-in of chunk c+1 = P_c * carry-in of chunk c + S_c.
// ws_S[c] is replaced by the carry-in of chunk c.  A workgroup takes 16 such chains and up to 256 chunks at a time: 16 threads of
// a chain fold up to 16 consecutive pairs each, all read at once, and replay them from the state that the threads before
// hand on through LDS (see k_ss_carry in selective_fwd.hip; one after the other the reads take 0.2 us a chunk).
constexpr int kCCarryLen = 16;
__global__ __launch_bounds__(256) void k_ss_ccarry(const CFwdParams p) {
    __shared__ float2 sP[kCCarryLen][17], sS[kCCarryLen][17];
    const int chain = threadIdx.x % 16, seg = threadIdx.x / 16;
    const int64_t total = (int64_t)p.B * p.D * p.N, id = blockIdx.x * (int64_t)16 + chain;
    const int64_t i = id < total ? id : total - 1;       // (past the end: the last one again, nothing is written)
    const int64_t first = i / p.N * p.nchunks * p.N + i % p.N;
    float2 x = p.x0 ? p.x0[i] : make_float2(0.0f, 0.0f);
    for (int c0 = 0; c0 < p.nchunks; c0 += 16 * kCCarryLen) {
        const int left = p.nchunks - c0, most = left < 16 * kCCarryLen ? left : 16 * kCCarryLen;
        const int len = (most + 15) / 16, c1 = c0 + seg * len;
        float2 P[kCCarryLen], S[kCCarryLen], fP = make_float2(1.0f, 0.0f), fS = make_float2(0.0f, 0.0f);
#pragma unroll
        for (int k = 0; k < kCCarryLen; ++k) {
            P[k] = make_float2(1.0f, 0.0f); S[k] = make_float2(0.0f, 0.0f);
            if (k < len) {
                const int c = c1 + k < p.nchunks ? c1 + k : p.nchunks - 1;
                P[k] = p.ws_P[first + (int64_t)c * p.N];
                S[k] = p.ws_S[first + (int64_t)c * p.N];
            }
        }
#pragma unroll
        for (int k = 0; k < kCCarryLen; ++k) {
            const bool pair = k < len && c1 + k + 1 < p.nchunks;      // nothing follows the last chunk: its pair was not computed
            P[k] = make_float2(pair ? P[k].x : 1.0f, pair ? P[k].y : 0.0f);
            S[k] = make_float2(pair ? S[k].x : 0.0f, pair ? S[k].y : 0.0f);
            fS = cxfma(P[k], fS, S[k]);
            fP = cxmul(fP, P[k]);
        }
        sP[seg][chain] = fP; sS[seg][chain] = fS;
        __syncthreads();
        float2 mine = x;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            if (s == seg) mine = x;
            x = cxfma(sP[s][chain], x, sS[s][chain]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kCCarryLen; ++k) {
            if (k < len && c1 + k < p.nchunks && id < total) p.ws_S[first + (int64_t)(c1 + k) * p.N] = mine;
            mine = cxfma(P[k], mine, S[k]);
        }
    }
}
hipError_t launch_ss_ccarry(const CFwdParams &p, hipStream_t s) {
    const int64_t total = (int64_t)p.B * p.D * p.N;
    hipLaunchKernelGGL(k_ss_ccarry, dim3((unsigned)((total + 15) / 16)), dim3(256), 0, s, p);
    return hipGetLastError();
}
#endif

}  // namespace lrnnx
