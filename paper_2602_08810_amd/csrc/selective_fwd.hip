// Forward selective scan for gfx950 (Eq. 2 of the paper with diagonal, input-dependent
// A(k), B(k), C(k); S6 row of Table 1; discretisation fused in, Sec. 3).
//
// Mapping.  Time runs along the lanes: a channel takes LPC lanes (16 or 64), each of which owns T consecutive steps (4, 8
// or 16), so the [B,D,L] tensors are read and written with 16-byte accesses that are contiguous across the lanes of a
// channel.  The W wavefronts of a workgroup (each with 64/LPC channels) walk the same time tile of LPC T steps, so the
// tile of Bm/Cm (shared by all channels) is staged once per workgroup into LDS as fp32, 16 states at a time, in an order
// that makes every access conflict-free.  States never leave registers (Sec. 3: no hidden-state materialisation): for
// each n the lane folds its steps into one affine pair, the channel's lanes take an inclusive prefix over their pairs
// with DPP moves, and the lane replays its steps from the carried-in state, accumulating y = sum_n C x on the fly.  The
// state after the tile is the last lane's; it waits in LDS for the next tile of the same row.
//
// What bounds it: vector-ALU issue; with three wavefronts a SIMD the ALU is busy all the time.  Plain fp32 instructions of
// two wavefronts issue side by side if the parts of a state run at the priorities of scan_common.hpp (120 -> 109 us on the
// shape below; 2048 rows, L = 65536: 642 -> 585, and with two states at a time 562).  Per state update: 7 slots for the
// multiplier (a product and an exponential), the input, the fold, the replay and the projection, and 1/T of the rest:
// 13 to 16 for the prefix, its start and its end, and of 26 a step (softplus, gate, conversions) shared by the N states.
// Hence 16 steps per lane, one LDS address for all of Bm and Cm, and tiles known to be whole without any check.
// The next tile's inputs are fetched before the state loop where the registers allow, else after it.
// Mamba-block training shape (B = 8, D = 1536, N = 16, L = 2048, bf16, with gate and checkpoints): 97 to 103 us, 102
// between the events of the benchmark; before the priorities 109 from a graph and 122, and an earlier kernel of 64 lanes, 8 steps and
// 13 slots an update 143; B = 16, D = 2560, L = 4096 without gate: 608 to 632 us, before 640 and 823.
// See fwd_shape() for the choice of LPC and T.
//
// The same kernel serves the three launches of the chunk-carry path for long L / few
// rows (blockIdx.z = chunk): MODE_AGG returns each chunk's affine aggregate,
// k_ss_carry chains them, MODE_APPLY reruns the chunk from its true carry-in.
#include "kernels.hpp"
#include "scan_common.hpp"
#include <type_traits>

namespace lrnnx {

// Inclusive prefix over the LPC lanes of each channel, first lane first; on return S holds it and xin the prefix of the
// lane before (a channel's first lane keeps what it came with).  A DPP read needs two wait states after the write of its
// register: the s_nop cost the wavefront a cycle each and the other wavefronts of the SIMD nothing.  With KEEP_P the
// product is complete as well.
template <int LPC, bool KEEP_P>
__device__ __forceinline__ void channel_scan(float &P, float &S, float &xin) {
    static_assert(LPC == 16 || (LPC == 64 && !KEEP_P), "lanes of a channel");
#define LRNNX_S(CTRL) "v_fmac_f32_dpp %0, %0, %1 " CTRL "\n\ts_nop 1\n\t"
#define LRNNX_PS(CTRL) LRNNX_F_STATE(0, 1, CTRL) "s_nop 0\n\t"
#define LRNNX_SCAN(LAST, MOVES)                                                                                          \
    asm("s_nop 1\n\t" LRNNX_PS("row_shr:1" LRNNX_ALLROWS) LRNNX_PS("row_shr:2" LRNNX_ALLROWS)                            \
        LRNNX_PS("row_shr:4" LRNNX_ALLROWS) LAST MOVES                                                                   \
        : "+v"(S), "+v"(P), "+v"(xin))
#define LRNNX_SHR8(KIND) LRNNX_##KIND("row_shr:8" LRNNX_ALLROWS)
#define LRNNX_BC15(KIND) LRNNX_##KIND("row_bcast:15 row_mask:0xa bank_mask:0xf")   /* lane 15 of rows 0, 2 -> rows 1, 3 */
#define LRNNX_BC31(KIND) LRNNX_##KIND("row_bcast:31 row_mask:0xc bank_mask:0xf")   /* lane 31 -> rows 2, 3 */
#define LRNNX_MV(CTRL) "v_mov_b32_dpp %2, %0 " CTRL "\n\t"
    if constexpr (LPC == 16) {
        if constexpr (KEEP_P) LRNNX_SCAN(LRNNX_SHR8(PS), LRNNX_MV("row_shr:1" LRNNX_ALLROWS));
        else LRNNX_SCAN(LRNNX_SHR8(S), LRNNX_MV("row_shr:1" LRNNX_ALLROWS));
    } else {
        LRNNX_SCAN(LRNNX_SHR8(PS) LRNNX_BC15(PS) LRNNX_BC31(S), LRNNX_MV("wave_shr:1" LRNNX_ALLROWS));
    }
#undef LRNNX_MV
#undef LRNNX_BC31
#undef LRNNX_BC15
#undef LRNNX_SHR8
#undef LRNNX_SCAN
#undef LRNNX_PS
#undef LRNNX_S
}
// The same for two states, whose instructions are each other's wait states.
template <int LPC, bool KEEP_P>
__device__ __forceinline__ void channel_scan2(float (&P)[2], float (&S)[2], float (&xin)[2]) {
    static_assert(LPC == 16 || (LPC == 64 && !KEEP_P), "lanes of a channel");
#define LRNNX_S2(CTRL) "v_fmac_f32_dpp %0, %0, %1 " CTRL "\n\tv_fmac_f32_dpp %3, %3, %4 " CTRL "\n\ts_nop 0\n\t"
#define LRNNX_PS2(CTRL) LRNNX_F_STATE(0, 1, CTRL) LRNNX_F_STATE(3, 4, CTRL)
#define LRNNX_SCAN2(LAST, CTRL)                                                                                          \
    asm("s_nop 1\n\t" LRNNX_PS2("row_shr:1" LRNNX_ALLROWS) LRNNX_PS2("row_shr:2" LRNNX_ALLROWS)                          \
        LRNNX_PS2("row_shr:4" LRNNX_ALLROWS) LAST "v_mov_b32_dpp %2, %0 " CTRL "\n\tv_mov_b32_dpp %5, %3 " CTRL          \
        : "+v"(S[0]), "+v"(P[0]), "+v"(xin[0]), "+v"(S[1]), "+v"(P[1]), "+v"(xin[1]))
    if constexpr (LPC == 16) {
        if constexpr (KEEP_P) LRNNX_SCAN2(LRNNX_PS2("row_shr:8" LRNNX_ALLROWS), "row_shr:1" LRNNX_ALLROWS);
        else LRNNX_SCAN2(LRNNX_S2("row_shr:8" LRNNX_ALLROWS), "row_shr:1" LRNNX_ALLROWS);
    } else {
        LRNNX_SCAN2(LRNNX_PS2("row_shr:8" LRNNX_ALLROWS) LRNNX_PS2("row_bcast:15 row_mask:0xa bank_mask:0xf")
                    LRNNX_S2("row_bcast:31 row_mask:0xc bank_mask:0xf"), "wave_shr:1" LRNNX_ALLROWS);
    }
#undef LRNNX_SCAN2
#undef LRNNX_PS2
#undef LRNNX_S2
}

// WG: wavefronts of a workgroup where a shape has more than one number of them (0: the usual one)
template <int LPC, int T, int WG = 0> struct FwdGeom {
    static constexpr int W = WG ? WG : LPC * T / 64 < 8 ? LPC * T / 64 : 8;      // wavefronts of a workgroup
    static constexpr int CPW = 64 / LPC;             // channels of a wavefront
    static constexpr int CH = W * CPW;               // channels of a workgroup
    static constexpr int TILE = LPC * T;
    static constexpr int Q = 4 * LPC + 256 / T;      // a quarter (T = 16), half (T = 8) or all (T = 4) of a staged row, see below
    static constexpr int ROW = Q * (T / 4);
};

// Workgroups that share a compute unit: three of four wavefronts with 16 lanes per channel (168 registers, three wavefronts a
// SIMD); with 64 lanes four of four wavefronts (4 steps) or two of eight (8 steps: 75 KB of LDS each), at 128 registers four a
// SIMD; one of twelve (8 steps, three wavefronts a SIMD); one of eight with 16 steps, whose staged tile takes more than half of the LDS.
// RANKED: a packed batch whose workgroups rank the sequences (ranked_sequences)
template <typename IO, int N, int DISC, bool WANT_Y, bool CKPT, int LPC, int TM, bool RANKED, int WG = 0>
__global__ __launch_bounds__((FwdGeom<LPC, TM, WG>::W * 64), (TM == 16 ? (LPC == 16 ? 3 : 2) : WG ? 3 : 4)) void k_ss_fwd(const FwdParams p) {
    using GE = FwdGeom<LPC, TM, WG>;
    constexpr int W = GE::W, CPW = GE::CPW, CH = GE::CH, TILE = GE::TILE, NT = W * 64 < TILE ? W * 64 : TILE;
    constexpr int RPT = TILE / NT;                   // rows of the maps a thread stages (the first NT threads do)
    constexpr int NS = N > 16 ? 16 : N, NH = N / NS; // states staged at a time, and how often
    constexpr bool EARLY = sizeof(IO) == 2 ? LPC > 16 || N <= 8 : LPC > 16 && N <= 8;
    constexpr bool LATE_Z = sizeof(IO) == 4 && TM == 16 && LPC == 16;
    constexpr bool AGG = !WANT_Y && !CKPT;           // the aggregate launch of the chunk-carry path
    // A sequence's last tile with half of its steps or fewer takes a half or a quarter of them a lane (11 x 1059 rows of 339 steps,
    // N = 16, bf16: call 35.9 -> 28.8 us).  With 16 lanes a channel only: a tile of 64 lanes of 4 steps has nothing to halve, and
    // the shapes with longer tiles are for long rows, which have one such tile.
    constexpr bool SHORT = LPC == 16;
    // Two states at a time: their chains (folds, scan, replay) fill each other's latencies, which counts where few wavefronts share a
    // SIMD: 2048 rows, L = 65536, N = 16, bf16 577 -> 564 us, 64 rows of 16384 steps 21.5 -> 20.5, states alone (B=16, D=2560,
    // L=4096) 432 -> 407.  Not where it takes the registers of a wavefront (16 lanes with outputs: 110 -> 124 us, 30 spilled), with
    // few states (N = 8: up to 6 % longer), and in float32 with 8 steps (2 % longer).
    constexpr bool PAIR = NS == 16 && (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) &&
                          (!WANT_Y || (LPC == 64 && !(TM == 8 && sizeof(IO) == 4)));
    static_assert(TILE % kCkptInterval == 0 && RPT * NT == TILE, "tile shape");
    __shared__ __attribute__((aligned(16))) float sBC[WANT_Y ? 2 * NS : NS + 1][GE::ROW];   // Bm, Cm
    __shared__ __attribute__((aligned(16))) float sA[CH + 1][N], sX[CH + 2][N];    // A; the state entering the next tile, and zeros
    __shared__ float sP[AGG ? CH : 1][N];            // aggregate: product of the multipliers so far

    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane % LPC;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.y;
    // a workgroup takes CH consecutive channels of ONE Bm/Cm group (it stages that group's maps in LDS)
    const int blk_per_grp = (p.dpg + CH - 1) / CH;
    const int grp = blockIdx.x / blk_per_grp;
    const int din0 = (blockIdx.x % blk_per_grp) * CH;
    const int ch = w * CPW + lane / LPC;             // this lane's channel of the workgroup
    const bool live = din0 + ch < p.dpg;
    const bool busy = din0 + w * CPW < p.dpg;        // wave-uniform: the wavefront has a channel at all
    const int d0 = grp * p.dpg + din0;
    const int d = grp * p.dpg + (live ? din0 + ch : p.dpg - 1);
    const int chunk = blockIdx.z;
    // packed variable-length mode (p.cu != nullptr, see seq_span): I/O rows have no batch stride, the maps are [G, p.L, N]
    int64_t L = p.L, toff = 0, bs = b;
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
    // from holding a register for each address throughout.
    auto fresh = [&]() { unsigned t = tid; asm volatile("" : "+v"(t)); return t; };
    auto row = [&](const void *base, int64_t sb, int64_t sd, int64_t l) {
        int c = din0 + w * CPW + (fresh() & 63) / LPC;
        c = c < p.dpg ? c : p.dpg - 1;
        return reinterpret_cast<const IO *>(base) + (bs * sb + (int64_t)(grp * p.dpg + c) * sd + toff + l);
    };
    const int64_t bc0 = ((bs * p.bcg + grp) * p.L + toff) * N;       // first element of the maps of this sequence
    const IO *Bm = reinterpret_cast<const IO *>(p.Bm) + bc0;
    const IO *Cm = reinterpret_cast<const IO *>(p.Cm) + bc0;
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
        float x = 0.0f;
        if (mode == (WANT_Y ? MODE_APPLY : MODE_CKPT_APPLY)) x = p.ws_S[(r * p.nchunks + chunk) * N + n];
        else if (mode != MODE_AGG && p.x0) x = p.x0[r * N + n];
        sX[c][n] = x;
        if constexpr (AGG) sP[c][n] = 1.0f;
    }
    if (lane < N) sX[CH][lane] = 0.0f;               // (every wavefront: the same value)
    const bool stages = NT == W * 64 || w < NT / 64;

    // A staged row of Bm or Cm: step 4 q + i of lane l (of TM) at q Q + 4 l + i.  The reads, 16 bytes from each lane,
    // are contiguous over the lanes and all share one address; Q leaves a gap of 256 / TM so that the 64 consecutive steps
    // which a wavefront stages at once fall into 64 banks.
    // ---- the inputs of a tile, raw.  Those of a whole tile (FULL: nothing to check per element) are fetched ahead, once
    // the state loop of the tile before is done, and used after its epilogue.
    // the last steps of the sequence: see tail_window (64 x 16 is for long rows, which have one such tile: left out there,
    // where the mere presence of that code cost the main loop 2 %)
    const bool window = GE::TILE <= 512 && vec && L >= TM;
    RawFew<IO, TM> r_u, r_dl;
    RawFew<IO, NS> r_B[RPT], r_C[WANT_Y ? RPT : 1];
    auto fetch_rows = [&](int64_t tile, auto FULL, auto &r_u, auto &r_dl) {
        constexpr int T = std::remove_reference_t<decltype(r_u)>::COUNT;
        const int64_t l0 = tile * TILE;
        const IO *u = row(p.u, p.u_sb, p.u_sd, l0), *dl = row(p.delta, p.dl_sb, p.dl_sd, l0);
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
        const int64_t l0 = tile * TILE;
        if (!stages) return;
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            int64_t l = l0 + (int)(fresh() + k * NT);
            if constexpr (!FULL) l = l < L ? l : L - 1;  // rows past the sequence: the last one again, discarded below
            load_few_raw<IO, NS>(Bm + (l * N + h * NS), 0, NS, true, r_B[k]);
            if constexpr (WANT_Y) load_few_raw<IO, NS>(Cm + (l * N + h * NS), 0, NS, true, r_C[k]);
        }
    };
    // after the last tile: these registers hold nothing any more (without it they would stay occupied throughout)
    auto forget = [](auto &r) {
#pragma unroll
        for (uint32_t &x : r.w) asm volatile("" : "=v"(x));
    };
    auto forget_maps = [&]() {
#pragma unroll
        for (int k = 0; k < RPT; ++k) { forget(r_B[k]); if constexpr (WANT_Y) forget(r_C[k]); }
    };
    // STEPS: steps of a lane, fewer in a short tile (the last one of a sequence), whose rows are fetched here
    auto do_tile = [&](int64_t tile, auto FULL, auto STEPS, bool ahead) {
        constexpr int T = STEPS;
        RawFew<IO, T> t_u, t_dl;
        auto &q_u = [&]() -> auto & { if constexpr (T == TM) return r_u; else return t_u; }();
        auto &q_dl = [&]() -> auto & { if constexpr (T == TM) return r_dl; else return t_dl; }();
        if constexpr (T != TM) { if (busy) fetch_rows(tile, FULL, t_u, t_dl); }
        const int64_t l0 = tile * TILE;
        const int rem = FULL ? TILE : (L - l0 < TILE ? (int)(L - l0) : TILE);
        float dl[T], du[T], yv[T], sum_dl = 0.0f;    // du: Delta*u for S6, u for the other schemes
        RawFew<IO, T> r_z;
        auto fetch_z = [&]() {
            if constexpr (WANT_Y) {
                if (!p.z) return;
                const IO *z = row(p.z, p.z_sb, p.z_sd, l0);
                const int r = (fresh() % LPC) * T;
                if constexpr (FULL) load_few_raw<IO, T>(z + r, 0, T, true, r_z);
                else if (window) load_few_raw<IO, T>(z + tail_window<T>(r, rem), 0, T, true, r_z);
                else load_few_raw<IO, T>(z, r, rem, vec, r_z);
            }
        };
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            // ---- stage the maps of NS states (all wavefronts) as fp32
            __syncthreads();
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                const unsigned r = fresh() + k * NT, q = (r % T) / 4;
                if ((T != TM && r >= LPC * T) || !stages) break;
                const unsigned off = q * GE::Q + (r / T) * 4 + (r % 4);
                float v[NS];
                unpack_few<IO, NS>(r_B[k], v);
#pragma unroll
                for (int n = 0; n < NS; ++n) sBC[n][off] = FULL || (int)r < rem ? v[n] : 0.0f;
                if constexpr (WANT_Y) {
                    unpack_few<IO, NS>(r_C[k], v);
#pragma unroll
                    for (int n = 0; n < NS; ++n) sBC[NS + n][off] = FULL || (int)r < rem ? v[n] : 0.0f;
                }
            }
            if constexpr (CKPT && TILE == kCkptInterval) {           // the state entering the tile is the carried one
                if (busy && h == 0)
                    for (int i = fresh() & 63; i < CPW * N; i += 64) {
                        const int c = w * CPW + i / N;
                        const int64_t r = p.cu ? (int64_t)(d0 + c) : (int64_t)b * p.D + d0 + c;
                        if (din0 + c < p.dpg) p.ckpt[(r * nck + ck_first + tile) * N + i % N] = sX[c][i % N];
                    }
            }
            __syncthreads();
            if (busy && h == 0) {
                // ---- this lane's steps of Delta, Delta u and D u
                if (!FULL && window) {
                    const int r = (fresh() % LPC) * T, by = r - tail_window<T>(r, rem);
                    tail_shift<IO, T>(q_u, by);
                    tail_shift<IO, T>(q_dl, by);
                }
                unpack_few<IO, T>(q_u, du);
                unpack_few<IO, T>(q_dl, dl);
#pragma unroll
                for (int t = 0; t < T; ++t) asm volatile("" : "+v"(du[t]), "+v"(dl[t]));
                if constexpr (!LATE_Z) fetch_z();
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
            auto fetch_next = [&](auto ROWS) {
                if (h + 1 < NH) { fetch_maps(tile, h + 1, FULL); return; }
                if (FULL && ahead) {
                    fetch_maps(tile + 1, 0, FULL);
                    if constexpr (ROWS && T == TM) fetch_rows(tile + 1, FULL, r_u, r_dl);
                } else { forget_maps(); forget(r_u); forget(r_dl); }
            };
            if (busy) {
                if constexpr (EARLY) fetch_next(std::true_type{});
                // The LDS reads run ahead of their use: Bm, A and the carried state of the next n during this one, Cm from the
                // top of the pass to its end.
                auto read = [&](const float *m, float *v) {
#pragma unroll
                    for (int q = 0; q < T / 4; ++q) {
                        const float4 f = *reinterpret_cast<const float4 *>(m + q * GE::Q);
                        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
                    }
                };
                const float *lB = &sBC[0][li * 4], *lA = &sA[ch][h * NS];
                const float *lX = &sX[li == 0 ? ch : CH][h * NS];    // the carried state enters through the channel's first lane
                auto checkpoint = [&](int n, float xin) {            // the state entering this lane's first step
                    if constexpr (CKPT && TILE != kCkptInterval) {
                        const int64_t ll = l0 + li * T;
                        if (li % ((int)kCkptInterval / T) == 0 && live && ll < L) {
                            const int64_t r = p.cu ? (int64_t)d : (int64_t)b * p.D + d;
                            p.ckpt[(r * nck + ck_first + ll / kCkptInterval) * N + h * NS + n] = xin;
                        }
                    }
                };
                auto leave = [&](int n, float x, float P) {
                    if (li == LPC - 1) {                 // the channel's last lane ends on the tile's last step
                        sX[ch][h * NS + n] = x;
                        if constexpr (AGG) sP[ch][h * NS + n] *= P;
                    }
                };
                if constexpr (PAIR) {
                    float An[2] = {lA[0], lA[1]}, xn[2] = {lX[0], lX[1]};
#pragma unroll 1
                    for (int n = 0; n < NS; n += 2) {
                        // Bm's reads are under way while the multipliers are formed, Cm's (four steps at a time, one such
                        // ahead) during the scan; A and the carried state one pair ahead
                        const ACoef ac[2] = {make_acoef<DISC>(An[0]), make_acoef<DISC>(An[1])};
                        float xin[2] = {xn[0], xn[1]}, a[2][T], x[2][T], P[2], S[2];
                        read(lB + n * GE::ROW, x[0]);
                        read(lB + (n + 1) * GE::ROW, x[1]);
                        An[0] = lA[n + 2]; An[1] = lA[n + 3]; xn[0] = lX[n + 2]; xn[1] = lX[n + 3];    // (after the last: not used)
                        slow_part();
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            float g;
#pragma unroll
                            for (int t = 0; t < T; ++t) disc_ag<DISC>(dl[t], ac[j], a[j][t], g);
                            P[j] = exp2_fast(sum_dl * ac[j].A2);         // product of the T multipliers
                        }
                        fast_part();
#pragma unroll
                        for (int t = 0; t < T; ++t)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                x[j][t] *= du[t];
                                S[j] = __builtin_fmaf(a[j][t], t ? S[j] : xin[j], x[j][t]);
                            }
                        float Ct[2][2][4];
                        const float *lC = lB + (NS + n) * GE::ROW;
                        auto read_C = [&](int q) {
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const float4 f = *reinterpret_cast<const float4 *>(lC + j * GE::ROW + q * GE::Q);
                                float *c = Ct[q % 2][j];
                                c[0] = f.x; c[1] = f.y; c[2] = f.z; c[3] = f.w;
                            }
                        };
                        if constexpr (WANT_Y) read_C(0);
                        slow_part();
                        channel_scan2<LPC, AGG>(P, S, xin);
                        fast_part();
#pragma unroll
                        for (int j = 0; j < 2; ++j) checkpoint(n + j, xin[j]);
                        if constexpr (WANT_Y) {
#pragma unroll
                            for (int t = 0; t < T; ++t) {
                                if (t % 4 == 0 && t + 4 < T) read_C(t / 4 + 1);
#pragma unroll
                                for (int j = 0; j < 2; ++j) {
                                    xin[j] = __builtin_fmaf(a[j][t], xin[j], x[j][t]);
                                    yv[t] = __builtin_fmaf(Ct[t / 4 % 2][j][t % 4], xin[j], yv[t]);
                                }
                            }
                        }
#pragma unroll
                        for (int j = 0; j < 2; ++j) leave(n + j, WANT_Y ? xin[j] : S[j], P[j]);
                    }
                } else {
                    float Bt[T], Ct[T], An = lA[0], xn = lX[0];
                    read(lB, Bt);
#pragma unroll 1
                    for (int n = 0; n < NS; ++n) {
                        const ACoef ac = make_acoef<DISC>(An);
                        float xin = xn;
                        auto next_n = [&]() {                // (after the last n: one row further, not used)
                            An = lA[n + 1]; xn = lX[n + 1]; read(lB + (n + 1) * GE::ROW, Bt);
                        };
                        float a[T], x[T], P, S;
                        if constexpr (WANT_Y) read(lB + (NS + n) * GE::ROW, Ct);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) x[t] = du[t] * Bt[t];
                            else x[t] = Bt[t];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) next_n();
                        slow_part();
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            float g;
                            disc_ag<DISC>(dl[t], ac, a[t], g);
                            if constexpr (DISC != DISC_ZOH_S6 && DISC != DISC_DIRAC) x[t] *= g * du[t];
                        }
                        if constexpr (DISC != DISC_ZOH_S6 && DISC != DISC_DIRAC) next_n();
                        S = __builtin_fmaf(a[0], xin, x[0]);
#pragma unroll
                        for (int t = 1; t < T; ++t) S = __builtin_fmaf(a[t], S, x[t]);
                        if constexpr (DISC == DISC_BILINEAR) {
                            P = a[0];
#pragma unroll
                            for (int t = 1; t < T; ++t) P *= a[t];
                        } else P = exp2_fast(sum_dl * ac.A2);            // product of the T multipliers
                        channel_scan<LPC, AGG>(P, S, xin);
                        fast_part();
                        checkpoint(n, xin);
                        if constexpr (WANT_Y) {
#pragma unroll
                            for (int t = 0; t < T; ++t) {
                                xin = __builtin_fmaf(a[t], xin, x[t]);
                                yv[t] = __builtin_fmaf(Ct[t], xin, yv[t]);
                            }
                        }
                        leave(n, WANT_Y ? xin : S, P);
                    }
                }
                if (LATE_Z && h + 1 == NH) fetch_z();
                if constexpr (!EARLY) fetch_next(std::true_type{});
            } else fetch_next(std::false_type{});
        }
        if constexpr (WANT_Y) {
            if (busy) {
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
                    IO *y = const_cast<IO *>(row(p.y, p.y_sb, p.y_sd, l0));
                    const int r = (fresh() % LPC) * T;
                    if constexpr (T < 8) store_few<IO, T>(y, r, rem, FULL || vec, yv);
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
        if (busy) fetch_rows(tile, std::true_type{}, r_u, r_dl);
        for (; tile < tilef; ++tile) do_tile(tile, std::true_type{}, std::integral_constant<int, TM>{}, tile + 1 < tilef);
    }
    for (; tile < tile1; ++tile) {                   // the rest of the sequence (all of it without vector access)
        fetch_maps(tile, 0, std::false_type{});
        if constexpr (SHORT) {
            const int64_t left = L - tile * TILE;
            if (left <= TILE / 4) { do_tile(tile, std::false_type{}, std::integral_constant<int, SHORT ? TM / 4 : TM>{}, false); continue; }
            if (left <= TILE / 2) { do_tile(tile, std::false_type{}, std::integral_constant<int, SHORT ? TM / 2 : TM>{}, false); continue; }
        }
        if (busy) fetch_rows(tile, std::false_type{}, r_u, r_dl);
        do_tile(tile, std::false_type{}, std::integral_constant<int, TM>{}, false);
    }

    // every wavefront wrote the end states of its own channels
    if (busy)
        for (int i = lane; i < CPW * N; i += 64) {
            const int c = w * CPW + i / N, n = i % N;
            if (din0 + c >= p.dpg) continue;
            const int64_t r = (int64_t)b * p.D + d0 + c;
            if constexpr (AGG) {
                p.ws_P[(r * p.nchunks + chunk) * N + n] = sP[c][n];
                p.ws_S[(r * p.nchunks + chunk) * N + n] = sX[c][n];
            } else if (p.x_last && tile1 == ntiles) {
                p.x_last[r * N + n] = sX[c][n];
            }
        }
}

// ---------------------------------------------------------------- launchers
// The shape of a single pass, by the time each would take.  A tile costs its fixed part and a part for each state (staging,
// barriers, the latency of a wavefront that is alone on its SIMD), and the same for each workgroup that shares the compute
// unit; the costs (in 10 ns) are fitted to 16 to 40960 rows of 64 to 65536 steps with N = 1 to 32.
//   16 lanes: the fewest instructions; needs about 8000 rows for three workgroups a compute unit
//             (8 x 1536 rows, L = 2048, N = 16, bf16: 97 us; 64 x 8: 104, 64 x 16: 121, 64 x 4: 133)
//   64 x 4:   the shortest tile and the quickest, for rows of up to 256 steps (256 rows, L = 256, N = 16, float32: 6.2 us,
//             64 x 8 10.0, 16 lanes 10.7) and with few states, where memory is the bound, for many rows (16 x 2560 rows,
//             L = 2048, N = 4, float32: 247 us, 16 lanes 274)
//   64 x 8:   a few thousand rows (4096 rows, L = 2048, N = 16, float32: 46 us; 16 lanes 73, 64 x 4 65)
//   64 x 8, twelve wavefronts: where workgroups of eight channels would be a little more than one a compute unit, which is as long as two, and
//             those of twelve are not (2049 to 3072 rows; one workgroup a compute unit, three wavefronts a SIMD instead of four; 2313 rows,
//             L = 1531, N = 16, float32: 36.3 -> 30.2 us, bf16 32.4 -> 26.9; 3000 rows, L = 4096: 83.0 -> 72.1, 72.4 -> 62.6; with nine or
//             ten wavefronts the same, with thirteen to sixteen, four on a SIMD, what eight take).  Of these rows not few tiles of 512 steps the last of which is at
//             most half full: 64 x 4 leaves that half out (2600 rows, L = 768, N = 16, float32: 20.1 us, twelve wavefronts 23.1, eight 26.7); nor, with
//             eight states or for states alone, for a 257th workgroup of one to four channels, which costs the one beside it little (2049 rows,
//             L = 5000, N = 8, float32: 53.3 us with eight wavefronts, 57.8).  3024 calls of 2049 to 3072 rows, 256 to 12000 steps, N = 8 to 32, both
//             types: 0.918 of the time without this shape (geometric mean), 11 slower by more than 2 %, at most 1.06 times (without those conditions 0.931, 524
//             and 1.28); 756 passes over states alone: 0.918, 3 and 1.02 (0.932, 136 and 1.21)
//   64 x 16:  one workgroup a compute unit (its tile takes the LDS), so at most 2048 rows, but fewer instructions
//             than 64 x 8 (768 rows, L = 32768, N = 16, bf16: 284 us; 64 x 8: 328)
// The costs were fitted before the issue priorities and the pairs of states changed the shapes unequally.  With the present kernels the
// choice is 1.8 % (float32) and 0.7 % (bfloat16) slower than the best of the first four and the chunked path over 729 calls of each type (before there was a fifth), at
// most 1.30 times: N = 1 on 16 to 1500 rows of 1531 steps takes 64 x 16, 11.4 us for the 8.8 of 64 x 4.
enum class FwdShape { l16, l64x4, l64x8, l64x16, l64x8w12 };
struct FwdCost { int tile, state, wg, wg_state; };
static constexpr FwdCost kFwdCost[2][5] = {{{0, 20, 249, 17}, {22, 12, 52, 8}, {0, 6, 183, 27}, {0, 0, 215, 65}, {0, 6, 296, 44}},          // float32
                                           {{19, 16, 136, 17}, {40, 9, 31, 7}, {0, 8, 132, 24}, {0, 0, 170, 53}, {0, 8, 214, 39}}};         // bfloat16
static constexpr FwdShape kFwdShapes[5] = {FwdShape::l16, FwdShape::l64x4, FwdShape::l64x8, FwdShape::l64x16, FwdShape::l64x8w12};
static int64_t fwd_cost(const FwdCost &c, int64_t N, int64_t tiles, int64_t wgs) {
    const int64_t share = (wgs + kNumCU - 1) / kNumCU;   // workgroups of a compute unit
    return tiles * (c.tile + c.state * N + share * (c.wg + c.wg_state * N));
}
static int64_t fwd_time(int64_t maps, int64_t dpg, int64_t N, int64_t L, bool f32, FwdShape shape) {
    static constexpr int steps[5] = {256, 256, 512, 1024, 512}, channels[5] = {16, 4, 8, 8, 12};
    const int i = (int)shape;
    const int64_t wgs = maps * ((dpg + channels[i] - 1) / channels[i]);
    if (shape == FwdShape::l64x16 && wgs > kNumCU) return INT64_MAX;
    if (shape == FwdShape::l64x8w12 && (wgs > kNumCU || N < 8 || maps * ((dpg + 7) / 8) <= kNumCU)) return INT64_MAX;
    return fwd_cost(kFwdCost[f32 ? 0 : 1][i], N, (L + steps[i] - 1) / steps[i], wgs);
}
// `outputs`: else the pass writes states alone.  `few`: up to there 64 x 4 is the faster where the last tile of 512 is at most half full (its time over that of
// twelve wavefronts, geometric means: float32 N = 8 0.82 at 768 steps, 0.94 at 2304, 1.00 at 3073; N = 16 0.85, 0.97 at 1280, 1.03 at 1537; N = 32 0.89, 0.97,
// 1.03; bf16 N = 8 0.84, 0.92 at 1280, 0.97 at 1792, 1.02 at 2049; N = 16 0.86, 0.96, 1.03 at 1537; N = 32 0.92, 1.02; states alone 0.86 to 0.99 at 768).
static FwdShape fwd_shape(int64_t maps, int64_t dpg, int64_t N, int64_t L, bool f32, bool outputs) {
    const bool twelve = fwd_time(maps, dpg, N, L, f32, FwdShape::l64x8w12) != INT64_MAX;
    const bool one_more = twelve && (N == 8 || !outputs) && maps * ((dpg + 7) / 8) == kNumCU + 1 && (dpg + 7) % 8 < 4;
    const int64_t few = !outputs ? (N > 8 ? 768 : 1280) : f32 ? (N > 8 ? 1280 : one_more ? 1792 : 3328) : N > 16 ? 768 : N > 8 ? 1280 : 1792;
    const bool half = twelve && (L + 511) % 512 < 256 && L <= few;
    FwdShape best = FwdShape::l16;
    int64_t least = INT64_MAX;
    for (const FwdShape shape : kFwdShapes) {
        if (half && (shape == FwdShape::l64x8 || shape == FwdShape::l64x8w12)) continue;
        const int64_t t = fwd_time(maps, one_more && shape == FwdShape::l64x8 ? 8 * kNumCU : dpg, N, L, f32, shape);       // (then maps is 1)
        if (t < least) { least = t; best = shape; }
    }
    return best;
}
// The shape for a packed batch, whose lengths only the device knows: as a rule 64 lanes of 4 steps, whose tiles of 256
// steps spend little past the ends of short sequences while a long one does not run on alone for long (31 sequences of 705
// steps on average, 522 channels, N = 8, bf16: 95 us; 16 lanes 122, 64 x 8 102).  With so many rows that the chip
// stays full, 16 lanes, which take fewer instructions: from 24576 rows (24 sequences, 1536 channels, N = 16, bf16: 141 us,
// 64 x 4: 195), of sequences of hardly a tile from 12288 (17 of 206 steps on average, 1068 channels: 38 us, 54), in
// float32 with 16 states or more from 14336 (6 sequences, 2560 channels, 8192 steps, N = 16: 153 us, 64 x 4: 197; 24
// sequences, 512 channels, 32768 steps: 289, 218), of sequences of hardly a tile from 8192 (24 of 85 steps, 512 channels: 29,
// 32).  With fewer states memory is the bound in float32, and 16 lanes, which fetch later, do not keep enough of it in flight
// (24 sequences of 8192 steps in all, 1536 channels, N = 4: 70 us, 64 x 4: 58) except on very many rows of short sequences (24
// of 85 steps, 2560 channels: 50, 58).  Long sequences take the longer tiles: 64 x 8 (5 of 3056 steps
// on average, 1724 channels: 173 us, 64 x 4: 188), very few rows of very long ones 64 x 16 (2 sequences of up to
// 23848 steps, 363 channels: 152 us, 64 x 4: 186).  (Figures of the kernels before their issue priorities.  With the present ones the choice is
// 1.8 % slower than the best in float32 and 2.8 % in bfloat16 over 236 batches of each type, at most 1.32 times: 24 sequences of
// 341 steps on average, 512 channels, N = 32, float32 82 us, 16 lanes 62.)
static FwdShape packed_shape(const FwdParams &p, bool f32) {
    const int64_t rows = (int64_t)p.B * p.D, mean = p.L / p.B;
    const bool brief = mean <= 256;
    const int64_t full = !f32 ? (brief ? 12288 : 24576) : p.N >= 16 ? (brief ? 8192 : 14336) : brief ? 32768 : INT64_MAX;
    if (rows >= full) return FwdShape::l16;
    if (rows <= 1024 && mean >= 4096) return FwdShape::l64x16;
    return rows >= 2048 && mean >= 2048 ? FwdShape::l64x8 : FwdShape::l64x4;
}

template <typename IO, int N, int DISC, int LPC, int T, int WG = 0>
static hipError_t launch_fwd_lanes(FwdParams p, hipStream_t s) {
    using GE = FwdGeom<LPC, T, WG>;
    // tiles_per_chunk counts tiles of 256 steps; a single pass is one chunk whatever the tile
    if (p.nchunks == 1) p.tiles_per_chunk = (p.L + GE::TILE - 1) / GE::TILE;
    dim3 grid(p.bcg * ((p.dpg + GE::CH - 1) / GE::CH), p.B, p.mode == MODE_AGG ? p.nchunks - 1 : p.nchunks);
    const bool want_y = (p.mode == MODE_FULL || p.mode == MODE_APPLY);
    const dim3 block(GE::W * 64);
    auto launch = [&](auto RANKED) {
        if (want_y && p.ckpt) hipLaunchKernelGGL((k_ss_fwd<IO, N, DISC, true, true, LPC, T, RANKED, WG>), grid, block, 0, s, p);
        else if (want_y) hipLaunchKernelGGL((k_ss_fwd<IO, N, DISC, true, false, LPC, T, RANKED, WG>), grid, block, 0, s, p);
        else if (p.ckpt) hipLaunchKernelGGL((k_ss_fwd<IO, N, DISC, false, true, LPC, T, RANKED, WG>), grid, block, 0, s, p);
        else if constexpr (LPC == 16 && !RANKED) hipLaunchKernelGGL((k_ss_fwd<IO, N, DISC, false, false, LPC, T, RANKED, WG>), grid, block, 0, s, p);
        else return hipErrorInvalidValue;                // the chunk-carry path takes 16 lanes per channel, and no packed batches
        return hipGetLastError();
    };
    // packed batches of more workgroups than the chip holds: longest sequences first
    if constexpr (LPC == 16 && N >= 8)
        if (ranked_sequences(p.cu, p.B, N, (int64_t)grid.x * grid.y)) return launch(std::true_type{});
    return launch(std::false_type{});
}

template <typename IO, int N, int DISC>
static hipError_t launch_fwd_n(const FwdParams &p, hipStream_t s) {
    // the aggregate launch skips the last chunk: nobody needs its pair
    if (p.mode == MODE_AGG && p.nchunks < 2) return hipSuccess;
    switch (p.cu ? packed_shape(p, sizeof(IO) == 4) : p.nchunks == 1 ? fwd_shape((int64_t)p.B * p.bcg, p.dpg, p.N, p.L, sizeof(IO) == 4, p.mode == MODE_FULL) : FwdShape::l16) {
        case FwdShape::l64x4: return launch_fwd_lanes<IO, N, DISC, 64, 4>(p, s);
        case FwdShape::l64x8: return launch_fwd_lanes<IO, N, DISC, 64, 8>(p, s);
        case FwdShape::l64x16: return launch_fwd_lanes<IO, N, DISC, 64, 16>(p, s);
        case FwdShape::l64x8w12:
            if constexpr (N >= 8) return launch_fwd_lanes<IO, N, DISC, 64, 8, 12>(p, s);
            break;
        default: break;
    }
    return launch_fwd_lanes<IO, N, DISC, 16, 16>(p, s);
}

template <typename IO, int DISC>
static hipError_t launch_fwd_disc(const FwdParams &p, hipStream_t s) {
    switch (p.N) {
        case 1: return launch_fwd_n<IO, 1, DISC>(p, s);
        case 2: return launch_fwd_n<IO, 2, DISC>(p, s);
        case 4: return launch_fwd_n<IO, 4, DISC>(p, s);
        case 8: return launch_fwd_n<IO, 8, DISC>(p, s);
        case 16: return launch_fwd_n<IO, 16, DISC>(p, s);
        case 32: return launch_fwd_n<IO, 32, DISC>(p, s);
    }
    return hipErrorInvalidValue;
}

template <typename IO>
static hipError_t launch_fwd_io(const FwdParams &p, int disc, hipStream_t s) {
    switch (disc) {
        case DISC_ZOH_S6: return launch_fwd_disc<IO, DISC_ZOH_S6>(p, s);
        case DISC_ZOH: return launch_fwd_disc<IO, DISC_ZOH>(p, s);
        case DISC_BILINEAR: return launch_fwd_disc<IO, DISC_BILINEAR>(p, s);
        case DISC_DIRAC: return launch_fwd_disc<IO, DISC_DIRAC>(p, s);
    }
    return hipErrorInvalidValue;
}

// float32 and bfloat16 are compiled side by side: selective_fwd_f32.hip includes this file for the former.
hipError_t launch_ss_fwd_f32(const FwdParams &p, int disc, hipStream_t s);
#ifdef LRNNX_FWD_F32
hipError_t launch_ss_fwd_f32(const FwdParams &p, int disc, hipStream_t s) { return launch_fwd_io<float>(p, disc, s); }
#else
hipError_t launch_ss_fwd(const FwdParams &p, int io_dtype, int disc, hipStream_t s) {
    return io_dtype == 1 ? launch_fwd_io<bf16_t>(p, disc, s) : launch_ss_fwd_f32(p, disc, s);
}

// the shape of a single pass over a batch, as a number (for tests of the choice)
int fwd_shape_number(int64_t maps, int64_t dpg, int64_t N, int64_t L, bool f32, bool outputs) { return (int)fwd_shape(maps, dpg, N, L, f32, outputs); }
int fwd_channels_per_workgroup() { return FwdGeom<16, 16>::CH; }
int fwd_tile_steps() { return FwdGeom<16, 16>::TILE; }

// Whether the chunk-carry path is faster than the best single pass, by 3 % at least since it takes scratch: it walks the sequence
// twice and launches three times, but on a full chip (costs fitted as above; the first two are those of the three launches).
// N = 16, bf16: 512 rows of 2048 steps 21.1 us against 21.7, 1024 rows of 2048 25.6 against 22.6; 16 rows of 65536 steps 21
// against 557.
bool fwd_chunks_pay(int64_t B, int64_t bcg, int64_t dpg, int64_t N, int64_t L, bool f32) {
    static constexpr FwdCost cost[2] = {{771, 41, 405, 30}, {865, 32, 188, 33}};
    const int64_t tiles = (L + fwd_tile_steps() - 1) / fwd_tile_steps();
    if (tiles < 2) return false;
    const int64_t channels = fwd_channels_per_workgroup();
    const int64_t chunked = fwd_cost(cost[f32 ? 0 : 1], N, 1, B * bcg * ((dpg + channels - 1) / channels) * tiles);
    constexpr int64_t launch = 220;
    for (const FwdShape shape : kFwdShapes) {
        const int64_t t = fwd_time(B * bcg, dpg, N, L, f32, shape);
        if (t != INT64_MAX && t + launch <= chunked + chunked * 3 / 100) return false;
    }
    return true;
}

// The same for the sweep that a backward call without checkpoints makes, of states alone, whose second pass saves nothing over the aggregates but the
// launches stay: costs of its own, of one chain a row (64 x 16) and of the three launches.  Sweeps on 256 workgroups of eight channels and less
// (with more, one chain was faster in every call measured).  870 sweeps of 16 to 3000 rows of 512 to 65536 steps, N = 1 to 32, both types: chunks
// are taken in one that is slower so (1.04 times); by the rule above in 30, up to 1.22 times (us, one chain and in chunks, bf16: 1024 rows of 4096
// steps, N = 32 50.6 and 61.6; 512 of 2048, N = 16 15.8 and 17.9).  700 drawn ones, all schemes, odd lengths, groups: in 5, up to 1.08 (20, 1.27).
bool sweep_chunks_pay(int64_t B, int64_t bcg, int64_t dpg, int64_t N, int64_t L, bool f32) {
    static constexpr FwdCost chain[2] = {{312, 0, 173, 38}, {302, 1, 122, 33}}, chunks[2] = {{785, 30, 238, 25}, {858, 24, 121, 28}};
    const int64_t tiles = (L + fwd_tile_steps() - 1) / fwd_tile_steps(), channels = fwd_channels_per_workgroup(), maps = B * bcg;
    if (tiles < 2 || maps * ((dpg + 7) / 8) > kNumCU) return false;
    const FwdCost &c = chain[f32 ? 0 : 1];
    const int64_t one = c.tile + c.state * N + (L + 1023) / 1024 * (c.wg + c.wg_state * N);
    const int64_t chunked = fwd_cost(chunks[f32 ? 0 : 1], N, 1, maps * ((dpg + channels - 1) / channels) * tiles);
    return chunked + chunked * 6 / 100 < one;
}

// Chains the chunk aggregates of one (b,d,n): carry-in of chunk c+1 = P_c * carry-in of chunk c + S_c.
// ws_S[c] is replaced by the carry-in of chunk c.  A workgroup takes 16 such chains and up to 256 chunks at a time: 16 threads
// of a chain fold up to 16 consecutive pairs each, all read at once, and replay them from the state that the threads before
// hand on through LDS.  One after the other the reads cost 0.2 us a chunk, half of the time of few long rows (16 rows of
// 65536 steps, N = 16, float32, 256 chunks: call 83 us, so 24).
constexpr int kCarryLen = 16;
__global__ __launch_bounds__(256) void k_ss_carry(const FwdParams p) {
    __shared__ float sP[kCarryLen][17], sS[kCarryLen][17];
    const int chain = threadIdx.x % 16, seg = threadIdx.x / 16;
    const int64_t total = (int64_t)p.B * p.D * p.N, id = blockIdx.x * (int64_t)16 + chain;
    const int64_t i = id < total ? id : total - 1;       // (past the end: the last one again, nothing is written)
    const int64_t first = i / p.N * p.nchunks * p.N + i % p.N;
    float x = p.x0 ? p.x0[i] : 0.0f;
    for (int c0 = 0; c0 < p.nchunks; c0 += 16 * kCarryLen) {
        const int left = p.nchunks - c0, most = left < 16 * kCarryLen ? left : 16 * kCarryLen;
        const int len = (most + 15) / 16, c1 = c0 + seg * len;
        float P[kCarryLen], S[kCarryLen], fP = 1.0f, fS = 0.0f;
#pragma unroll
        for (int k = 0; k < kCarryLen; ++k) {
            P[k] = 1.0f; S[k] = 0.0f;
            if (k < len) {
                const int c = c1 + k < p.nchunks ? c1 + k : p.nchunks - 1;
                P[k] = p.ws_P[first + (int64_t)c * p.N];
                S[k] = p.ws_S[first + (int64_t)c * p.N];
            }
        }
#pragma unroll
        for (int k = 0; k < kCarryLen; ++k) {
            const bool pair = k < len && c1 + k + 1 < p.nchunks;      // nothing follows the last chunk: its pair was not computed
            P[k] = pair ? P[k] : 1.0f; S[k] = pair ? S[k] : 0.0f;
            fS = __builtin_fmaf(P[k], fS, S[k]);
            fP *= P[k];
        }
        sP[seg][chain] = fP; sS[seg][chain] = fS;
        __syncthreads();
        float mine = x;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            if (s == seg) mine = x;
            x = __builtin_fmaf(sP[s][chain], x, sS[s][chain]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kCarryLen; ++k) {
            if (k < len && c1 + k < p.nchunks && id < total) p.ws_S[first + (int64_t)(c1 + k) * p.N] = mine;
            mine = __builtin_fmaf(P[k], mine, S[k]);
        }
    }
}

// Fills up to five buffers of 32-bit words, each with its own word, in one launch (a fill kernel rather than
// hipMemsetAsync, so that a caller may capture the library call in a HIP graph).
__global__ void k_fill(const FillList z) {
    fill_words(z, blockIdx.x * (int64_t)blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

hipError_t launch_ss_carry(const FwdParams &p, hipStream_t s) {
    const int64_t total = (int64_t)p.B * p.D * p.N;
    hipLaunchKernelGGL(k_ss_carry, dim3((unsigned)((total + 15) / 16)), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_fill(const FillList &z, hipStream_t s) {
    const int64_t most = fill_words_most(z);
    if (most <= 0) return hipSuccess;
    int64_t blocks = (most + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, s, z);
    return hipGetLastError();
}
#endif

}  // namespace lrnnx
