// Backward selective scan for gfx950: reverse-mode derivative of Eq. 2 of the paper (diagonal,
// input-dependent A(k), B(k), C(k)) with the fused discretisations of Sec. 3.  The state is never
// stored per step (Sec. 3): every time tile is recomputed from the checkpoint the forward wrote.
//
// For one (b,d) row and one state n, with H_l = dLoss/dx_l:
//     H_l      = Cm_{l,n} dypre_l + a_{l+1} H_{l+1}                 (same affine scan, time reversed)
//     dCm_{l,n} += dypre_l x_l          dBm_{l,n} += H_l g_l u_l
//     du_l     += H_l g_l Bm_{l,n}      da_l = H_l x_{l-1}          dg_l = H_l Bm_{l,n} u_l
//     dDelta_l += da_l da/dDelta + dg_l dg/dDelta                    dA_n += da_l da/dA + dg_l dg/dA
//
// Mapping.  A workgroup of W = N/4 wavefronts works on one tile of 256 steps at a time, last tile first, and on two
// channels at a time: the halves of a wavefront are the two channels, and lane i of a half owns T = 8 consecutive steps
// of the tile.  A wavefront holds four states, one after the other in the same registers, so a prefix over the tile is
// a scan of 32 lanes shared by 8 steps (with N = 16 two at a time, whose scans over 16 lanes are one: see bwd_pairs).  The
// workgroup loops over G channels; a lane keeps its columns of Bm and Cm (4 states x 8 steps) and the running sums of dBm and dCm over channels in registers, so the reduction over channels costs
// no traffic inside the loop.  What is summed over states (ypre for dz, du, dDelta) is added over the wavefront's
// states in registers and over wavefronts through LDS: after a barrier every thread finishes a few consecutive steps
// of one channel (epilogue) and prepares the same steps of the next pair of channels (prologue).
//
// What bounds it: vector-ALU issue and, with two wavefronts a SIMD, the waits of a wavefront that the other one does not
// fill (a seventh of its time, for LDS and at the one barrier of a pass).  With N = 16, 24.3 vector instructions per state update, or 26.1
// issue slots if an exponential counts as two: 17 instructions of arithmetic, 5.4 for folds' ends and scans, the rest prologue, epilogue
// and the work per tile.  B=8, D=1536, N=16, L=2048, bf16: 261 to 275 us, 3.9 to 4.1 cycles a slot, and 23 us for the sums of dBm and dCm;
// B=16, D=2560, L=4096 1600 to 1627.  What brought it there, in us on the former shape: time on 32 lanes of 8 steps instead of 64 of 4
// with all four states of a wavefront scanned together 440 -> 358; parts of a pass at the issue priorities of scan_common.hpp, prologue and
// epilogue at the highest, since a whole workgroup waits for the last at its barrier, 369 -> 338 (both parts at one priority
// 351); LDS accesses of prologue and epilogue without bank conflicts, the epilogue's reads under way together 325; two states at
// a time 318; nothing spilled 8 less.  Then, back to back: the steps' places in LDS by a shift, a mask and an exclusive or, one address for
// all planes of a pair, sums over rows by masked lanes, both buffers' passes written out 287 -> 278; the reads of the main part behind the
// epilogue's 272; the maps through LDS 269; no launch that clears dA, dD and dbias, see RowSums.  Where the main loop falls in memory
// is 1.5 % (1592 to 1650 us on the latter shape with the same instructions, padded by 0 to 12 words).
// Also tried: four channels per wavefront on rows of 16 lanes with 16 steps each (twice the LDS
// traffic and one workgroup per compute unit: 560 us), halves holding different states at three wavefronts per SIMD (a
// swap-and-add per sum: 431 us); the next tile's first steps and maps under way in the last pass of this one (274 and 275 us; with the
// registers for it spilled 315); the epilogue before the main part (292); the two workgroups of a compute unit set off apart (no gain).
#include "kernels.hpp"
#include "scan_common.hpp"
#include <type_traits>

namespace lrnnx {


// Both scans of one state over the 32 lanes of each half-wavefront: on return S is the inclusive prefix (lane 0 of the
// half first) and Q the inclusive suffix (lane 31 first) of the pairs (P, S) and (P, Q), xin the prefix of the lane
// before (lane 0 keeps what it came with) and Gin the suffix of the lane after (lane 31 keeps it).  The two scans
// alternate, so that a DPP read of a register comes at least two instructions after its last write.  The suffix of a
// half's upper row reaches the last lane of the lower row by a shift of the whole wavefront, and the row's other lanes
// from there.  Two blocks, each with its own wait states at its head: as one block the compiler can place nothing between
// them, and the backward pass of B=16, D=2560, L=4096 took 1 % longer (2707 us with recompute, 2679).
__device__ __forceinline__ void half_scans(float P, float &S, float &Q, float &xin, float &Gin) {
    float Pr = P;
    asm("s_nop 1\n\t"
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:1" LRNNX_ALLROWS, "row_shl:1" LRNNX_ALLROWS)
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:2" LRNNX_ALLROWS, "row_shl:2" LRNNX_ALLROWS)
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:4" LRNNX_ALLROWS, "row_shl:4" LRNNX_ALLROWS)
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:8" LRNNX_ALLROWS, "row_shl:8" LRNNX_ALLROWS)
        : "+v"(S), "+v"(P), "+v"(Q), "+v"(Pr));
    float Qn;                                        // lane 15 of rows 0 and 2: the first lane of the row after
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %5 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "v_mov_b32_dpp %4, %1 wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_mov_b32_dpp %2, %0 wave_shr:1 row_mask:0xa bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %6 row_newbcast:15 row_mask:0x5 bank_mask:0xf\n\t"
        "v_mov_b32_dpp %2, %0 row_shr:1 row_mask:0x5 bank_mask:0xf\n\t"
        "s_nop 0\n\t"
        "v_mov_b32_dpp %3, %1 wave_shl:1 row_mask:0x5 bank_mask:0xf\n\t"
        "v_mov_b32_dpp %3, %1 row_shl:1 row_mask:0xa bank_mask:0xf"
        : "+v"(S), "+v"(Q), "+v"(xin), "+v"(Gin), "=&v"(Qn) : "v"(P), "v"(Pr));
}

// Both scans over the 16 lanes of each row: S becomes the inclusive prefix (lane 0 first) and Q the inclusive suffix (lane
// 15 first) of the pairs (P, S) and (P, Q), x the prefix of the lane before (lane 0 keeps what it came with) and g the suffix
// of the lane after (lane 15 keeps it).
__device__ __forceinline__ void row_scans(float P, float &S, float &Q, float &x, float &g) {
    float Pr = P;
    asm("s_nop 1\n\t"
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:1" LRNNX_ALLROWS, "row_shl:1" LRNNX_ALLROWS)
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:2" LRNNX_ALLROWS, "row_shl:2" LRNNX_ALLROWS)
        LRNNX_FR_STATE(0, 1, 2, 3, "row_shr:4" LRNNX_ALLROWS, "row_shl:4" LRNNX_ALLROWS)
        "v_fmac_f32_dpp %0, %0, %1 row_shr:8" LRNNX_ALLROWS "\n\t"
        "v_fmac_f32_dpp %2, %2, %3 row_shl:8" LRNNX_ALLROWS "\n\t"
        "s_nop 0\n\t"
        "v_mov_b32_dpp %4, %0 row_shr:1" LRNNX_ALLROWS "\n\t"
        "v_mov_b32_dpp %5, %2 row_shl:1" LRNNX_ALLROWS
        : "+v"(S), "+v"(P), "+v"(Q), "+v"(Pr), "+v"(x), "+v"(g));
}

// Both scans of two states over the tile, after their lanes' folds (P, S, Q: multiplier, end state from zero and adjoint handed on
// from zero; one register for each state).  The rows of a half hold alternate pieces of eight steps, so a row swap gives row 0
// both pieces of the first state and row 1 both of the second, and one scan over 16 lanes serves the two.  xc is the state that
// enters the tile (lane 0 of the row of that state, zero elsewhere), hc the adjoint that enters it from the later side (lane 15).
// On return xin and Gin are what enters each lane's piece of each state; the result is the adjoint that leaves the tile on the
// earlier side (lane 0 of each row).
__device__ __forceinline__ float pair_scans(float P0, float P1, float S0, float S1, float Q0, float Q1, float xc, float hc,
                                            float &xin0, float &xin1, float &Gin0, float &Gin1) {
    swap_rows(P0, P1); swap_rows(S0, S1); swap_rows(Q0, Q1);             // now 0: the earlier piece, 1: the later one
    const float P = P0 * P1;
    float S = __builtin_fmaf(P1, S0, S1), Q = __builtin_fmaf(P0, Q1, Q0);
    S = __builtin_fmaf(P, xc, S);
    Q = __builtin_fmaf(P, hc, Q);
    row_scans(P, S, Q, xc, hc);
    xin0 = xc; xin1 = __builtin_fmaf(P0, xc, S0);
    Gin1 = hc; Gin0 = __builtin_fmaf(P1, hc, Q1);
    swap_rows(xin0, xin1); swap_rows(Gin0, Gin1);
    return Q;
}

// Sums over the 16 lanes of each row, several at a time: a step that folds halves of a row (or of its halves) writes half of the lanes of one
// register from one sum and the other half from another (bank_mask: groups of four lanes), so that no value has to be selected.
// Four sums: on return lane i of a row holds sum i / 4.
__device__ __forceinline__ float row_sums4(float a, float b, float c, float d) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3" : "+v"(a), "+v"(b));
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(a), "+v"(b) : "v"(c), "v"(d));
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %0, %1, %1 row_ror:4 row_mask:0xf bank_mask:0xa" : "+v"(a) : "v"(b));
    a += dpp<0xB1>(0.0f, a);                         // quad_perm [1,0,3,2]
    return a + dpp<0x4E>(0.0f, a);                   // quad_perm [2,3,0,1]
}
// Two sums: lanes 0 to 7 of a row hold the first, 8 to 15 the second.
__device__ __forceinline__ float row_sums2(float a, float b) {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(a) : "v"(b));
    a += dpp<0x141>(0.0f, a);                        // row_half_mirror
    a += dpp<0xB1>(0.0f, a);                         // quad_perm [1,0,3,2]
    return a + dpp<0x4E>(0.0f, a);                   // quad_perm [2,3,0,1]
}

// the eight steps of the tile that lane li of a half holds; PAIR: its two rows of 16 lanes hold alternate pieces
template <bool PAIR> __device__ __forceinline__ int piece_of(int li) { return PAIR ? ((li & 15) << 1) | (li >> 4 & 1) : li; }

// CNT consecutive steps of a tile of 256 in LDS.  Step f of a whole tile sits at float f with its bits 2 and 3 turned by bits 5 and 6: a
// lane's 8 steps are two 16-byte accesses (the second at the first's place ^ 4), those of 8 lanes, which go out together, fall into 32 different
// banks whether the lanes hold consecutive pieces of the tile or alternate ones, and so do the few steps of consecutive threads of the prologue
// and epilogue, whose place is a shift, a mask and an exclusive or of the thread's number.  f is a multiple of CNT.
// A short tile (T = 4 or 2 steps a lane) takes the first 128 or 64 floats, [lane][step % T].
template <bool PAIR, int T> __device__ __forceinline__ int lane_slot(int li) {
    if constexpr (T == 8) { const int p = piece_of<PAIR>(li); return p << 3 ^ (p & 12); }
    else return T == 2 ? li << 1 : (li << 2) ^ (PAIR ? (li & 16) >> 1 : 0);
}
template <bool PAIR, int T> __device__ __forceinline__ int step_slot(int f) {
    if constexpr (T == 8) return f ^ (f >> 3 & 12);
    const int g = f / T, li = PAIR ? (g >> 1) | ((g & 1) << 4) : g;
    return lane_slot<PAIR, T>(li) + f % T;
}
template <int CNT>
__device__ __forceinline__ void lds_steps_read(const float *plane, int slot, float *out) {
    const float *p = plane + slot;
    if constexpr (CNT == 1) out[0] = p[0];
    else if constexpr (CNT == 2) { const float2 v = *reinterpret_cast<const float2 *>(p); out[0] = v.x; out[1] = v.y; }
    else {
#pragma unroll
        for (int q = 0; q < CNT / 4; ++q) {
            const float4 v = *reinterpret_cast<const float4 *>(plane + (q ? slot ^ 4 : slot));
            out[4 * q] = v.x; out[4 * q + 1] = v.y; out[4 * q + 2] = v.z; out[4 * q + 3] = v.w;
        }
    }
}
template <int CNT>
__device__ __forceinline__ void lds_steps_write(float *plane, int slot, const float *v) {
    float *p = plane + slot;
    if constexpr (CNT == 1) p[0] = v[0];
    else if constexpr (CNT == 2) *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    else {
#pragma unroll
        for (int q = 0; q < CNT / 4; ++q)
            *reinterpret_cast<float4 *>(plane + (q ? slot ^ 4 : slot)) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
}

// CNT consecutive elements of a row, wholly inside it: wave-uniform base plus a lane's 32-bit offset
template <typename IO, int CNT>
__device__ __forceinline__ void load_at(const IO *row, unsigned f, RawFew<IO, CNT> &r) {
    load_few_raw<IO, CNT>(reinterpret_cast<const IO *>(reinterpret_cast<const char *>(row) + f * (unsigned)sizeof(IO)), 0, CNT, true, r);
}
template <typename IO, int CNT>
__device__ __forceinline__ void store_at(IO *row, unsigned f, const float *v) {
    store_few<IO, CNT>(reinterpret_cast<IO *>(reinterpret_cast<char *>(row) + f * (unsigned)sizeof(IO)), 0, CNT, true, v);
}

template <int CNT>
__device__ __forceinline__ void lds_few(const float *p, float *out) {       // CNT = 1, 2 or 4, p aligned to as many floats
    if constexpr (CNT == 4) { const float4 v = *reinterpret_cast<const float4 *>(p); out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w; }
    else if constexpr (CNT == 2) { const float2 v = *reinterpret_cast<const float2 *>(p); out[0] = v.x; out[1] = v.y; }
    else out[0] = p[0];
}

// Geometry of a workgroup for N states.
template <int N> struct BwdGeom {
    static constexpr int W = N == 4 ? 2 : (N >= 4 ? N / 4 : 1);      // wavefronts
    static constexpr int NS = N / W;                 // states of a wavefront, one after the other
    static constexpr int NT = W * 64;
    static constexpr int CP = 2;                     // channels per pass
    static constexpr int TPT = CP * kBwdTileSteps / NT;       // steps of a thread in prologue and epilogue
    static constexpr int NTC = kBwdTileSteps / TPT;           // threads that share a channel there
    // one wavefront: a lane's steps of the main part are its own of the prologue and epilogue, nothing goes through LDS;
    // two: two barriers per pass, single buffers (the LDS of a compute unit then holds eight wavefronts); more: one
    // barrier per pass, double buffers
    static constexpr bool OWN = W == 1;
    static constexpr int NB = W >= 4 ? 2 : 1;        // buffers
};

// Whether a wavefront takes two states at a time, one scan over 16 lanes for both (pair_scans): 5.4 vector instructions a
// state update for folds' ends and scans instead of 6.9, but both states' multipliers and inputs are held at once.  It pays for
// many states, whose tiles are long in work: N = 16, B=16, D=2560, L=4096, bf16 1805 -> 1721 us, L=2048 of D=1536 325 -> 315,
// N = 32 0.98 to 1.02; N = 8 5 to 20 % slower; the exact zero-order hold (gains beside the multipliers) 17 to 43 %, bilinear 2 % (all of it
// while the row addresses of the maps were spilled beside).
template <int N, int DISC> constexpr bool bwd_pairs() { return N == 16 && (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC); }

// channels per workgroup for a sequence of ntiles tiles: fewer than G in a packed batch with a work cap
__device__ __forceinline__ int channels_of(const BwdParams &p, int64_t ntiles) {
    if (p.wcap <= 0) return p.G;
    const int64_t fit = p.wcap / (ntiles > 0 ? ntiles : 1);
    return fit < p.gmin ? p.gmin : (fit < p.G ? (int)fit & ~1 : p.G);      // (channels are walked in pairs)
}

// Two wavefronts a SIMD, also where the registers would let in a third (few states without a gate): single-wavefront workgroups then crowd
// some SIMDs and leave others to one (N = 4, bf16, 140 rows of 42166 steps 58 and 66 us with up to three; with the forward pass,
// 6144 rows of 2048 steps 111 and 117, N = 1 67 and 70).
template <typename IO, int N, int DISC, bool HAS_Z, bool PART>
__global__ __launch_bounds__(BwdGeom<N>::NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_ss_bwd(const BwdParams p) {
    using GE = BwdGeom<N>;
    constexpr int W = GE::W, NS = GE::NS, NT = GE::NT, CP = GE::CP;
    constexpr int TILE = kBwdTileSteps;
    static_assert(TILE == kCkptInterval && TILE == 32 * 8, "a tile is one checkpoint interval and one half-wavefront");

    constexpr bool OWN = GE::OWN;
    constexpr int NB = GE::NB;
    constexpr bool PAIR = bwd_pairs<N, DISC>();
    static_assert(!PAIR || (!OWN && NS % 2 == 0), "whole pairs of states, steps through LDS");
    // What the wavefronts exchange of a pair of channels, a block for each buffer, so that one address reaches all of it: planes of CP x
    // TILE steps (delta, u, dypre; then ypre, du, ddelta partials of each wavefront), then A and the state entering the tile [2][CP][N].
    constexpr int PL = OWN ? 0 : CP * TILE, AC = (3 + 3 * W) * PL, BUF = AC + 2 * CP * N;
    __shared__ __attribute__((aligned(16))) float sPair[NB * BUF];
    __shared__ __attribute__((aligned(16))) float sH[kBwdMaxG * N];   // a_{l0} H_{l0} carried to the earlier tile, per (channel, n)
    __shared__ float sdA[kBwdMaxG * N];
    __shared__ float sdDb[2][kBwdMaxG];
    __shared__ float sDskip[kBwdMaxG], sBias[kBwdMaxG + CP];

    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane & 31, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = w * NS;                           // this wavefront's first state
    int b = blockIdx.y;
    int64_t L = p.L, toff = 0, bs = b;
    if (p.cu) {
        const SeqSpan q = seq_span(p.cu, p.B, p.L, b, p.ranked, p.order);           // the longest sequences start first
        b = q.b; toff = q.toff; L = q.L; bs = 0;
    }
    const int64_t slot0 = p.cu ? toff / TILE + b : (int64_t)b * p.part_tiles;    // first tile of this entry among all tiles
    // Chunked launch: this workgroup walks chunk blockIdx.z of its rows only, i.e. the steps toff .. toff + L - 1 of
    // the time axis, starting from that chunk's carried adjoint.  Chunks are counted from the start of the sequence;
    // the last one takes whatever is left (see chunk_span in selective_bwd_carry.hip), and the workgroups of a packed
    // sequence that ends before their chunk leave here, all threads together and before any barrier (chunk 0 stays
    // even for an empty sequence: it writes that sequence's dx0).
    const int chunk = blockIdx.z;
    const int64_t ntiles_seq = (L + TILE - 1) / TILE;
    int64_t tile_first = 0;                          // first tile of the chunk within its sequence
    if (p.nchunks > 1) {
        tile_first = chunk * p.tiles_per_chunk;
        const int64_t span = p.tiles_per_chunk * TILE;
        const int64_t left = L - chunk * span;
        if (chunk > 0 && left <= 0) return;
        toff += chunk * span;
        L = (chunk == p.nchunks - 1 || left < span) ? left : span;
    }
    const int64_t ntiles = (L + TILE - 1) / TILE;
    // a workgroup takes up to G consecutive channels of ONE Bm/Cm group; in a packed batch with a work cap fewer when
    // its sequence is long, and the workgroups of the launch that its sequence then does not need leave here, all
    // threads together and before any barrier
    const int G = channels_of(p, ntiles_seq);
    const int blocks_per_grp = (p.dpg + G - 1) / G;
    if ((int)blockIdx.x >= p.bcg * blocks_per_grp) return;
    const int grp = blockIdx.x / blocks_per_grp;
    const int din0 = (blockIdx.x % blocks_per_grp) * G;
    const int d0 = grp * p.dpg + din0;
    const int Gact = (p.dpg - din0 < G) ? p.dpg - din0 : G;
    // checkpoints of this workgroup's rows: [B,D,nck,N], or packed [D,nslots,N] with sequence b at slot toff/interval + b
    const int64_t nck = p.cu ? p.nslots : (p.L + kCkptInterval - 1) / kCkptInterval;
    const int64_t ck0 = p.cu ? toff / kCkptInterval + b : toff / kCkptInterval;
    const float *ckrow = p.ckpt + (((p.cu ? (int64_t)d0 : (int64_t)b * p.D + d0) * nck) + ck0) * N;
    const bool vec = p.vec != 0;

    // (an odd last channel has a partner in its pass, whose steps are empty and whose results go nowhere: its places in the tables exist,
    // G being even, and hold zeros)
    const int Gpair = (Gact + 1) & ~1;
    for (int i = tid; i < Gpair * N; i += NT) {
        float h = 0.0f;
        if (p.nchunks > 1 && i < Gact * N) h = p.hc[(((int64_t)b * p.D + d0 + i / N) * p.nchunks + chunk) * N + i % N];
        sH[i] = h; sdA[i] = 0.0f;
    }
    for (int i = tid; i < Gpair; i += NT) {
        sdDb[0][i] = 0.0f; sdDb[1][i] = 0.0f;
        sDskip[i] = p.Dskip && i < Gact ? p.Dskip[d0 + i] : 0.0f;
        sBias[i] = p.bias && i < Gact ? p.bias[d0 + i] : 0.0f;
    }

    const int64_t bc0 = ((p.cu ? (int64_t)grp : (int64_t)b * p.bcg + grp) * p.L + toff) * N;   // first element of the maps of this sequence
    const IO *Bm = reinterpret_cast<const IO *>(p.Bm) + bc0;
    const IO *Cm = reinterpret_cast<const IO *>(p.Cm) + bc0;

    // The addresses that follow from the thread's number are formed where they are needed: hoisted out of the loops by the
    // compiler they would sit in registers all through the main pass, which has none to spare: it spilled them, and a reload waits
    // for every access before it, at the head of a tile for the atomics of the one before (6 packed sequences of 32768 steps, 1536
    // channels, N = 16, bf16: 1240 us, now 1042; 24 of 16384: 450 and 430).
    auto fresh = [](unsigned v) { asm volatile("" : "+v"(v)); return v; };
    constexpr int LAST = PAIR ? 15 : 31;             // of the lanes that are scanned together
    const unsigned first_lane = (li & LAST) == 0 ? ~0u : 0u, last_lane = (li & LAST) == LAST ? ~0u : 0u;

    // One tile.  FULL: all of its steps are valid and every row takes vector accesses, nothing to check per element (a
    // taken branch costs a wavefront about a hundred cycles).  A sequence's last tile, if it has at most 128 or 64 steps, takes
    // T = 4 or 2 of them a lane instead of 8: half or a quarter of the work per step and state; the scans, the barriers and the
    // maps' loads stay.  Training steps of packed batches, with the forward pass's short tiles: 87 sequences of 67 steps, 538 channels, N = 8, float32
    // 162 -> 122 us, 74 of 119, 204 channels, N = 16, bf16 132 -> 111; whole tiles and longer tails as before.
    auto do_tile = [&](int64_t tile, auto full, auto per_lane) {
        constexpr bool FULL = decltype(full)::value;
        // The launch's parameters, read again here: what the tiles need of them would otherwise be held in scalar registers, or for lack of
        // those in lanes of vector registers, all through the kernel, once for each kind of tile (125 scalars spilled, so 54).
        typedef const __attribute__((address_space(4))) BwdParams KernArgs;          // (the kernel's only argument)
        KernArgs *args = (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        KernArgs &q = *args;
        constexpr int T = decltype(per_lane)::value;
        // prologue and epilogue: steps of a thread, threads that share a channel there, and this thread's channel of a pair (with short
        // tiles some wavefronts may have none)
        constexpr int TPT = GE::TPT * T / 8 > 0 ? GE::TPT * T / 8 : 1, NTC = 32 * T / TPT;
        constexpr bool ALL = CP * NTC == NT;
        static_assert(T == 8 || NTC >= 64, "a wavefront's steps are those of one channel");
        int c_own = tid / NTC;
        if constexpr (NTC >= 64) c_own = __builtin_amdgcn_readfirstlane(c_own);
        const bool busy = ALL || c_own < CP;
        if constexpr (!ALL) c_own = busy ? c_own : CP - 1;
        const int64_t l0 = tile * TILE;
        const int rem = FULL ? TILE : ((L - l0 < TILE) ? (int)(L - l0) : TILE);      // valid steps of this tile (at least one)

        // ---- the rows of Bm and Cm: all without a branch (past the end of the tile the last valid row is read again and then discarded), so that all
        // loads of a lane are in flight together.  From four wavefronts on they are read as they lie, 16 bytes a lane, and each lane takes its
        // columns from LDS, where the rows of eight steps have a gap of 16 bytes against bank conflicts.  Loaded by column each access met 32
        // cache lines, and those of eight wavefronts held up what came behind them (B=8, D=1536, N=16, L=2048, bf16: 274 -> 269.5 us).
        constexpr bool STAGED = NB == 2;
        constexpr int RB = N * (int)sizeof(IO), ROWS = 32 * T, CHUNKS = STAGED ? RB / 16 : 1, CPT = STAGED ? (ROWS * CHUNKS + NT - 1) / NT : 1;       // bytes of a row, its chunks, chunks of a thread
        RawFew<IO, STAGED ? 16 / (int)sizeof(IO) : NS> rB[STAGED ? CPT : T], rC[STAGED ? CPT : T];
        {
            const IO *BmT = Bm + l0 * N, *CmT = Cm + l0 * N;
            const unsigned t0 = fresh(tid);
            if constexpr (STAGED) {
#pragma unroll
                for (int k = 0; k < CPT; ++k) {
                    const unsigned i = t0 + k * NT;
                    int row = i / CHUNKS;
                    if (!FULL || ROWS * CHUNKS % NT) row = row < rem ? row : rem - 1;
                    const unsigned at = row * N + i % CHUNKS * (16 / (int)sizeof(IO));
                    load_at<IO, 16 / (int)sizeof(IO)>(BmT, at, rB[k]);
                    load_at<IO, 16 / (int)sizeof(IO)>(CmT, at, rC[k]);
                }
            } else {
                const int first = piece_of<PAIR>((int)(t0 & 31)) * T;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int step = first + t;
                    const int row = step < rem ? step : rem - 1;
                    load_few_raw<IO, NS>(BmT + (unsigned)(row * N + n0), 0, NS, true, rB[t]);
                    load_few_raw<IO, NS>(CmT + (unsigned)(row * N + n0), 0, NS, true, rC[t]);
                }
            }
        }
        // (in the places of partial sums, of the first buffer and of the second; the first pair's inputs lie before those)
        char *mB = reinterpret_cast<char *>(sPair + 3 * PL), *mC = reinterpret_cast<char *>(sPair + (3 * PL + (NB - 1) * BUF));
        auto row_at = [](unsigned row) { return row * RB + row / 8 * 16; };
        static_assert(!STAGED || 256 * RB + 32 * 16 <= 3 * W * PL * (int)sizeof(float), "a map in the partial sums' place");
        auto stage_maps = [&]() {
            const unsigned t0 = fresh(tid);
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                const unsigned i = t0 + k * NT, at = row_at(i / CHUNKS) + i % CHUNKS * 16;
                if (ROWS * CHUNKS % NT && i >= ROWS * CHUNKS) break;
                *reinterpret_cast<uint4 *>(mB + at) = make_uint4(rB[k].w[0], rB[k].w[1], rB[k].w[2], rB[k].w[3]);
                *reinterpret_cast<uint4 *>(mC + at) = make_uint4(rC[k].w[0], rC[k].w[1], rC[k].w[2], rC[k].w[3]);
            }
        };

        // ---- per-step inputs of a pair of channels are fetched one pair ahead.  Row pointers: this thread's channel of
        // the pair the next fetch reads and the next epilogue writes (past the last channel they stay on a valid one).
        RawFew<IO, TPT> r_u, r_dl, r_dy, r_z;
        const int64_t tl = toff + l0;
        const int c_first = c_own < Gact ? c_own : Gact - 1;
        const int64_t dch = d0 + c_first;
        const IO *n_u = reinterpret_cast<const IO *>(q.u) + bs * q.u_sb + dch * q.u_sd + tl;
        const IO *n_dl = reinterpret_cast<const IO *>(q.delta) + bs * q.dl_sb + dch * q.dl_sd + tl;
        const IO *n_dy = reinterpret_cast<const IO *>(q.dy) + bs * q.dy_sb + dch * q.dy_sd + tl;
        const IO *n_z = HAS_Z ? reinterpret_cast<const IO *>(q.z) + bs * q.z_sb + dch * q.z_sd + tl : n_dy;
        const int64_t z_sd = HAS_Z ? q.z_sd : q.dy_sd;
        IO *o_du = reinterpret_cast<IO *>(q.du) + bs * q.du_sb + dch * q.du_sd + tl;
        IO *o_dd = reinterpret_cast<IO *>(q.ddelta) + bs * q.dd_sb + dch * q.dd_sd + tl;
        const bool want_dz = HAS_Z && q.dz;
        IO *o_dz = reinterpret_cast<IO *>(q.dz) + bs * q.dz_sb + dch * q.dz_sd + tl;
        int n_g = 0;                                                 // first channel of the pair of the next fetch
        // A and the checkpointed state of the pair, [CP][N] each: the first wavefront fetches the former, the second the latter (lanes past
        // their number again what the others do); a workgroup of one wavefront has a thread for each value
        const bool has_ac = OWN ? tid < 2 * CP * N : w < 2, is_ck = OWN ? tid >= CP * N : w != 0;
        const float *n_ac = is_ck ? ckrow + tile * N : q.A + (int64_t)d0 * N;
        const unsigned ac_sd = is_ck ? (unsigned)(nck * N) : N;      // floats between two channels
        float r_ac = 0.0f;
        auto put_ac = [&](unsigned t0, int buf) {
            if (has_ac) (sPair + buf + AC + (OWN ? 0 : w * CP * N))[OWN ? t0 : t0 & (CP * N - 1)] = r_ac;
        };
        const bool window = TPT > 1 && vec && L >= TPT;              // the last steps of the sequence: see tail_window
        auto fetch = [&](unsigned t0) {
            const unsigned f0 = (t0 % NTC) * TPT;
            if (!busy) {
            } else if (FULL) {
                load_at<IO, TPT>(n_u, f0, r_u);
                load_at<IO, TPT>(n_dl, f0, r_dl);
                load_at<IO, TPT>(n_dy, f0, r_dy);
                if constexpr (HAS_Z) load_at<IO, TPT>(n_z, f0, r_z);
            } else if (window) {
                const int o = tail_window<TPT>((int)f0, rem);
                load_few_raw<IO, TPT>(n_u + o, 0, TPT, true, r_u);
                load_few_raw<IO, TPT>(n_dl + o, 0, TPT, true, r_dl);
                load_few_raw<IO, TPT>(n_dy + o, 0, TPT, true, r_dy);
                if constexpr (HAS_Z) load_few_raw<IO, TPT>(n_z + o, 0, TPT, true, r_z);
            } else {
                load_few_raw<IO, TPT>(n_u, (int)f0, rem, vec, r_u);
                load_few_raw<IO, TPT>(n_dl, (int)f0, rem, vec, r_dl);
                load_few_raw<IO, TPT>(n_dy, (int)f0, rem, vec, r_dy);
                if constexpr (HAS_Z) load_few_raw<IO, TPT>(n_z, (int)f0, rem, vec, r_z);
            }
            if (has_ac) {
                const unsigned second = n_g + 1 < Gact ? ac_sd : 0u;     // (no second channel: the first again)
                const unsigned at = (t0 % N + (0u - (t0 / N % CP) & second)) * 4u;
                r_ac = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(n_ac) + at);
            }
            n_g += CP;
            if (n_g < Gact) n_ac += (int64_t)CP * ac_sd;
            if (n_g + c_own < Gact) { n_u += CP * q.u_sd; n_dl += CP * q.dl_sd; n_dy += CP * q.dy_sd; n_z += CP * z_sd; }
        };
        fetch(fresh(tid));

        // ---- Bm, Cm columns and the sums of dBm, dCm over channels stay in registers
        float Bv[NS][T], Cv[NS][T], dB[NS][T], dC[NS][T];
        auto take_maps = [&]() {
            const int first = piece_of<PAIR>((int)(fresh(tid) & 31)) * T;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                float tb[NS], tc[NS];
                if constexpr (STAGED) {
                    const unsigned at = row_at(first + t) + n0 * (unsigned)sizeof(IO);
                    load_row<IO, NS>(reinterpret_cast<const IO *>(mB + at), tb);
                    load_row<IO, NS>(reinterpret_cast<const IO *>(mC + at), tc);
                } else {
                    unpack_few<IO, NS>(rB[t], tb);
                    unpack_few<IO, NS>(rC[t], tc);
                }
                const bool ok = FULL || first + t < rem;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    Bv[s][t] = ok ? tb[s] : 0.0f; Cv[s][t] = ok ? tc[s] : 0.0f;
                    dB[s][t] = 0.0f; dC[s][t] = 0.0f;
                }
            }
        };
        if constexpr (!STAGED) take_maps();

        // kept in registers from a pair's prologue to its epilogue: d softplus / ds and the factor that turns ypre into dz
        struct Kept { float sg[TPT], zf[TPT]; } even, odd;
        // ---- prologue of the pair whose inputs have been fetched: each thread prepares TPT steps of its channel
        auto step_inputs = [&](int ch, float bias, unsigned t0, Kept &k, float (&u)[TPT], float (&dl)[TPT], float (&dy)[TPT]) {
            float z[TPT];
            if (!FULL && window) {
                const int f0 = (int)((t0 % NTC) * TPT), by = f0 - tail_window<TPT>(f0, rem);
                tail_shift<IO, TPT>(r_u, by);
                tail_shift<IO, TPT>(r_dl, by);
                tail_shift<IO, TPT>(r_dy, by);
                if constexpr (HAS_Z) tail_shift<IO, TPT>(r_z, by);
            }
            unpack_few<IO, TPT>(r_u, u);
            unpack_few<IO, TPT>(r_dl, dl);
            unpack_few<IO, TPT>(r_dy, dy);
            if constexpr (HAS_Z) unpack_few<IO, TPT>(r_z, z);
#pragma unroll
            for (int i = 0; i < TPT; ++i) {
                const float v = dl[i] + bias;
                float sp, sg;
                softplus_sigmoid<sizeof(IO) == 4>(v, sp, sg);
                dl[i] = q.softplus ? sp : v;
                k.sg[i] = q.softplus ? sg : 1.0f;
                if constexpr (HAS_Z) gate_bwd(z[i], dy[i], k.zf[i]);
            }
            if (__builtin_expect(!FULL || ch >= Gact, !FULL)) {      // steps past the end: Delta = 0 (a = 1), no input, no gradient
                const int f0 = (t0 % NTC) * TPT;
#pragma unroll
                for (int i = 0; i < TPT; ++i)
                    if (f0 + i >= rem || ch >= Gact) { dl[i] = 0.0f; u[i] = 0.0f; dy[i] = 0.0f; }
                asm volatile("");                        // (a branch that is hardly ever taken, not six selects in every pass)
            }
        };
        // where this thread's steps of its channel are in a plane
        auto thread_slot = [&](unsigned t0) {
            // (a whole tile: the thread's number holds the channel above the step)
            if constexpr (T == 8 && ALL) return step_slot<PAIR, T>((int)(t0 * TPT));
            else return step_slot<PAIR, T>((int)((t0 % NTC) * TPT)) + c_own * TILE;
        };
        auto prologue = [&](int ch, float bias, unsigned t0, Kept &k, int buf) {
            if (busy) {
                float u[TPT], dl[TPT], dy[TPT];
                step_inputs(ch, bias, t0, k, u, dl, dy);
                float *in = sPair + buf + (unsigned)thread_slot(t0);
                lds_steps_write<TPT>(in, 0, dl);
                lds_steps_write<TPT>(in + PL, 0, u);
                lds_steps_write<TPT>(in + 2 * PL, 0, dy);
            }
            put_ac(t0, buf);
        };
        // ---- epilogue: du, ddelta, dz of this thread's steps from the sums over states
        auto finish = [&](const int g, const Kept &k, unsigned t0, unsigned f0, const float (&e_dl)[TPT], const float (&e_u)[TPT], const float (&e_dy)[TPT],
                          const float (&s_yp)[TPT], const float (&s_du)[TPT], const float (&s_dd)[TPT], const float Dsk) {
            const int ch = g + c_own;
            const bool live = ch < Gact;
            float o_u[TPT], o_d[TPT], o_z[TPT];
            float dD_part, db_part;
#pragma unroll
            for (int i = 0; i < TPT; ++i) {
                const float ed = e_dl[i], eu = e_u[i], ey = e_dy[i];
                float su = s_du[i], sd = s_dd[i];
                if constexpr (DISC == DISC_ZOH_S6) {
                    // the wavefronts' sums are sum_n H B: dDelta += u sum_n H B, du = Delta sum_n H B
                    sd = __builtin_fmaf(eu, su, sd);
                    su *= ed;
                }
                o_u[i] = __builtin_fmaf(ey, Dsk, su);
                o_d[i] = sd * k.sg[i];
                if constexpr (HAS_Z) o_z[i] = __builtin_fmaf(Dsk, eu, s_yp[i]) * k.zf[i];
                const float db = (FULL || (int)f0 + i < rem) ? o_d[i] : 0.0f;
                dD_part = i ? __builtin_fmaf(ey, eu, dD_part) : ey * eu;
                db_part = i ? db_part + db : db;
            }
            if (live) {
                if (FULL) {
                    store_at<IO, TPT>(o_du, f0, o_u);
                    store_at<IO, TPT>(o_dd, f0, o_d);
                    if constexpr (HAS_Z) { if (want_dz) store_at<IO, TPT>(o_dz, f0, o_z); }
                } else {
                    store_few<IO, TPT>(o_du, (int)f0, rem, vec, o_u);
                    store_few<IO, TPT>(o_dd, (int)f0, rem, vec, o_d);
                    if constexpr (HAS_Z) { if (want_dz) store_few<IO, TPT>(o_dz, (int)f0, rem, vec, o_z); }
                }
            }
            const float sum = row_sums2(dD_part, db_part);
            if (__builtin_amdgcn_inverse_ballot_w64(0x0101010101010101)) lds_add(&sdDb[0][0] + ch + (t0 & 8) * (kBwdMaxG / 8), sum);
            o_du += CP * q.du_sd; o_dd += CP * q.dd_sd;
            if constexpr (HAS_Z) o_dz += CP * q.dz_sd;
        };
        auto epilogue = [&](const int g, const Kept &k, const int buf, auto read_next) {
            if (!busy) return;
            const unsigned t0 = fresh(tid), f0 = (t0 % NTC) * TPT;
            const float *at = sPair + buf + (unsigned)thread_slot(t0);
            float e_in[3][TPT], s_yp[TPT], s_du[TPT], s_dd[TPT], v[W][3][TPT];
#pragma unroll
            for (int ww = 0; ww < W; ++ww)
#pragma unroll
                for (int j = HAS_Z ? 0 : 1; j < 3; ++j) lds_steps_read<TPT>(at + (3 + 3 * ww + j) * PL, 0, v[ww][j]);
#pragma unroll
            for (int j = 0; j < 3; ++j) lds_steps_read<TPT>(at + j * PL, 0, e_in[j]);
            const float Dsk = sDskip[g + c_own];
            read_next();
            // all reads before the first use: left to itself the compiler waits for each wavefront's sums before it reads the next
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < TPT; ++i) {
                s_yp[i] = HAS_Z ? v[0][0][i] : 0.0f; s_du[i] = v[0][1][i]; s_dd[i] = v[0][2][i];
#pragma unroll
                for (int ww = 1; ww < W; ++ww) {
                    if constexpr (HAS_Z) s_yp[i] += v[ww][0][i];
                    s_du[i] += v[ww][1][i]; s_dd[i] += v[ww][2][i];
                }
            }
            finish(g, k, t0, f0, e_in[0], e_in[1], e_in[2], s_yp, s_du, s_dd, Dsk);
        };
        // ---- main: this lane's 8 steps of its channel, one state after the other
        auto states = [&](const int g, const int buf, const unsigned ln, float (&dl)[T], float (&du)[T], const float (&dy)[T],
                          float (&yp)[T], float (&pu)[T], float (&pd)[T]) {
                // this lane's channel in the tables of A and the state entering the tile, and in those of the adjoint and dA
                const unsigned cN = (ln & 32) * N >> 5;
                const float *ac = sPair + buf + AC + n0 + cN;
                float *at = sH + g * N + n0 + cN;
                float Ak[NS], ck[PAIR ? 1 : NS], hc[PAIR ? 1 : NS];
                lds_few<NS>(ac, Ak);
                if constexpr (!PAIR) {
                    lds_few<NS>(ac + CP * N, ck);
                    lds_few<NS>(at, hc);
                }
                if constexpr (DISC == DISC_ZOH_S6) {
#pragma unroll
                    for (int t = 0; t < T; ++t) du[t] *= dl[t];      // S6 only ever needs Delta*u; the others keep u
                }
                float sum_dl = dl[0];
#pragma unroll
                for (int t = 1; t < T; ++t) sum_dl += dl[t];
                float dA[NS];
                if constexpr (PAIR) {
                    const unsigned row = ln >> 4 & 1;                // of the half, and the state of a pair that it scans
#pragma unroll
                    for (int s = 0; s < NS; s += 2) {
                        float a[2][T], x[2][T], P[2], S[2], Q[2], xin[2], Gin[2];
                        slow_part();
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            // the lane's folds, as below but from zero: what enters the tile joins the scan
                            const ACoef co = make_acoef<DISC>(Ak[s + j]);
#pragma unroll
                            for (int t = 0; t < T; ++t) {
                                float g;
                                disc_ag<DISC>(dl[t], co, a[j][t], g);
                                x[j][t] = du[t] * Bv[s + j][t];
                            }
                            S[j] = x[j][0]; Q[j] = a[j][T - 1] * (Cv[s + j][T - 1] * dy[T - 1]);
#pragma unroll
                            for (int t = 1; t < T; ++t) S[j] = __builtin_fmaf(a[j][t], S[j], x[j][t]);
#pragma unroll
                            for (int t = T - 2; t >= 0; --t) Q[j] = a[j][t] * __builtin_fmaf(Cv[s + j][t], dy[t], Q[j]);
                            P[j] = exp2_fast(sum_dl * co.A2);
                        }
                        const float xc = i2f(f2i((ac + row)[CP * N + s]) & (int)first_lane);
                        const float hc2 = i2f(f2i((at + row)[s]) & (int)last_lane);
                        const float out = pair_scans(P[0], P[1], S[0], S[1], Q[0], Q[1], xc, hc2, xin[0], xin[1], Gin[0], Gin[1]);
                        if (first_lane) (at + row)[s] = out;             // carried to the earlier tile
                        fast_part();
                        // replay of both states side by side (earliest step first), then of both adjoints (last step first): two
                        // chains whose instructions fill each other's result latencies
                        float xp[2] = {xin[0], xin[1]}, dAp[2] = {0.0f, 0.0f};
#pragma unroll
                        for (int t = 0; t < T; ++t)
#pragma unroll
                            for (int j = 0; j < 2; ++j) { xp[j] = __builtin_fmaf(a[j][t], xp[j], x[j][t]); x[j][t] = xp[j]; }
#pragma unroll
                        for (int t = T - 1; t >= 0; --t)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                auto acc = [&](float &sum, float m1, float m2) { sum = (s + j == 0) ? m1 * m2 : __builtin_fmaf(m1, m2, sum); };
                                const float H = __builtin_fmaf(Cv[s + j][t], dy[t], Gin[j]);
                                Gin[j] = a[j][t] * H;
                                dC[s + j][t] = __builtin_fmaf(dy[t], x[j][t], dC[s + j][t]);
                                if constexpr (HAS_Z) acc(yp[t], Cv[s + j][t], x[j][t]);
                                acc(pu[t], H, Bv[s + j][t]);         // (S6 and dirac: see below)
                                dB[s + j][t] = __builtin_fmaf(H, du[t], dB[s + j][t]);
                                const float q = Gin[j] * (t > 0 ? x[j][t - 1] : xin[j]);
                                acc(pd[t], q, Ak[s + j]);
                                dAp[j] = __builtin_fmaf(q, dl[t], dAp[j]);
                                // (computed here, as below)
                                if constexpr (HAS_Z) asm volatile("" : "+v"(yp[t]));
                                asm volatile("" : "+v"(dC[s + j][t]), "+v"(dB[s + j][t]), "+v"(pu[t]), "+v"(pd[t]), "+v"(dAp[j]));
                            }
                        dA[s] = dAp[0]; dA[s + 1] = dAp[1];
                    }
                } else
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const ACoef co = make_acoef<DISC>(Ak[s]);
                    slow_part();
                    // the checkpointed state enters through the half's first lane, the carried adjoint through its last
                    float xin = i2f(f2i(ck[s]) & (int)first_lane), Gin = i2f(f2i(hc[s]) & (int)last_lane);
                    float a[T], x[T], gg[T];
                    [[maybe_unused]] float q[T];                     // bilinear, see bilinear_q
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        // (an own copy for each state: multiples and powers of Delta are not kept in registers for the next)
                        if constexpr (DISC == DISC_ZOH || DISC == DISC_BILINEAR) asm volatile("" : "+v"(dl[t]));
                        if constexpr (DISC == DISC_BILINEAR) {
                            q[t] = bilinear_q(dl[t], co);
                            a[t] = bilinear_a(q[t]);
                            gg[t] = dl[t] * q[t];
                        } else disc_ag<DISC>(dl[t], co, a[t], gg[t]);
                        if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) x[t] = du[t] * Bv[s][t];
                        else x[t] = gg[t] * du[t] * Bv[s][t];
                    }
                    // folds of the lane's steps: S the end state, Q = a_0 (c_0 + a_1 (c_1 + ...)) the adjoint handed on,
                    // both with multiplier P
                    float S = __builtin_fmaf(a[0], xin, x[0]), Q = Gin, P;
#pragma unroll
                    for (int t = 1; t < T; ++t) S = __builtin_fmaf(a[t], S, x[t]);
#pragma unroll
                    for (int t = T - 1; t >= 0; --t) Q = a[t] * __builtin_fmaf(Cv[s][t], dy[t], Q);
                    if constexpr (DISC == DISC_BILINEAR) {
                        if constexpr (T == 8) P = ((a[0] * a[1]) * (a[2] * a[3])) * ((a[4] * a[5]) * (a[6] * a[7]));
                        else if constexpr (T == 4) P = (a[0] * a[1]) * (a[2] * a[3]);
                        else P = a[0] * a[1];
                    } else P = exp2_fast(sum_dl * co.A2);
                    if constexpr (DISC == DISC_BILINEAR) {           // (there are no registers to keep the multipliers beside q)
#pragma unroll
                        for (int t = 0; t < T; ++t) asm volatile("" : "+v"(q[t]));
                    }
                    half_scans(P, S, Q, xin, Gin);
                    if (first_lane) at[s] = Q;                       // carried to the earlier tile
                    fast_part();
                    // replay of the states (earliest step first) and of the adjoint (last step first), side by side: two chains
                    // whose instructions fill each other's result latencies.  zoh and bilinear, which need more registers and
                    // have more instructions a step to fill them with, take the adjoint step by step below instead (side by
                    // side zoh spilled 50 registers).
                    constexpr bool APART = DISC == DISC_ZOH || DISC == DISC_BILINEAR;
                    float R[T], G[T];
                    {
                        float xp = xin;
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            const int r = T - 1 - t;
                            if constexpr (!APART) R[r] = __builtin_fmaf(Cv[s][r], dy[r], Gin);                 // H_r
                            if constexpr (DISC == DISC_BILINEAR) a[t] = bilinear_a(q[t]);
                            xp = __builtin_fmaf(a[t], xp, x[t]); x[t] = xp;
                            if constexpr (!APART) {
                                Gin = a[r] * R[r];                                       // a_r H_r
                                G[r] = Gin;
                            }
                        }
                    }
                    auto acc = [&](float &sum, float m1, float m2) { sum = (s == 0) ? m1 * m2 : __builtin_fmaf(m1, m2, sum); };
                    float dAp = 0.0f;
#pragma unroll
                    for (int t = T - 1; t >= 0; --t) {
                        const float xprev = t > 0 ? x[t - 1] : xin;
                        if constexpr (APART) {
                            asm volatile("" : "+v"(dl[t]));
                            R[t] = __builtin_fmaf(Cv[s][t], dy[t], Gin);
                            if constexpr (DISC == DISC_BILINEAR) {
                                G[t] = q[t] * R[t];
                                Gin = __builtin_fmaf(2.0f, G[t], -R[t]);         // a R
                            } else Gin = a[t] * R[t];
                        }
                        dC[s][t] = __builtin_fmaf(dy[t], x[t], dC[s][t]);
                        if constexpr (HAS_Z) acc(yp[t], Cv[s][t], x[t]);
                        if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) {
                            // S6: g = Delta (du and dDelta share sum_n H B, scaled in the epilogue); dirac: g = 1, and
                            // only a = e^{Delta A} depends on Delta and A
                            acc(pu[t], R[t], Bv[s][t]);
                            dB[s][t] = __builtin_fmaf(R[t], du[t], dB[s][t]);
                            const float q = G[t] * xprev;
                            acc(pd[t], q, co.A);
                            dAp = __builtin_fmaf(q, dl[t], dAp);
                        } else if constexpr (DISC == DISC_ZOH) {
                            // da/dDelta = A a, da/dA = Delta a, dg/dDelta = a: the common factor a is taken out
                            const float g_A = zoh_gain_dA(dl[t], co, a[t], gg[t]);
                            const float hb = R[t] * Bv[s][t];
                            const float dg = hb * du[t];
                            const float q = Gin * xprev;
                            acc(pu[t], hb, gg[t]);
                            dB[s][t] = __builtin_fmaf(R[t] * gg[t], du[t], dB[s][t]);
                            if (s == 0) pd[t] = __builtin_fmaf(q, co.A, dg * a[t]);
                            else pd[t] = __builtin_fmaf(q, co.A, __builtin_fmaf(dg, a[t], pd[t]));
                            dAp = __builtin_fmaf(q, dl[t], __builtin_fmaf(dg, g_A, dAp));
                        } else {
                            // bilinear: g = Delta q, and all four partials are multiples of q^2: da/dDelta = A q^2, da/dA = Delta q^2,
                            // dg/dDelta = q^2, dg/dA = Delta^2 q^2 / 2.  One factor q sits in G = q R.
                            const float qB = G[t] * Bv[s][t], da = G[t] * xprev, dg = qB * du[t];
                            acc(pu[t], qB, dl[t]);
                            dB[s][t] = __builtin_fmaf(G[t] * dl[t], du[t], dB[s][t]);
                            acc(pd[t], __builtin_fmaf(da, co.A, dg), q[t]);
                            dAp = __builtin_fmaf(__builtin_fmaf(0.5f * dl[t], dg, da) * dl[t], q[t], dAp);
                        }
                        // computed here: left to itself the compiler moves the products of one state down to the sums of the
                        // next one's, and spills what it then has to keep
                        if constexpr (HAS_Z) asm volatile("" : "+v"(yp[t]));
                        asm volatile("" : "+v"(dC[s][t]), "+v"(dB[s][t]), "+v"(pu[t]), "+v"(pd[t]), "+v"(dAp));
                    }
                    dA[s] = dAp;
                }
                slow_part();
                // dA: over the 16 lanes of a row
                float *sum = sdA + g * N + n0 + cN;
                if constexpr (NS == 4) {
                    const float v = row_sums4(dA[0], dA[1], dA[2], dA[3]);
                    if (__builtin_amdgcn_inverse_ballot_w64(0x1111111111111111)) lds_add(sum + (ln >> 2 & 3), v);
                } else {
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        float v = dA[s];
                        v += dpp<0xB1>(0.0f, v);
                        v += dpp<0x4E>(0.0f, v);
                        v += dpp<0x124>(0.0f, v);
                        v += dpp<0x128>(0.0f, v);
                        if ((ln & 15) == 0) lds_add(sum + s, v);
                    }
                }
        };
        __syncthreads();                                 // the tables (first tile) are in place; the tile before is done
        if constexpr (STAGED) stage_maps();
        if constexpr (OWN) {
            for (int g = 0; g < Gact; g += CP) {
                const unsigned t0 = fresh(tid);
                float u[T], dl[T], dy[T], du[T], yp[T], pu[T], pd[T];
                step_inputs(g + c_own, sBias[g + c_own], t0, even, u, dl, dy);
                put_ac(t0, 0);
                fetch(t0);
#pragma unroll
                for (int t = 0; t < T; ++t) du[t] = u[t];
                __syncthreads();                         // (one wavefront: orders the LDS accesses only)
                states(g, 0, t0, dl, du, dy, yp, pu, pd);
                finish(g, even, t0, (t0 % NTC) * TPT, dl, u, dy, yp, pu, pd, sDskip[g + c_own < Gact ? g + c_own : Gact - 1]);
                __syncthreads();
            }
        } else {
            // A pass's steps are read from LDS behind the epilogue's reads and ahead of its arithmetic, and the next pair's biases ahead of
            // the stores of the partial sums: what is read is there when it is needed (277.7 -> 271.6 us on the training shape above).
            float dl[T], du[T], dy[T], bias;
            auto lane_at = [&](unsigned ln) { return (unsigned)lane_slot<PAIR, T>(ln & 31) + (ln & 32) * (TILE / 32); };
            unsigned l4 = 0;                             // where this lane's steps are in a plane (float32: formed again, a register less)
            auto main_read = [&](const int buf) {
                l4 = lane_at(fresh(lane));
                lds_steps_read<T>(sPair + buf, l4, dl);
                lds_steps_read<T>(sPair + buf + PL, l4, du);
                lds_steps_read<T>(sPair + buf + 2 * PL, l4, dy);
            };
            auto main_part = [&](const int g, const int buf) {
                const unsigned ln = fresh(lane);
                float yp[T], pu[T], pd[T];
                states(g, buf, ln, dl, du, dy, yp, pu, pd);
                edge_part();
                if constexpr (sizeof(IO) == 4) l4 = lane_at(fresh(ln));
                bias = sBias[g + CP + c_own];                // (past the last pair: not used)
                float *part = sPair + buf + (3 + 3 * w) * PL;
                if constexpr (HAS_Z) lds_steps_write<T>(part, l4, yp);
                lds_steps_write<T>(part + PL, l4, pu);
                lds_steps_write<T>(part + 2 * PL, l4, pd);
            };
            auto next_inputs = [&](const int g, Kept &k, const int buf) {          // (past the last pair: unused)
                const unsigned t0 = fresh(tid);
                prologue(g + c_own, bias, t0, k, buf);
                fetch(t0);
            };
            constexpr auto nothing = [] {};
            bias = sBias[c_own];
            next_inputs(0, even, 0);
            if constexpr (STAGED) { __syncthreads(); take_maps(); }
            if constexpr (NB == 2) {
                // Between two barriers a wavefront finishes the pair before (its partial sums are complete), runs the main
                // part of this pair and prepares the next one: nobody waits in between.  (Two barriers per pair cost 4 %.)  Written out for the
                // two buffers: with the buffer in a variable the kept values are copied and addresses formed in every pass.
                auto pass = [&](const int g, Kept &kept, const int buf, Kept &other, const int next) {
                    __syncthreads();
                    if (g > 0) epilogue(g - CP, other, next, [&] { main_read(buf); }); else main_read(buf);
                    main_part(g, buf);
                    next_inputs(g + CP, other, next);
                };
                int g = 0;
                if constexpr (FULL) {
                    for (; g + CP < Gact; g += 2 * CP) {
                        pass(g, even, 0, odd, BUF);
                        pass(g + CP, odd, BUF, even, 0);
                    }
                    if (g < Gact) {
                        pass(g, even, 0, odd, BUF);
                        __syncthreads();
                        epilogue(g, even, 0, nothing);
                    } else {
                        __syncthreads();
                        epilogue(g - CP, odd, BUF, nothing);
                    }
                } else {
                    int buf = 0;
                    for (; g < Gact; g += CP, buf = BUF - buf) {
                        __syncthreads();
                        if (g > 0) epilogue(g - CP, odd, BUF - buf, nothing);
                        odd = even;
                        main_read(buf);
                        main_part(g, buf);
                        next_inputs(g + CP, even, BUF - buf);
                    }
                    __syncthreads();
                    epilogue(g - CP, odd, BUF - buf, nothing);
                }
            } else {
                for (int g = 0; g < Gact; g += CP) {
                    __syncthreads();
                    odd = even;
                    main_read(0);
                    main_part(g, 0);
                    __syncthreads();
                    epilogue(g, odd, 0, nothing);
                    next_inputs(g + CP, even, 0);
                }
            }
        }

        // ---- the tile's sums of dBm and dCm over this workgroup's channels
        // (the two halves hold different channels: summed by a swap that leaves the lower half with the first half of a lane's
        // steps, the upper half with the others)
        constexpr int TH = T / 2;
        float oB[NS][TH], oC[NS][TH];
        auto put = [](float *m, const float (&v)[TH]) {
            if constexpr (TH == 4) *reinterpret_cast<float4 *>(m) = make_float4(v[0], v[1], v[2], v[3]);
            else if constexpr (TH == 2) *reinterpret_cast<float2 *>(m) = make_float2(v[0], v[1]);
            else m[0] = v[0];
        };
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int t = 0; t < TH; ++t) {
                const auto r = __builtin_amdgcn_permlane32_swap((unsigned)f2i(dB[s][t]), (unsigned)f2i(dB[s][t + TH]), false, false);
                const auto q = __builtin_amdgcn_permlane32_swap((unsigned)f2i(dC[s][t]), (unsigned)f2i(dC[s][t + TH]), false, false);
                oB[s][t] = i2f((int)r[0]) + i2f((int)r[1]);
                oC[s][t] = i2f((int)q[0]) + i2f((int)q[1]);
            }
        if constexpr (PART) {
            // to this workgroup's own slot of the workspace, as 16-byte pieces in the order the lanes hold them (the sum
            // over workgroups and the transposition to [L,N] are k_ss_bwd_maps's)
            const int r = piece_of<PAIR>(li) * T + half * TH;            // [step % 8 / 4][step / 8][step % 4], for any T
            const int at = T == 8 ? (half * 32 + piece_of<PAIR>(li)) * 4 : ((r & 4) << 5) + (r >> 3 << 2) + (r & 3);
            float *pt = q.part + (((slot0 + tile_first + tile) * gridDim.x + blockIdx.x) * 2 * N + n0) * TILE + at;
#pragma unroll
            for (int s = 0; s < NS; ++s) { put(pt + s * TILE, oB[s]); put(pt + (N + s) * TILE, oC[s]); }
        } else {
            // without a workspace: float atomics, on consecutive addresses (the sums change their order in LDS: lanes that add
            // 8 steps apart take a transaction each, 8 times as long)
            const unsigned t0 = fresh(tid), st0 = piece_of<PAIR>(t0 & 31) * T + (t0 >> 5 & 1) * TH;
            if constexpr (OWN) {
                float *gB = q.dBm + bc0 + l0 * N, *gC = q.dCm + bc0 + l0 * N;
#pragma unroll
                for (int t = 0; t < TH; ++t)
                    if ((int)st0 + t < rem) {
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            unsafeAtomicAdd(gB + (st0 + t) * N + s, oB[s][t]);
                            unsafeAtomicAdd(gC + (st0 + t) * N + s, oC[s][t]);
                        }
                    }
            } else {
                static_assert(OWN || N * TILE <= NB * BUF, "one map's sums in the pairs' place");
                float *buf = sPair;
                auto flush = [&](float (&o)[NS][TH], float *g) {
                    __syncthreads();
#pragma unroll
                    for (int s = 0; s < NS; ++s) put(buf + (n0 + s) * TILE + st0, o[s]);
                    __syncthreads();
#pragma unroll 1
                    for (int i = t0; i < rem * N; i += NT) unsafeAtomicAdd(g + bc0 + l0 * N + i, buf[(i % N) * TILE + i / N]);
                };
                flush(oB, q.dBm);
                flush(oC, q.dCm);
            }
        }
    };
    const int whole = vec ? (int)(L / TILE) : 0;         // tiles known to be whole
    int64_t tile = ntiles - 1;
    if constexpr (!OWN) {
        const int64_t left = L - tile * TILE;        // steps of the last tile
        if (tile >= 0 && left <= 128) {
            if (left <= 64) do_tile(tile, std::false_type{}, std::integral_constant<int, 2>{});
            else do_tile(tile, std::false_type{}, std::integral_constant<int, 4>{});
            --tile;
        }
    }
    for (; tile >= 0; --tile) {
        constexpr std::integral_constant<int, 8> eight{};
        if (tile < whole) do_tile(tile, std::true_type{}, eight); else do_tile(tile, std::false_type{}, eight);
    }
    __syncthreads();
    // ---- per-channel results of this workgroup
    const bool own = PART && p.rows.sb >= 0;         // see RowSums
    float *oA = p.dA, *oD = p.dD, *ob = p.dbias;
    if (own) {
        const int64_t at = b * p.rows.sb;
        oA = p.rows.A + at; oD = oD ? p.rows.D + at : oD; ob = ob ? p.rows.b + at : ob;
    }
    auto leave = [&](float *at, float v) { if (own) *at = v; else unsafeAtomicAdd(at, v); };
    for (int i = tid; i < Gact * N; i += NT) {
        leave(oA + (int64_t)d0 * N + i, sdA[i]);
        if (p.dx0 && chunk == 0) p.dx0[((int64_t)b * p.D + d0) * N + i] = sH[i];
    }
    for (int g = tid; g < Gact; g += NT) {
        if (oD) leave(oD + d0 + g, sdDb[0][g]);
        if (ob) leave(ob + d0 + g, sdDb[1][g]);
    }
}

// a boundary as a step of the axis, and the sequence whose tiles start last at or before a slot: sequence b's start at cu[b] / 256 + b
__device__ __forceinline__ int64_t axis_step(int64_t o, int64_t Lp) { return o < 0 ? 0 : (o > Lp ? Lp : o); }
__device__ __forceinline__ int seq_of_slot(const int64_t *cu, int B, int64_t Lp, int64_t slot) {
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (axis_step(cu[mid], Lp) / kBwdTileSteps + mid <= slot) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// dBm, dCm [.., L, N] from the tile sums the workgroups of k_ss_bwd left in the workspace: a workgroup adds one piece of a
// tile (blockIdx.x) of one of the two maps (blockIdx.y) of one group (blockIdx.z) over the channel blocks, always in the same order, and
// transposes it through LDS.  With many tiles it is bound by the reads of the workspace, whole lines of 128 bytes (half lines, as the pieces
// of 32 states, or of 16 complex ones, once were: 32 blocks of 64 tiles 41 us, now 22 or 6.0 TB/s).  With few tiles of many channel blocks a
// chain of reads is what it waits for: KS threads then share an element, each a quarter of the blocks, and a
// workgroup takes a quarter of the piece (whole call, bf16, L = 512: 1024 rows, N = 16 49 us, so 41; 4096 rows 73 and 57, N = 4
// 57 and 42).
template <int N> struct BwdMaps {
    // pieces of a tile, of one thread an element: of time as long as what is read of a state stays whole lines, then of the states
    static constexpr int TIME = N >= 16 ? 4 : N >= 8 ? N / 4 : 1, STATES = N > 16 ? N / 16 : 1, PIECES = TIME * STATES;
};
template <int N, int KS>
__global__ __launch_bounds__(256) void k_ss_bwd_maps(const BwdParams p, int gx) {
    constexpr int PT = N * kBwdTileSteps;            // floats of one map's sums of one tile
    // the quarter of a piece is one of time as long as what is read of a state stays whole lines of 128 bytes, and one of the
    // states beyond that (cut to 32 bytes, the sums of 4096 rows of 2048 steps, N = 16, took 40 us longer)
    constexpr int LS = KS == 1 || N >= 16 ? 1 : KS * 4 / N, NP = KS / LS * BwdMaps<N>::STATES;
    constexpr int PIECES = BwdMaps<N>::TIME * LS;
    constexpr int LP = 32 / PIECES;                  // lanes (of 8 steps) of a piece
    constexpr int SP = LP * 8;                       // its steps
    constexpr int NW = N / NP;                       // its states
    constexpr int NE = NW * LP * 2;                  // its elements of four steps
    static_assert(LP * PIECES == 32 && (KS == 1 ? NE <= 256 : NE == 64 && KS == 4), "a thread for each element, a wavefront for each share of the blocks");
    __shared__ float sT[SP * (NW + 1)];
    __shared__ float4 sK[KS > 1 ? KS * NE : 1];
    if (blockIdx.x >= p.rows.first) {
        const int64_t nA = (int64_t)p.D * N;
        const unsigned nz = p.rows.clear, at = blockIdx.x - p.rows.first;
        if (at < nz) {                               // a packed batch: the rows of this map outside every sequence are zero
            float *out = (blockIdx.y ? p.dCm : p.dBm) + (int64_t)blockIdx.z * p.L * N;
            const int s = threadIdx.x & 63;
            static_assert(kRowSumsMaxB <= 64, "a lane for each sequence");
            if (__builtin_amdgcn_ballot_w64(s < p.B && axis_step(p.cu[s], p.L) > axis_step(p.cu[s + 1], p.L))) {
                // Boundaries that descend somewhere are not refused.  What they leave out may lie anywhere, and what is before the first or
                // after the last may be some sequence's: row by row those that no other workgroup of this launch writes.
                for (int64_t r = at * 256 + threadIdx.x; r < p.L; r += (int64_t)nz * 256) {
                    bool written = false;
                    for (int b = 0; b < p.B; ++b) {
                        const SeqSpan q = seq_span_fwd<false>(p.cu, p.B, p.L, b);
                        const int64_t in = r - q.toff;
                        written |= in >= 0 && in < q.L && seq_of_slot(p.cu, p.B, p.L, (q.toff / kBwdTileSteps + b) + in / kBwdTileSteps) == b;
                    }
                    if (!written)
                        for (int n = 0; n < N; ++n) out[r * N + n] = 0.0f;
                }
                return;
            }
            const int64_t head = axis_step(p.cu[0], p.L), rows = head + p.L - axis_step(p.cu[p.B], p.L);
            for (int64_t i = at * 256 + threadIdx.x; i < rows * N; i += (int64_t)nz * 256)
                out[i < head * N ? i : p.L * N - rows * N + i] = 0.0f;
            return;
        }
        // dA, dD, dbias from what the workgroups left for each batch entry
        const int64_t e = (int64_t)(at - nz) * 256 + threadIdx.x;
        if (blockIdx.y || blockIdx.z || e >= nA + 2 * p.D) return;
        float *out = e < nA ? p.dA + e : e < nA + p.D ? (p.dD ? p.dD + (e - nA) : nullptr) : (p.dbias ? p.dbias + (e - nA - p.D) : nullptr);
        if (!out) return;
        float sum = 0.0f;
#pragma unroll 8
        for (int b = 0; b < p.B; ++b) sum += p.rows.A[b * p.rows.sb + e];
        *out = sum;
        return;
    }
    const int n0 = (blockIdx.x % NP) * NW;
    const int piece = (blockIdx.x / NP) % PIECES;
    const int64_t slot = blockIdx.x / (NP * PIECES);
    int64_t b, tile, toff = 0, L = p.L;
    if (p.cu) {
        b = seq_of_slot(p.cu, p.B, p.L, slot);
        const SeqSpan q = seq_span(p.cu, p.B, p.L, (int)b, false);
        toff = q.toff; L = q.L;
        tile = slot - (toff / kBwdTileSteps + b);
    } else {
        b = slot / p.part_tiles;
        tile = slot % p.part_tiles;
    }
    const int64_t l0 = tile * kBwdTileSteps + piece * SP;
    if (tile < 0 || l0 >= L) return;
    const int G = channels_of(p, (L + kBwdTileSteps - 1) / kBwdTileSteps);
    const int nblk = (p.dpg + G - 1) / G;
    const int grp = blockIdx.z;

    const int tid = threadIdx.x, el = tid % NE;
    // (wave-uniform, and with it the number of reads: a loop that lanes leave one by one reads one value at a time)
    const int ks = KS > 1 ? __builtin_amdgcn_readfirstlane(tid / NE) : 0;
    // this thread's four steps: of lane li of the piece (8 steps each), the first or the second four
    const int li = el % LP, q = (el / LP) & 1, n = el / (2 * LP);
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    auto add = [&](const auto v) { a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w; };
    if (KS > 1 || tid < NE) {
        const int at = (n0 + n) * kBwdTileSteps + q * 128 + (piece * LP + li) * 4;
        const float *src = p.part + ((slot * gx + (int64_t)grp * nblk) * 2 + blockIdx.y) * PT + at;
        const int k0 = nblk * ks / KS, k1 = nblk * (ks + 1) / KS;
        // read once and never again: non-temporal (packed batch of 24 sequences, 16384 steps, D = 1536: training step 572 -> 565 us)
        typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll 8
        for (int k = k0; k < k1; ++k) add(__builtin_nontemporal_load(reinterpret_cast<const f4 *>(src + (int64_t)k * 2 * PT)));
        if constexpr (KS > 1) sK[ks * NE + el] = a;
    }
    if constexpr (KS > 1) {
        __syncthreads();
        if (ks == 0) {
#pragma unroll
            for (int k = 1; k < KS; ++k) add(sK[k * NE + el]);
        }
    }
    if (ks == 0 && tid < NE) {
        float *t = sT + (li * 8 + q * 4) * (NW + 1) + n;
        t[0] = a.x; t[NW + 1] = a.y; t[2 * (NW + 1)] = a.z; t[3 * (NW + 1)] = a.w;
    }
    __syncthreads();
    float *out = (blockIdx.y ? p.dCm : p.dBm) + ((p.cu ? (int64_t)grp : b * p.bcg + grp) * p.L + toff + l0) * N;
    const int rows = L - l0 < SP ? (int)(L - l0) : SP;
    if constexpr (N >= 4) {
        const int r = tid / (NW / 4), m = (tid % (NW / 4)) * 4;
        static_assert(SP * NW / 4 <= 256, "one 16-byte piece per thread");
        if (r < rows) {
            const float *t = sT + r * (NW + 1) + m;
            *reinterpret_cast<float4 *>(out + r * N + n0 + m) = make_float4(t[0], t[1], t[2], t[3]);
        }
    } else {
        for (int i = tid; i < rows * N; i += 256) out[i] = sT[(i / N) * (N + 1) + i % N];
    }
}


// ---------------------------------------------------------------- launchers
// HAS_Z (gated) is a template parameter: without it the kernel does not rebuild ypre = sum_n C x for dz.  So is whether the
// tile sums go to the workspace: the code that adds them with atomics instead would cost the other kernel registers.
template <typename IO, int N, int DISC>
static hipError_t launch_bwd_n(const BwdParams &p, hipStream_t s) {
    dim3 grid(bwd_grid_x(p), p.B, p.nchunks > 1 ? p.nchunks : 1);
    const dim3 block(BwdGeom<N>::NT);
    if (p.part && p.z) hipLaunchKernelGGL((k_ss_bwd<IO, N, DISC, true, true>), grid, block, 0, s, p);
    else if (p.part) hipLaunchKernelGGL((k_ss_bwd<IO, N, DISC, false, true>), grid, block, 0, s, p);
    else if (p.z) hipLaunchKernelGGL((k_ss_bwd<IO, N, DISC, true, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((k_ss_bwd<IO, N, DISC, false, false>), grid, block, 0, s, p);
    return p.part ? launch_bwd_maps(p, (int)grid.x, s) : hipGetLastError();
}

template <typename IO, int DISC>
static hipError_t launch_bwd_disc(const BwdParams &p, hipStream_t s) {
    switch (p.N) {
        case 1: return launch_bwd_n<IO, 1, DISC>(p, s);
        case 2: return launch_bwd_n<IO, 2, DISC>(p, s);
        case 4: return launch_bwd_n<IO, 4, DISC>(p, s);
        case 8: return launch_bwd_n<IO, 8, DISC>(p, s);
        case 16: return launch_bwd_n<IO, 16, DISC>(p, s);
        case 32: return launch_bwd_n<IO, 32, DISC>(p, s);
    }
    return hipErrorInvalidValue;
}

template <typename IO>
static hipError_t launch_bwd_io(const BwdParams &p, int disc, hipStream_t s) {
    switch (disc) {
        case DISC_ZOH_S6: return launch_bwd_disc<IO, DISC_ZOH_S6>(p, s);
        case DISC_ZOH: return launch_bwd_disc<IO, DISC_ZOH>(p, s);
        case DISC_BILINEAR: return launch_bwd_disc<IO, DISC_BILINEAR>(p, s);
        case DISC_DIRAC: return launch_bwd_disc<IO, DISC_DIRAC>(p, s);
    }
    return hipErrorInvalidValue;
}

// float32 and bfloat16 are compiled side by side: selective_bwd_f32.hip includes this file for the former.
hipError_t launch_ss_bwd_f32(const BwdParams &p, int disc, hipStream_t s);
#ifdef LRNNX_BWD_F32
hipError_t launch_ss_bwd_f32(const BwdParams &p, int disc, hipStream_t s) { return launch_bwd_io<float>(p, disc, s); }
#else
hipError_t launch_ss_bwd(const BwdParams &p, int io_dtype, int disc, hipStream_t s) {
    if (p.G > kBwdMaxG) return hipErrorInvalidValue;       // (more channels than the tables in LDS hold)
    return io_dtype == 1 ? launch_bwd_io<bf16_t>(p, disc, s) : launch_ss_bwd_f32(p, disc, s);
}

// Workgroups that look after the rows of one map (`floats` a row) outside every sequence of a packed batch.  The host knows the length of the axis,
// not how much of it is unused: a workgroup for every 8192 floats of the map, and up to 512 of them.  Backward calls, bf16, us, with 16 workgroups and with
// these: 4 sequences, 2048 steps in all, 64 channels, N = 16, on an axis of 65536 steps 37.3 and 29.9, of 262144 70.3 and 36.9; 16 sequences, 4096 steps,
// 128 channels, N = 4, of 524288 37.7 and 22.6; with no step unused as before (27.6; 8 x 512 channels, 8192 steps 74.4).
unsigned bwd_clear_wgs(int64_t L, int floats) {
    const int64_t wgs = L * floats / 8192;
    return wgs < 16 ? 16 : wgs > 512 ? 512 : (unsigned)wgs;
}

template <int N>
static hipError_t launch_bwd_maps_n(const BwdParams &p, int gx, hipStream_t s) {
    const int64_t slots = p.cu ? p.nslots : (int64_t)p.B * p.part_tiles, pieces = slots * BwdMaps<N>::PIECES;
    // few workgroups, and more blocks than a thread's first two rounds of reads: measured over N = 4 to 32, 2 to 96 tiles, 10 to 128 blocks, the
    // choice is 1.1 % slower than the better of the two (geometric mean), at most 1.26 times.  N = 16, one and four threads an element, us: 64 blocks
    // of 8 tiles 10.6 and 3.5, of 32 tiles 12.7 and 12.4, of 64 tiles 20.9 and 24.7; 16 blocks of 8 tiles 3.1 and 3.2.
    constexpr int KS = N >= 4 ? 4 : 1;
    // A packed batch has slots without a tile, whose workgroups end at once and leave uneven numbers on the CUs: up to three a CU four threads can be the
    // faster (N = 16, D = 1536, one and four, us: 8 x 2048 steps 29.1 and 25.7, 24 of 16384 in all 27.2 and 26.8), with 32 states they are not.  Over 107
    // packed backward calls in that range (N = 4 to 16, real and complex, 256 to 4096 channels) the two are even: 1.000, 0.967 to 1.029.
    const int64_t wgs = pieces * 2 * p.bcg;
    const bool split = KS > 1 && gx / p.bcg > 16 && (2 * wgs < 3 * kNumCU || (p.cu && N <= 16 && wgs < 3 * kNumCU));
    dim3 g2((unsigned)(split ? pieces * KS : pieces), 2, p.bcg);
    BwdParams q = p;
    q.rows.first = g2.x;
    q.rows.clear = p.rows.sb >= 0 && p.cu ? bwd_clear_wgs(p.L, N) : 0;
    g2.x += q.rows.clear;
    if (p.rows.sb > 0) g2.x += (unsigned)(((int64_t)p.D * (N + 2) + 255) / 256);
    if (split) hipLaunchKernelGGL((k_ss_bwd_maps<N, KS>), g2, dim3(256), 0, s, q, gx);
    else hipLaunchKernelGGL((k_ss_bwd_maps<N, 1>), g2, dim3(256), 0, s, q, gx);
    return hipGetLastError();
}
hipError_t launch_bwd_maps(const BwdParams &p, int gx, hipStream_t s) {
    switch (p.N) {
        case 1: return launch_bwd_maps_n<1>(p, gx, s);
        case 2: return launch_bwd_maps_n<2>(p, gx, s);
        case 4: return launch_bwd_maps_n<4>(p, gx, s);
        case 8: return launch_bwd_maps_n<8>(p, gx, s);
        case 16: return launch_bwd_maps_n<16>(p, gx, s);
        case 32: return launch_bwd_maps_n<32>(p, gx, s);
    }
    return hipErrorInvalidValue;
}

// Workgroups the chip holds at once: two wavefronts per SIMD are what the registers allow.
int bwd_places(int N) { return 2048 / (N == 4 ? 2 : (N >= 4 ? N / 4 : 1)); }

// channels per workgroup: D here is the number of channels that share one pair of Bm/Cm maps.  `balanced` says
// that all batch entries have the same length; otherwise (packed variable-length batches) four times as many,
// smaller, workgroups let the dispatcher even out sequences of different lengths.
static int channels_for(int B, int D, int64_t full, bool balanced) {
    int64_t G = ((int64_t)B * D) / (balanced ? full : 2048);
    // All workgroups of a balanced launch take equally long: a few more than the chip holds would run as a second,
    // almost empty round (518 instead of 512 workgroups: 40 % slower).  So as many channel blocks per row group as
    // fit into a whole number of rounds, not one more (several rounds only when a block cannot hold more channels).
    if (balanced) {
        int64_t rounds = 1;
        while ((int64_t)B * ((D + kBwdMaxG - 1) / kBwdMaxG) > rounds * full && rounds < 64) ++rounds;
        const int64_t nb = rounds * full / B;          // channel blocks per row group
        if (nb >= 1) G = (D + nb - 1) / nb;
    }
    if (G < 8) G = 8;
    if (G > kBwdMaxG) G = kBwdMaxG;
    if (G > D) G = D;
    const int64_t groups = (D + G - 1) / G;
    return (int)((D + groups - 1) / groups);           // even split
}
// a workgroup walks its channels in pairs
static int whole_passes(int G) {
    return (G + 1) / 2 * 2;
}
int bwd_channels_per_group(int B, int D, int N, int64_t, bool balanced) {
    return whole_passes(channels_for(B, D, bwd_places(N), balanced));
}

void packed_shape(int B, int D, int dpg, int64_t L, int64_t max_seqlen, int Gbal, int most, double gain, int places, int *G, int *wcap, int *gmin) {
    *wcap = 0; *gmin = *G;
    if (max_seqlen <= 0) return;
    // what each place of the chip gets at perfect balance, in channel-tiles: D channels x the tiles of all sequences
    // (each sequence rounded up by half a tile on average), and the channels of the longest sequence that come to that
    const double tiles = (double)L / kBwdTileSteps + 0.5 * B;
    const double cap = (double)D * tiles / places;
    const int64_t longest = (max_seqlen + kBwdTileSteps - 1) / kBwdTileSteps;
    const double fit = cap / (double)longest;
    // sequences of about one length: the launch shape of a batch [B,D,L] (whole rounds of equal workgroups, as many
    // channels each as that allows) is within a tenth of perfect balance and pays staging and flush less often
    if (Gbal > *G && (double)Gbal <= 1.1 * fit) { *G = *gmin = Gbal; return; }
    // Otherwise the workgroups start longest first, and what evens the launch out is that the last ones are short, not that there are
    // many: as long as the longest sequence's workgroups are a fifth below a place's share and there are two workgroups for each
    // place, more channels each cost no balance, and the tile sums and what is paid per tile and workgroup become less (24 sequences,
    // 16384 steps, 1536 channels, N = 16, bf16: 18 -> 26 channels, training step 531 -> 512 us).  Backward calls that this widens, bf16, 3 to 96
    // sequences of 4096 to 32768 steps in all, 256 to 4096 channels, lengths from nearly equal to log-normal with sigma 1.2, time after / before: real
    // pass, 130 calls with N = 16 and 32, 0.915 (geometric mean; 0.58 to 1.12); with fewer states the launch is as wide already.
    // Complex pass, 90 calls with N = 4 to 16, 0.976 (0.82 to 1.15), and a third more channels or nothing (`gain`) 0.976 with half of the losses
    // above 5 %; the real pass loses with such a bound (0.922).
    const int64_t two = (int64_t)B * D / (2 * places);
    const int64_t wide = 0.8 * fit < (double)two ? (int64_t)(0.8 * fit) : two;
    if (fit >= (double)*G && wide > *G) {
        const int64_t g = wide < most ? wide : most, blocks = (dpg + g - 1) / g;
        const int even = (int)((dpg + blocks - 1) / blocks + 1) & ~1;
        if (even > *G && even >= gain * *G) *G = *gmin = even;
    }
    if (fit >= (double)*G || *G <= kBwdMinG) return;    // the longest sequence is no longer than a fair share: no cap
    *wcap = cap < 1.0 ? 1 : (cap > 1e9 ? 1000000000 : (int)cap);
    *gmin = fit < (double)kBwdMinG ? kBwdMinG : (int)fit & ~1;
}
void bwd_packed_shape(int B, int D, int bcg, int N, int64_t L, int64_t max_seqlen, int *G, int *wcap, int *gmin) {
    packed_shape(B, D, D / bcg, L, max_seqlen, bwd_channels_per_group(B * bcg, D / bcg, N, L, true), kBwdMaxG, 1.0, bwd_places(N), G, wcap, gmin);
}

// launch shape incl. the chunked path for few rows and long sequences (selective_bwd_carry.hip)
BwdPlan bwd_plan(int rowsg, int dpg, int N, int64_t L, int mode, bool balanced) {
    const int G = channels_for(rowsg, dpg, bwd_places(N), balanced), pairs = whole_passes(G);
    const bool roomy = bwd_part_bytes(N, (L + kBwdTileSteps - 1) / kBwdTileSteps, (int64_t)rowsg * ((dpg + pairs - 1) / pairs)) < kBwdSumsCap;
    BwdPlan pl = plan_time_chunks(rowsg, dpg, L, balanced ? mode : 1, G, bwd_places(N), kBwdMaxG, roomy);
    pl.G = whole_passes(pl.G);
    return pl;
}

// grid.x of a backward launch and the workspace its tile sums of dBm and dCm take
int bwd_grid_x(const BwdParams &p) {
    const int gmin = p.wcap > 0 ? p.gmin : p.G;                       // fewest channels a workgroup may take
    return p.bcg * ((p.dpg + gmin - 1) / gmin);
}
size_t bwd_part_bytes(int N, int64_t tile_slots, int64_t grid_x) {
    return (size_t)tile_slots * grid_x * 2 * N * kBwdTileSteps * sizeof(float);
}
#endif

}  // namespace lrnnx
