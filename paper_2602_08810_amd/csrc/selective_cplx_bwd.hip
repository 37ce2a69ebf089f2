// Backward selective scan with a COMPLEX diagonal state matrix for gfx950: reverse-mode derivative of
//     x_{l,n} = a(Delta_l, A[d,n]) x_{l-1,n} + g(Delta_l, A[d,n]) Bm[b,l,n] u[b,d,l]        (complex)
//     y[b,d,l] = Re( sum_n Cm[b,l,n] x_{l,n} ) + Dskip[d] u[b,d,l],  then the optional gate
// (Eq. 2 of the paper with a complex diagonal A as in the layers of Sec. 2.2.1, states recomputed from checkpoints
// as Sec. 3 prescribes for the real scan).
//
// The gradient of the real loss with respect to a complex quantity q is dLoss/dRe q + i dLoss/dIm q.  The kernel carries
// the conjugates of all of them: with K_l the conjugate of grad x_l every conjugation of the chain rule drops out (a and g
// are holomorphic in A), and it is put back where a gradient leaves the kernel.  For one (b,d) row and one state n:
//     K_l       = Cm_l dypre_l + a_{l+1} K_{l+1}                    (the same affine scan, time reversed)
//     dCm_l*   += dypre_l x_l              dBm_l* += K_l g_l u_l
//     du_l     += Re(K_l g_l Bm_l)         grad a_l* = K_l x_{l-1}        grad g_l* = K_l Bm_l u_l
//     dDelta_l += Re(grad a_l* da/dDelta + grad g_l* dg/dDelta)
//     dA_n*    += grad a_l* da/dA + grad g_l* dg/dA
//
// Mapping: that of the real backward kernel (selective_bwd.hip).  A workgroup of W = N/2 wavefronts works on one tile of 256
// steps at a time, last tile first, and on two channels at a time: the halves of a wavefront are the two channels, a lane of
// a half owns T = 8 consecutive steps.  A wavefront holds two states.  The two rows of 16 lanes of a half hold alternate
// pieces of the tile: lane i of row r has the steps 16 i + 8 r .. 16 i + 8 r + 7.  After the lanes' folds a row swap then
// gives the lanes of row 0 both pieces of state 0 and those of row 1 both pieces of state 1, so that one scan over the 16
// lanes of a row serves both states (piece_scans): 92 vector instructions for both scans of two states, 174 with a scan over
// 32 lanes for each.  A lane's sums of dBm and dCm over the channels of the workgroup stay in registers; both maps of the tile
// sit in LDS as fp32 pairs, and what is summed over states (ypre, du, dDelta) goes through LDS once per pair of channels.
//
// What bounds it: vector-ALU issue, 65 instructions per state update (57.6 of them in the main part, among them 18 folds and
// replays with two multiply-adds a component, 9 for the multiplier, 6 for the scans), the rest is
// lost where a wavefront waits for LDS or at the one barrier of a pass and the other of its SIMD cannot fill in alone.
// B=8, D=1536, N=16, L=2048, bf16: 1505 us with time on 64 lanes of 4 steps and a scan of 64 lanes for each state (116
// instructions an update), then 935, with its parts at the priorities of scan_common.hpp 736,
// and without bank conflicts in prologue and epilogue 678.  B=4, D=2560, L=2048: call
// 1288 us, then 811 before the priorities; N = 4: 686 and 265.
#include "kernels.hpp"
#include "scan_common.hpp"
#include "cplx_common.hpp"
#include <type_traits>

namespace lrnnx {

// Geometry of a workgroup for N states.
template <int N> struct CBwdGeom {
    static constexpr int NS = N >= 2 ? 2 : 1;        // states of a wavefront
    static constexpr int W = N / NS;                 // wavefronts
    static constexpr int NT = W * 64;
    static constexpr int CP = 2;                     // channels per pass
    static constexpr bool OWN = W == 1;              // a lane's steps of the main part are its own of prologue and epilogue
    // eight wavefronts: the first four prepare the next pair while the last four finish the one before (two steps a thread:
    // with one step a thread the fixed part of both would be paid twice)
    static constexpr bool SPLIT = W == 8;
    static constexpr int NA = SPLIT ? NT / 2 : NT;   // threads of a prologue or an epilogue
    static constexpr int TPT = CP * kBwdTileSteps / NA;       // steps of a thread there
    static constexpr int NTC = kBwdTileSteps / TPT;           // threads that share a channel there
    static constexpr int NB = W >= 4 ? 2 : 1;        // buffers of the inputs
    // planes of the inputs: Delta, u, dypre (eight wavefronts: and d softplus, dz factor; one wavefront: u and the latter two,
    // which it needs again only after its main part)
    static constexpr int IN = SPLIT ? 5 : 3;
};

// The lane of a half that owns piece q of the tile (8 steps each), and the place of step f in a plane of 256 floats in LDS:
// [step % 8 / 4][lane][step % 4], the second half rotated by 16 floats and the lanes of the odd row by 8, so that a lane's 8
// steps and the few steps of consecutive threads are both free of bank conflicts (see step_slot in selective_bwd.hip).
__device__ __forceinline__ int piece_lane(int q) { return ((q & 1) << 4) + (q >> 1); }
__device__ __forceinline__ int lane_slot(int li) { return (li << 2) ^ ((li & 16) >> 1); }
__device__ __forceinline__ int cstep_slot(int f) {
    return ((f & 4) << 5) + (lane_slot(piece_lane(f >> 3)) ^ ((f & 4) << 2)) + (f & 3);
}
template <int CNT>
__device__ __forceinline__ void csteps_read(const float *plane, int slot, float *out) {
    if constexpr (CNT == 2) { const float2 v = *reinterpret_cast<const float2 *>(plane + slot); out[0] = v.x; out[1] = v.y; }
    else {
#pragma unroll
        for (int q = 0; q < CNT / 4; ++q) {
            const float4 v = *reinterpret_cast<const float4 *>(plane + (q ? (slot ^ 16) + 128 : slot));
            out[4 * q] = v.x; out[4 * q + 1] = v.y; out[4 * q + 2] = v.z; out[4 * q + 3] = v.w;
        }
    }
}
template <int CNT>
__device__ __forceinline__ void csteps_write(float *plane, int slot, const float *v) {
    if constexpr (CNT == 2) *reinterpret_cast<float2 *>(plane + slot) = make_float2(v[0], v[1]);
    else {
#pragma unroll
        for (int q = 0; q < CNT / 4; ++q)
            *reinterpret_cast<float4 *>(plane + (q ? (slot ^ 16) + 128 : slot)) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
}

// Over the 16 lanes of each row: S becomes the inclusive prefix (lane 0 first) of the pairs (P, S), Q the inclusive suffix
// (lane 15 first) of the pairs (P, Q); X the prefix of the lane before, Y the suffix of the lane after (lane 0 resp. 15
// keeps what it came with).  A step needs the product over the lanes up to its own for S and from its own on for Q: the
// latter is the former of a lane further on.  Lanes whose source does not exist are left unchanged (the products are then
// not complete, and not used).  A DPP read comes two instructions or more after the write of its register.
__device__ __forceinline__ void crow_scans(float2 P, float2 &S, float2 &Q, float2 &X, float2 &Y) {
    float t, u, nx, ny, rx, ry;
#define LRNNX_ROW " row_mask:0xf bank_mask:0xf\n\t"
    // S += shr(S) P, Q += shl(Q) R of distance D; (NX, NY): the product over twice the distance
#define LRNNX_CS(D, PX, PY, RX, RY, M1, M2, M3, M4)                                                                       \
    "v_mov_b32 %4, %0\n\tv_mov_b32 %5, %2\n\t" M1                                                                          \
    "v_fmac_f32_dpp %0, %0, " PX " row_shr:" #D LRNNX_ROW "v_fmac_f32_dpp %2, %2, " RX " row_shl:" #D LRNNX_ROW M2         \
    "v_fmac_f32_dpp %0, -%1, " PY " row_shr:" #D LRNNX_ROW "v_fmac_f32_dpp %2, -%3, " RY " row_shl:" #D LRNNX_ROW M3       \
    "v_fmac_f32_dpp %1, %1, " PX " row_shr:" #D LRNNX_ROW "v_fmac_f32_dpp %3, %3, " RX " row_shl:" #D LRNNX_ROW            \
    "v_fmac_f32_dpp %1, %4, " PY " row_shr:" #D LRNNX_ROW "v_fmac_f32_dpp %3, %5, " RY " row_shl:" #D LRNNX_ROW M4
#define LRNNX_CSP(D, E, PX, PY, RX, RY, NX, NY)                                                                           \
    LRNNX_CS(D, PX, PY, RX, RY, "v_mul_f32_dpp " NX ", " PX ", " PX " row_shr:" #D LRNNX_ROW,                              \
             "v_fmac_f32_dpp " NX ", -" PY ", " PY " row_shr:" #D LRNNX_ROW "v_mul_f32_dpp " NY ", " PX ", " PY " row_shr:" #D LRNNX_ROW, \
             "v_fmac_f32_dpp " NY ", " PY ", " PX " row_shr:" #D LRNNX_ROW,                                                \
             "v_mov_b32_dpp %8, " NX " row_shl:" #E LRNNX_ROW "v_mov_b32_dpp %9, " NY " row_shl:" #E LRNNX_ROW)
    asm("s_nop 1\n\t"
        LRNNX_CSP(1, 1, "%10", "%11", "%10", "%11", "%6", "%7")
        LRNNX_CSP(2, 3, "%6", "%7", "%8", "%9", "%10", "%11")
        LRNNX_CSP(4, 7, "%10", "%11", "%8", "%9", "%6", "%7")
        LRNNX_CS(8, "%6", "%7", "%8", "%9", "", "", "",
                 "v_mov_b32_dpp %12, %0 row_shr:1" LRNNX_ROW "v_mov_b32_dpp %14, %2 row_shl:1" LRNNX_ROW
                 "v_mov_b32_dpp %13, %1 row_shr:1" LRNNX_ROW "v_mov_b32_dpp %15, %3 row_shl:1 row_mask:0xf bank_mask:0xf")
        : "+v"(S.x), "+v"(S.y), "+v"(Q.x), "+v"(Q.y), "=&v"(t), "=&v"(u), "=&v"(nx), "=&v"(ny), "=&v"(rx), "=&v"(ry),
          "+v"(P.x), "+v"(P.y), "+v"(X.x), "+v"(X.y), "+v"(Y.x), "+v"(Y.y));
#undef LRNNX_CSP
#undef LRNNX_CS
#undef LRNNX_ROW
}

__device__ __forceinline__ void swap_rows(float2 &a, float2 &b) { swap_rows(a.x, b.x); swap_rows(a.y, b.y); }

// Both scans of a state over the tile, in a row of lanes that holds its even pieces (E) and its odd ones (O): xc is the
// state entering the tile (lane 0 of the row, zero elsewhere), hc the adjoint entering it from the later side (lane 15).
// On return xE, xO are the states entering the pieces, gE, gO the adjoints entering them from the later side; the result is
// the adjoint leaving the tile on the earlier side (lane 0).
__device__ __forceinline__ float2 piece_scans(float2 PE, float2 SE, float2 QE, float2 PO, float2 SO, float2 QO, float2 xc,
                                              float2 hc, float2 &xE, float2 &xO, float2 &gE, float2 &gO) {
    const float2 P = cxmul(PE, PO);
    float2 S = cxfma(PO, SE, SO), Q = cxfma(PE, QO, QE);
    S = cxfma(P, xc, S);
    Q = cxfma(P, hc, Q);
    crow_scans(P, S, Q, xc, hc);
    xE = xc; gO = hc;
    xO = cxfma(PE, xE, SE);
    gE = cxfma(PO, gO, QO);
    return Q;
}

template <typename IO, int N, int DISC, bool HAS_Z>
__global__ __launch_bounds__(CBwdGeom<N>::NT, 2) void k_ss_cbwd(const CBwdParams p) {
    using CW = typename cword<IO>::type;
    using GE = CBwdGeom<N>;
    constexpr int W = GE::W, NS = GE::NS, NT = GE::NT, CP = GE::CP, TPT = GE::TPT, NTC = GE::NTC, NA = GE::NA, NB = GE::NB;
    constexpr bool OWN = GE::OWN, SPLIT = GE::SPLIT;
    constexpr int T = 8, TILE = kBwdTileSteps;
    // Two states side by side; the exact zero-order hold takes one after the other, since it also keeps the gains, and so does the
    // bilinear scheme with N = 2 in float32, which spills 61 registers with both and 36 with one (8 x 1536 rows, L = 2048: 386 and 315 us;
    // bfloat16: 251 and 256)
    constexpr bool PAIR = NS == 2 && DISC != DISC_ZOH && !(DISC == DISC_BILINEAR && N == 2 && sizeof(IO) == 4);
    static_assert(TILE == kCkptInterval && TILE == 32 * T, "a tile is one checkpoint interval and one half-wavefront");

    __shared__ __attribute__((aligned(16))) float sIn[NB][CP][GE::IN][TILE];
    __shared__ __attribute__((aligned(16))) float sPart[CP][W][3][OWN ? 4 : TILE];      // per wavefront: ypre, du, ddelta partials
    __shared__ __attribute__((aligned(16))) float2 sB[N * TILE], sC[N * TILE];          // maps of the tile, see map_at
    __shared__ __attribute__((aligned(16))) float2 sH[kMaxGc * N];      // a_{l0} K_{l0} carried to the earlier tile, per (channel, n)
    __shared__ __attribute__((aligned(16))) float2 sAC[NB][2][CP][N];   // A and the state entering the tile, of a pair
    __shared__ float2 sdA[kMaxGc * N];
    __shared__ float sdD[kMaxGc], sdb[kMaxGc], sDskip[kMaxGc], sBias[kMaxGc];
    __shared__ __attribute__((aligned(8))) float2 sZero;
    __shared__ int sDone;                            // wavefronts that have finished with the partial sums of a pass, all passes

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = w * NS;                           // this wavefront's first state
    int b = blockIdx.y;
    // packed variable-length mode (p.cu != nullptr, see seq_span): I/O rows have no batch stride, the maps and their gradients are
    // [G, p.L, N]
    int64_t L = p.L, toff = 0, bs = b;
    if (p.cu) {
        const SeqSpan q = seq_span(p.cu, p.B, p.L, b, p.ranked, p.order);           // the longest sequences start first
        b = q.b; toff = q.toff; L = q.L; bs = 0;
    }
    // Chunked launch: this workgroup walks chunk blockIdx.z of its rows only, i.e. the steps toff .. toff + L - 1 of
    // the time axis, starting from that chunk's carried adjoint.  Chunks are counted from the start of the sequence;
    // the last one takes whatever is left (see chunk_span in selective_bwd_carry.hip), and the workgroups of a packed
    // sequence that ends before their chunk leave here, all threads together and before any barrier (chunk 0 stays
    // even for an empty sequence: it writes that sequence's dx0).
    const int chunk = blockIdx.z;
    const int64_t slot0 = p.cu ? toff / TILE + b : (int64_t)b * p.part_tiles;    // first tile of this entry among all tiles
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
    int G = p.G;
    if (p.wcap > 0) {
        const int64_t fit = p.wcap / (ntiles > 0 ? ntiles : 1);
        G = fit < p.gmin ? p.gmin : (fit < G ? (int)fit & ~1 : G);       // (channels are walked in pairs)
    }
    const int blocks_per_grp = (p.dpg + G - 1) / G;
    if ((int)blockIdx.x >= p.bcg * blocks_per_grp) return;
    const int grp = blockIdx.x / blocks_per_grp;
    const int din0 = (blockIdx.x % blocks_per_grp) * G;
    const int d0 = grp * p.dpg + din0;
    const int Gact = (p.dpg - din0 < G) ? p.dpg - din0 : G;
    // checkpoints of this workgroup's rows: [B,D,nck,N], or packed [D,nslots,N] with sequence b at slot toff/interval + b
    const int64_t nck = p.cu ? p.nslots : (p.L + kCkptInterval - 1) / kCkptInterval;
    const int64_t ck0 = p.cu ? toff / kCkptInterval + b : toff / kCkptInterval;
    const float2 *ckrow = p.ckpt + (((p.cu ? (int64_t)d0 : (int64_t)b * p.D + d0) * nck) + ck0) * N;
    const bool vec = p.vec != 0;

    for (int i = tid; i < Gact * N; i += NT) {
        float2 h = make_float2(0.0f, 0.0f);
        if (p.nchunks > 1) { h = p.hc[(((int64_t)b * p.D + d0 + i / N) * p.nchunks + chunk) * N + i % N]; h.y = -h.y; }
        sH[i] = h; sdA[i] = make_float2(0.0f, 0.0f);
    }
    for (int i = tid; i < Gact; i += NT) {
        sdD[i] = 0.0f; sdb[i] = 0.0f;
        sDskip[i] = p.Dskip ? p.Dskip[d0 + i] : 0.0f;
        sBias[i] = p.bias ? p.bias[d0 + i] : 0.0f;
    }
    if (tid == 0) { sZero = make_float2(0.0f, 0.0f); sDone = 0; }
    [[maybe_unused]] int done = 0;                   // what sDone has to reach before the partial sums may be written again

    const int64_t bc0 = ((bs * p.bcg + grp) * p.L + toff) * N;       // first complex element of the maps of this sequence and group
    const CW *Bm = reinterpret_cast<const CW *>(p.Bm) + bc0;
    const CW *Cm = reinterpret_cast<const CW *>(p.Cm) + bc0;

    // prologue and epilogue: this thread's channel of a pair (wave-uniform where a channel takes whole wavefronts)
    const bool pro = !SPLIT || w < W / 2, epi = !SPLIT || w >= W / 2;
    int c_own = tid % NA / NTC;
    if constexpr (NTC >= 64) c_own = __builtin_amdgcn_readfirstlane(c_own);
    // The addresses that follow from the thread's number are formed where they are needed: hoisted out of the loops by the
    // compiler they would sit in registers all through the main pass, which has none to spare.
    auto fresh = [](unsigned v) { asm volatile("" : "+v"(v)); return v; };
    // first step of a thread in prologue and epilogue (a wavefront alone: the lane's own steps)
    auto first_step = [](unsigned t) {
        if constexpr (OWN) return (int)(((t & 15) * 2 + ((t >> 4) & 1)) * T);
        else return (int)(t % NTC) * TPT;
    };
    // two steps of a map in LDS: [n][step % 8 / 2][lane][step % 2], lanes permuted per block of four states against the
    // conflicts of the staging writes
    auto map_at = [](int n, int k, int l) { return ((n * 4 + k) * 32 + (l ^ ((n >> 2 & 3) << 1))) * 2; };

    for (int64_t tile = ntiles - 1; tile >= 0; --tile) {
        const int64_t l0 = tile * TILE;
        const int rem = (L - l0 < TILE) ? (int)(L - l0) : TILE;      // valid steps of this tile (at least one)
        const bool full = rem == TILE;
        __syncthreads();                             // the tables (first tile) are in place; the tile before is done with LDS

        // ---- both maps into LDS as fp32 pairs: two steps of up to four states a thread
        {
            constexpr int QN = N < 4 ? N : 4, PER = N / QN;
            const CW *BmT = Bm + l0 * N, *CmT = Cm + l0 * N;
#pragma unroll
            for (int it = 0; it < 128 * PER / NT; ++it) {
                const int t0 = (int)fresh(tid) + it * NT, pr = t0 / PER, q = t0 % PER;
                CW rB[2][QN], rC[2][QN];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int row = pr * 2 + j < rem ? pr * 2 + j : rem - 1;
                    load_cwords<CW, QN>(BmT + (unsigned)(row * N + q * QN), rB[j]);
                    load_cwords<CW, QN>(CmT + (unsigned)(row * N + q * QN), rC[j]);
                }
                const bool ok0 = pr * 2 < rem, ok1 = pr * 2 + 1 < rem;
#pragma unroll
                for (int s = 0; s < QN; ++s) {
                    const int at = map_at(q * QN + s, pr & 3, piece_lane(pr >> 2));
                    auto put = [&](float2 *m, CW w0, CW w1) {
                        const float2 v0 = cword<IO>::unpack(w0), v1 = cword<IO>::unpack(w1);
                        *reinterpret_cast<float4 *>(&m[at]) = make_float4(ok0 ? v0.x : 0.0f, ok0 ? v0.y : 0.0f, ok1 ? v1.x : 0.0f, ok1 ? v1.y : 0.0f);
                    };
                    put(sB, rB[0][s], rB[1][s]);
                    put(sC, rC[0][s], rC[1][s]);
                }
            }
        }

        // ---- per-step inputs of a pair of channels are fetched one pair ahead.  Row pointers: this thread's channel of
        // the pair the next fetch reads and the next epilogue writes (past the last channel they stay on a valid one).
        RawFew<IO, TPT> r_u, r_dl, r_dy, r_z;
        const int64_t tl = toff + l0;
        const int c_first = c_own < Gact ? c_own : Gact - 1;
        const int64_t dch = d0 + c_first;
        const IO *n_u = reinterpret_cast<const IO *>(p.u) + bs * p.u_sb + dch * p.u_sd + tl;
        const IO *n_dl = reinterpret_cast<const IO *>(p.delta) + bs * p.dl_sb + dch * p.dl_sd + tl;
        const IO *n_dy = reinterpret_cast<const IO *>(p.dy) + bs * p.dy_sb + dch * p.dy_sd + tl;
        const IO *n_z = HAS_Z ? reinterpret_cast<const IO *>(p.z) + bs * p.z_sb + dch * p.z_sd + tl : n_dy;
        const int64_t z_sd = HAS_Z ? p.z_sd : p.dy_sd;
        IO *o_du = reinterpret_cast<IO *>(p.du) + bs * p.du_sb + dch * p.du_sd + tl;
        IO *o_dd = reinterpret_cast<IO *>(p.ddelta) + bs * p.dd_sb + dch * p.dd_sd + tl;
        IO *o_dz = HAS_Z && p.dz ? reinterpret_cast<IO *>(p.dz) + bs * p.dz_sb + dch * p.dz_sd + tl : nullptr;
        int n_g = 0;                                                 // first channel of the pair of the next fetch
        // A and the checkpointed state of the pair: one value each for the first 2 * CP * N threads
        const float2 *n_A = p.A + (int64_t)d0 * N, *n_ck = ckrow + tile * N;
        const unsigned ck_sd = (unsigned)(nck * N);                  // elements between the checkpoints of two channels
        float2 r_ac = make_float2(0.0f, 0.0f);
        const bool window = vec && L >= TPT;                         // the last steps of the sequence: see tail_window
        auto fetch = [&](unsigned t0) {
            const int f0 = first_step(t0);
            if (window) {
                const int o = f0 < rem - TPT ? f0 : rem - TPT;       // (tail_window)
                load_few_raw<IO, TPT>(n_u + o, 0, TPT, true, r_u);
                load_few_raw<IO, TPT>(n_dl + o, 0, TPT, true, r_dl);
                load_few_raw<IO, TPT>(n_dy + o, 0, TPT, true, r_dy);
                if constexpr (HAS_Z) load_few_raw<IO, TPT>(n_z + o, 0, TPT, true, r_z);
            } else {
                load_few_raw<IO, TPT>(n_u, f0, rem, vec, r_u);
                load_few_raw<IO, TPT>(n_dl, f0, rem, vec, r_dl);
                load_few_raw<IO, TPT>(n_dy, f0, rem, vec, r_dy);
                if constexpr (HAS_Z) load_few_raw<IO, TPT>(n_z, f0, rem, vec, r_z);
            }
            if (t0 < 2 * CP * N) {
                const bool second = (t0 / N) % CP && n_g + 1 < Gact;     // else the first channel of the pair again
                const float2 *q = t0 < CP * N ? n_A : n_ck;
                r_ac = q[t0 % N + (second ? (t0 < CP * N ? (unsigned)N : ck_sd) : 0u)];
            }
            n_g += CP;
            if (n_g < Gact) { n_A += CP * N; n_ck += (int64_t)CP * ck_sd; }
            if (n_g + c_own < Gact) { n_u += CP * p.u_sd; n_dl += CP * p.dl_sd; n_dy += CP * p.dy_sd; n_z += CP * z_sd; }
        };
        if (pro) fetch(tid);

        float2 dB[NS][T], dC[NS][T];                 // this lane's sums of dBm* and dCm* over channels
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int t = 0; t < T; ++t) { dB[s][t] = make_float2(0.0f, 0.0f); dC[s][t] = make_float2(0.0f, 0.0f); }

        // kept from a pair's prologue to its epilogue: d softplus / ds and the factor that turns ypre into dz (in registers
        // where the same threads do both)
        float e_sg[TPT], e_zf[TPT], n_sg[TPT], n_zf[TPT];
        // ---- prologue of the pair whose inputs have been fetched: each thread prepares TPT steps of its channel
        auto step_inputs = [&](int ch, unsigned t0, float (&u)[TPT], float (&dl)[TPT], float (&dy)[TPT]) {
            const float bias = sBias[ch < Gact ? ch : Gact - 1];
            const int f0 = first_step(t0);
            float z[TPT];
            if (!full && window) {
                const int by = f0 - (f0 < rem - TPT ? f0 : rem - TPT);
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
                dl[i] = p.softplus ? sp : v;
                n_sg[i] = p.softplus ? sg : 1.0f;
                if constexpr (HAS_Z) gate_bwd(z[i], dy[i], n_zf[i]);
            }
            if (!full || ch >= Gact) {                   // steps past the end: Delta = 0 (a = 1), no input, no gradient
#pragma unroll
                for (int i = 0; i < TPT; ++i)
                    if (f0 + i >= rem || ch >= Gact) { dl[i] = 0.0f; u[i] = 0.0f; dy[i] = 0.0f; }
            }
        };
        auto prologue = [&](int ch, unsigned t0, int buf) {
            float u[TPT], dl[TPT], dy[TPT];
            step_inputs(ch, t0, u, dl, dy);
            const int slot = cstep_slot(first_step(t0));
            csteps_write<TPT>(sIn[buf][c_own][0], slot, dl);
            csteps_write<TPT>(sIn[buf][c_own][1], slot, u);
            csteps_write<TPT>(sIn[buf][c_own][2], slot, dy);
            if constexpr (SPLIT) {
                csteps_write<TPT>(sIn[buf][c_own][3], slot, n_sg);
                if constexpr (HAS_Z) csteps_write<TPT>(sIn[buf][c_own][4], slot, n_zf);
            }
            if (t0 < 2 * CP * N) (&sAC[buf][0][0][0])[t0] = r_ac;
        };
        auto rotate = [&]() {
            if constexpr (!SPLIT && !OWN) {
#pragma unroll
                for (int i = 0; i < TPT; ++i) { e_sg[i] = n_sg[i]; if constexpr (HAS_Z) e_zf[i] = n_zf[i]; }
            }
        };
        // ---- epilogue: du, ddelta, dz of this thread's steps from the sums over states
        auto finish = [&](const int g, unsigned t0, const float (&e_dl)[TPT], const float (&e_u)[TPT], const float (&e_dy)[TPT],
                          const float (&s_yp)[TPT], const float (&s_du)[TPT], const float (&s_dd)[TPT]) {
            const int ch = g + c_own, f0 = first_step(t0);
            const bool live = ch < Gact;
            const float Dsk = sDskip[live ? ch : Gact - 1];
            float o_u[TPT], o_d[TPT], o_z[TPT];
            float dD_part = 0.0f, db_part = 0.0f;
#pragma unroll
            for (int i = 0; i < TPT; ++i) {
                const float ed = e_dl[i], eu = e_u[i], ey = e_dy[i];
                float su = s_du[i], sd = s_dd[i];
                if constexpr (DISC == DISC_ZOH_S6) {
                    // the wavefronts' sums are sum_n Re(K B): dDelta += u times it, du = Delta times it
                    sd = __builtin_fmaf(eu, su, sd);
                    su *= ed;
                }
                o_u[i] = __builtin_fmaf(ey, Dsk, su);
                o_d[i] = sd * e_sg[i];
                if constexpr (HAS_Z) o_z[i] = __builtin_fmaf(Dsk, eu, s_yp[i]) * e_zf[i];
                dD_part = __builtin_fmaf(ey, eu, dD_part);
                db_part += (full || f0 + i < rem) ? o_d[i] : 0.0f;
            }
            if (live) {
                store_few<IO, TPT>(o_du, f0, rem, vec, o_u);
                store_few<IO, TPT>(o_dd, f0, rem, vec, o_d);
                if constexpr (HAS_Z) { if (o_dz) store_few<IO, TPT>(o_dz, f0, rem, vec, o_z); }
            }
            {
                // joint reduction of the two per-lane sums over a row of lanes
                const bool odd = t0 & 1;
                float v = odd ? db_part : dD_part;
                v += dpp<0xB1>(0.0f, odd ? dD_part : db_part);           // quad_perm [1,0,3,2]
                v += dpp<0x4E>(0.0f, v);                                  // quad_perm [2,3,0,1]
                v += dpp<0x124>(0.0f, v);                                 // row_ror:4
                v += dpp<0x128>(0.0f, v);                                 // row_ror:8
                if ((t0 & 15) < 2 && live) lds_add(&(odd ? sdb : sdD)[ch], v);
            }
            o_du += CP * p.du_sd; o_dd += CP * p.dd_sd;
            if constexpr (HAS_Z) { if (o_dz) o_dz += CP * p.dz_sd; }
        };
        auto epilogue = [&](const int g, const int buf) {
            const unsigned t0 = fresh(tid % NA);
            const int slot = cstep_slot(first_step(t0));
            float e_in[3][TPT], s_yp[TPT], s_du[TPT], s_dd[TPT];
#pragma unroll
            for (int j = 0; j < 3; ++j) csteps_read<TPT>(sIn[buf][c_own][j], slot, e_in[j]);
            if constexpr (SPLIT) {
                csteps_read<TPT>(sIn[buf][c_own][3], slot, e_sg);
                if constexpr (HAS_Z) csteps_read<TPT>(sIn[buf][c_own][4], slot, e_zf);
            }
#pragma unroll
            for (int i = 0; i < TPT; ++i) { s_yp[i] = 0.0f; s_du[i] = 0.0f; s_dd[i] = 0.0f; }
#pragma unroll
            for (int ww = 0; ww < W; ++ww) {
                float v[TPT];
                if constexpr (HAS_Z) {
                    csteps_read<TPT>(sPart[c_own][ww][0], slot, v);
#pragma unroll
                    for (int i = 0; i < TPT; ++i) s_yp[i] = ww ? s_yp[i] + v[i] : v[i];
                }
                csteps_read<TPT>(sPart[c_own][ww][1], slot, v);
#pragma unroll
                for (int i = 0; i < TPT; ++i) s_du[i] = ww ? s_du[i] + v[i] : v[i];
                csteps_read<TPT>(sPart[c_own][ww][2], slot, v);
#pragma unroll
                for (int i = 0; i < TPT; ++i) s_dd[i] = ww ? s_dd[i] + v[i] : v[i];
            }
            finish(g, t0, e_in[0], e_in[1], e_in[2], s_yp, s_du, s_dd);
        };

        // ---- main: this lane's 8 steps of its channel for the wavefront's states
        auto states = [&](const int g, const int buf, const unsigned ln, const float (&dl)[T], float (&du)[T], const float (&dy)[T],
                          float (&yp)[T], float (&pu)[T], float (&pd)[T]) {
            const unsigned c = ln >> 5, li = ln & 15, row = ln >> 4 & 1;
            const int ch = g + (int)c < Gact ? g + (int)c : g;             // (the half past the last channel repeats the first, unused)
            const bool own = g + (int)c < Gact;
            const int at = ch * N + n0;
            if constexpr (DISC == DISC_ZOH_S6) {
#pragma unroll
                for (int t = 0; t < T; ++t) du[t] *= dl[t];      // S6 only ever needs Delta*u; the others keep u
            }
            float sum_dl = dl[0];
#pragma unroll
            for (int t = 1; t < T; ++t) sum_dl += dl[t];
            auto maps = [&](const float2 *m, int s, float2 (&v)[T]) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 f = *reinterpret_cast<const float4 *>(m + map_at(n0 + s, k, ln & 31));
                    v[2 * k] = make_float2(f.x, f.y); v[2 * k + 1] = make_float2(f.z, f.w);
                }
            };
            // the lane's steps as one affine pair each way: S the end state from zero, Q = a_0 (c_0 + a_1 (c_1 + ...)) the
            // adjoint handed on, both with multiplier P
            // (bilinear: hd holds q, from which multiplier and gain follow, see cbilinear_q)
            auto mult = [](float2 h) { if constexpr (DISC == DISC_BILINEAR) return cbilinear_a(h); else return h; };
            auto fold = [&](int s, float2 (&hd)[T], float2 (&x)[T], float2 (&gg)[T], float2 &P, float2 &S, float2 &Q) {
                const float2 Av = sAC[buf][0][c][n0 + s];
                const CCoef cc = make_ccoef(Av.x, Av.y);
                float2 Bv[T], Cv[T], a[T];
                maps(sB, s, Bv);
                maps(sC, s, Cv);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if constexpr (DISC == DISC_BILINEAR) {
                        hd[t] = cbilinear_q(dl[t], cc);
                        gg[t] = make_float2(dl[t] * hd[t].x, dl[t] * hd[t].y);
                    } else cdisc_ag<DISC>(dl[t], cc, hd[t], gg[t]);
                    a[t] = mult(hd[t]);
                    if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) x[t] = make_float2(du[t] * Bv[t].x, du[t] * Bv[t].y);
                    else x[t] = cxmul(make_float2(gg[t].x * du[t], gg[t].y * du[t]), Bv[t]);
                }
                if constexpr (DISC != DISC_BILINEAR) P = cexp_dt(sum_dl, cc.A2r, cc.Arev);       // product of the T multipliers
                fast_part();
                S = x[0];
#pragma unroll
                for (int t = 1; t < T; ++t) S = cxfma(a[t], S, x[t]);
                Q = cxmul(a[T - 1], make_float2(Cv[T - 1].x * dy[T - 1], Cv[T - 1].y * dy[T - 1]));
#pragma unroll
                for (int t = T - 2; t >= 0; --t)
                    Q = cxmul(a[t], make_float2(__builtin_fmaf(Cv[t].x, dy[t], Q.x), __builtin_fmaf(Cv[t].y, dy[t], Q.y)));
                if constexpr (DISC == DISC_BILINEAR)
                    P = cxmul(cxmul(cxmul(a[0], a[1]), cxmul(a[2], a[3])), cxmul(cxmul(a[4], a[5]), cxmul(a[6], a[7])));
                if constexpr (DISC == DISC_BILINEAR) {   // (there are no registers to keep the multipliers beside q)
#pragma unroll
                    for (int t = 0; t < T; ++t) asm volatile("" : "+v"(hd[t].x), "+v"(hd[t].y));
                }
            };
            float2 dA[NS];
            // the states (earliest step first), then the adjoint (last step first) with all that is summed over it
            auto replay = [&](int s, const float2 (&hd)[T], float2 (&x)[T], const float2 (&gg)[T], const float2 xin, float2 Gin) {
                const float2 Av = sAC[buf][0][c][n0 + s];
                float2 Bv[T], Cv[T];
                maps(sC, s, Cv);
                maps(sB, s, Bv);
                {
                    float2 xp = xin;
#pragma unroll
                    for (int t = 0; t < T; ++t) { xp = cxfma(mult(hd[t]), xp, x[t]); x[t] = xp; }
                }
                float2 dAp = make_float2(0.0f, 0.0f);
                auto acc = [&](float &sum, float m1, float m2) { sum = (s == 0) ? m1 * m2 : __builtin_fmaf(m1, m2, sum); };
#pragma unroll
                for (int t = T - 1; t >= 0; --t) {
                    const float2 xprev = t > 0 ? x[t - 1] : xin;
                    const float2 K = make_float2(__builtin_fmaf(Cv[t].x, dy[t], Gin.x), __builtin_fmaf(Cv[t].y, dy[t], Gin.y));
                    [[maybe_unused]] float2 qK;                          // bilinear: q K; a K = 2 q K - K
                    if constexpr (DISC == DISC_BILINEAR) {
                        qK = cxmul(hd[t], K);
                        Gin = make_float2(__builtin_fmaf(2.0f, qK.x, -K.x), __builtin_fmaf(2.0f, qK.y, -K.y));
                    } else Gin = cxmul(hd[t], K);
                    dC[s][t] = make_float2(__builtin_fmaf(dy[t], x[t].x, dC[s][t].x), __builtin_fmaf(dy[t], x[t].y, dC[s][t].y));
                    if constexpr (HAS_Z) {
                        acc(yp[t], Cv[t].x, x[t].x);
                        yp[t] = __builtin_fmaf(-Cv[t].y, x[t].y, yp[t]);
                    }
                    if constexpr (DISC == DISC_ZOH_S6 || DISC == DISC_DIRAC) {
                        // S6: g = Delta (du and dDelta share sum_n Re(K B), scaled in the epilogue); dirac: g = 1
                        acc(pu[t], K.x, Bv[t].x);
                        pu[t] = __builtin_fmaf(-K.y, Bv[t].y, pu[t]);
                        dB[s][t] = make_float2(__builtin_fmaf(K.x, du[t], dB[s][t].x), __builtin_fmaf(K.y, du[t], dB[s][t].y));
                        const float2 q = cxmul(Gin, xprev);              // grad a* a; da/dDelta = A a, da/dA = Delta a
                        acc(pd[t], q.x, Av.x);
                        pd[t] = __builtin_fmaf(-q.y, Av.y, pd[t]);
                        dAp = make_float2(__builtin_fmaf(q.x, dl[t], dAp.x), __builtin_fmaf(q.y, dl[t], dAp.y));
                    } else if constexpr (DISC == DISC_ZOH) {
                        // da/dDelta = A a, da/dA = Delta a, dg/dDelta = a
                        const float2 hb = cxmul(K, Bv[t]);
                        const float2 gq = make_float2(hb.x * du[t], hb.y * du[t]);             // grad g*
                        const CCoef cc = make_ccoef(Av.x, Av.y);
                        const float2 a = hd[t], g = gg[t], g_A = czoh_gain_dA(dl[t], cc, a, g);
                        const float2 q = cxmul(Gin, xprev);
                        acc(pd[t], q.x, Av.x);
                        pd[t] = __builtin_fmaf(-q.y, Av.y, pd[t]);
                        pd[t] = __builtin_fmaf(gq.x, a.x, __builtin_fmaf(-gq.y, a.y, pd[t]));
                        dAp = cxfma(gq, g_A, make_float2(__builtin_fmaf(q.x, dl[t], dAp.x), __builtin_fmaf(q.y, dl[t], dAp.y)));
                        acc(pu[t], hb.x, g.x);
                        pu[t] = __builtin_fmaf(-hb.y, g.y, pu[t]);
                        const float2 kg = cxmul(K, g);
                        dB[s][t] = make_float2(__builtin_fmaf(kg.x, du[t], dB[s][t].x), __builtin_fmaf(kg.y, du[t], dB[s][t].y));
                    } else {
                        // bilinear: g = Delta q, and all four partials are multiples of q^2: da/dDelta = A q^2, da/dA = Delta q^2,
                        // dg/dDelta = q^2, dg/dA = Delta^2 q^2 / 2.  One factor q sits in q K (twelve instructions less than q^2 apart:
                        // 8 x 1536 rows, L = 2048, bf16, N = 16 945 -> 895 us, N = 4 306 -> 291).
                        const float2 q = hd[t], qB = cxmul(qK, Bv[t]), ga = cxmul(qK, xprev);
                        const float2 gq = make_float2(qB.x * du[t], qB.y * du[t]);
                        float dt = dl[t];
                        if constexpr (N == 2) asm volatile("" : "+v"(dt));       // (its products are not kept for the other state: no registers)
                        const float gd = dt * du[t];
                        acc(pu[t], dt, qB.x);
                        dB[s][t] = make_float2(__builtin_fmaf(qK.x, gd, dB[s][t].x), __builtin_fmaf(qK.y, gd, dB[s][t].y));
                        const float2 t1 = cxfma(ga, Av, gq);
                        acc(pd[t], t1.x, q.x);
                        pd[t] = __builtin_fmaf(-t1.y, q.y, pd[t]);
                        const float h = 0.5f * dt;
                        const float2 t2 = make_float2(__builtin_fmaf(gq.x, h, ga.x) * dt, __builtin_fmaf(gq.y, h, ga.y) * dt);
                        dAp = cxfma(t2, q, dAp);
                    }
                    // computed here: left to itself the compiler moves the products of one state down to the sums of the
                    // next one's, and spills what it then has to keep
                    if constexpr (HAS_Z) asm volatile("" : "+v"(yp[t]));
                    asm volatile("" : "+v"(dC[s][t].x), "+v"(dC[s][t].y), "+v"(dB[s][t].x), "+v"(dB[s][t].y), "+v"(pu[t]), "+v"(pd[t]),
                                      "+v"(dAp.x), "+v"(dAp.y));
                }
                dA[s] = dAp;
            };
            const bool first = li == 0, last = li == 15;
            if constexpr (PAIR) {
                float2 a[2][T], x[2][T], gg[T], P[2], S[2], Q[2], xin[2], Gin[2];
                slow_part();
                fold(0, a[0], x[0], gg, P[0], S[0], Q[0]);
                slow_part();
                fold(1, a[1], x[1], gg, P[1], S[1], Q[1]);
                // row 0 takes both pieces of state 0, row 1 those of state 1
                const float2 xc = *(first ? &sAC[buf][1][c][n0 + row] : &sZero), hc = *(last ? &sH[at + row] : &sZero);
                slow_part();
                swap_rows(P[0], P[1]); swap_rows(S[0], S[1]); swap_rows(Q[0], Q[1]);
                const float2 out = piece_scans(P[0], S[0], Q[0], P[1], S[1], Q[1], xc, hc, xin[0], xin[1], Gin[0], Gin[1]);
                swap_rows(xin[0], xin[1]); swap_rows(Gin[0], Gin[1]);
                if (own && first) sH[at + row] = out;            // carried to the earlier tile
                fast_part();
                replay(0, a[0], x[0], gg, xin[0], Gin[0]);
                __builtin_amdgcn_sched_barrier(0);
                replay(1, a[1], x[1], gg, xin[1], Gin[1]);
                slow_part();
            } else {
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    float2 a[T], x[T], gg[T], P, S, Q, xE, xO, gE, gO;
                    fold(s, a, x, gg, P, S, Q);
                    // (both rows hold the same)
                    const float2 xc = *(first ? &sAC[buf][1][c][n0 + s] : &sZero), hc = *(last ? &sH[at + s] : &sZero);
                    float2 P1 = P, S1 = S, Q1 = Q;
                    swap_rows(P, P1); swap_rows(S, S1); swap_rows(Q, Q1);
                    const float2 out = piece_scans(P, S, Q, P1, S1, Q1, xc, hc, xE, xO, gE, gO);
                    if (own && first && row == 0) sH[at + s] = out;
                    const float2 xin = make_float2(row ? xO.x : xE.x, row ? xO.y : xE.y), Gin = make_float2(row ? gO.x : gE.x, row ? gO.y : gE.y);
                    replay(s, a, x, gg, xin, Gin);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // dA over the 16 lanes of a row.  With two states two exchange steps leave each lane of a quad with the quad's sum of
            // ONE of the four values (lane % 4 = 0, 1, 2, 3: value 0, 2, 1, 3), two rotations sum the quads
            float *sum = reinterpret_cast<float *>(&sdA[at]);
            if constexpr (NS == 2) {
                const float v4[4] = {dA[0].x, dA[0].y, dA[1].x, dA[1].y};
                const bool b0 = ln & 1, b1 = ln & 2;
                float kA = b0 ? v4[2] : v4[0], kB = b0 ? v4[3] : v4[1];
                kA += dpp<0xB1>(0.0f, b0 ? v4[0] : v4[2]);           // quad_perm [1,0,3,2]
                kB += dpp<0xB1>(0.0f, b0 ? v4[1] : v4[3]);
                float v = b1 ? kB : kA;
                v += dpp<0x4E>(0.0f, b1 ? kA : kB);                  // quad_perm [2,3,0,1]
                v += dpp<0x124>(0.0f, v);                            // row_ror:4
                v += dpp<0x128>(0.0f, v);                            // row_ror:8
                if (own && li < 4) lds_add(sum + ((ln & 1) << 1) + ((ln >> 1) & 1), v);
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    float v = j ? dA[0].y : dA[0].x;
                    v += dpp<0xB1>(0.0f, v);
                    v += dpp<0x4E>(0.0f, v);
                    v += dpp<0x124>(0.0f, v);
                    v += dpp<0x128>(0.0f, v);
                    if (own && li == 0) lds_add(sum + j, v);
                }
            }
        };
        if constexpr (OWN) {
            __syncthreads();                             // (one wavefront: orders the LDS accesses only)
            for (int g = 0; g < Gact; g += CP) {
                const unsigned t0 = fresh(tid);
                const int c = t0 >> 5, l4 = lane_slot(t0 & 31);
                float u[T], dl[T], dy[T], yp[T], pu[T], pd[T];
                step_inputs(g + c_own, t0, u, dl, dy);
                csteps_write<T>(sIn[0][c][0], l4, u);
                csteps_write<T>(sIn[0][c][1], l4, n_sg);
                if constexpr (HAS_Z) csteps_write<T>(sIn[0][c][2], l4, n_zf);
                if (t0 < 2 * CP * N) (&sAC[0][0][0][0])[t0] = r_ac;
                fetch(t0);
                __syncthreads();
                states(g, 0, t0, dl, u, dy, yp, pu, pd);
                csteps_read<T>(sIn[0][c][0], l4, u);
                csteps_read<T>(sIn[0][c][1], l4, e_sg);
                if constexpr (HAS_Z) csteps_read<T>(sIn[0][c][2], l4, e_zf);
                finish(g, t0, dl, u, dy, yp, pu, pd);
                __syncthreads();
            }
        } else {
            // Between two barriers a wavefront finishes the pair before (its partial sums are complete), runs the main part
            // of this pair and prepares the next one.  There is one set of partial sums: before a wavefront writes its own it
            // sees to it that those who read the pair before are through, which they have been for nearly a whole pass
            // (they count themselves in sDone on their way, and wait for nobody before that).
            auto main_part = [&](const int g, const int buf) {
                const unsigned ln = fresh(lane), c = ln >> 5;
                const int l4 = lane_slot(ln & 31);
                float dl[T], du[T], dy[T], yp[T], pu[T], pd[T];
                csteps_read<T>(sIn[buf][c][0], l4, dl);
                csteps_read<T>(sIn[buf][c][1], l4, du);
                csteps_read<T>(sIn[buf][c][2], l4, dy);
                states(g, buf, ln, dl, du, dy, yp, pu, pd);
                fast_part();
                if constexpr (NB == 2) {
                    asm volatile("" ::: "memory");
                    while (__hip_atomic_load(&sDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < done) {}
                    asm volatile("" ::: "memory");
                }
                edge_part();
                if constexpr (HAS_Z) csteps_write<T>(sPart[c][w][0], l4, yp);
                csteps_write<T>(sPart[c][w][1], l4, pu);
                csteps_write<T>(sPart[c][w][2], l4, pd);
            };
            auto next_inputs = [&](const int g, const int buf) {          // (past the last pair: unused)
                if (!pro) return;
                const unsigned t0 = fresh(tid);
                prologue(g + c_own, t0, buf);
                fetch(t0);
            };
            next_inputs(0, 0);
            if constexpr (NB == 2) {
                int g = 0, buf = 0;
                for (; g < Gact; g += CP, buf ^= 1) {
                    __syncthreads();
                    if (g > 0) {
                        if (epi) {
                            epilogue(g - CP, buf ^ 1);
                            asm volatile("" ::: "memory");
                            if (lane == 0) (void)__hip_atomic_fetch_add(&sDone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                        done += SPLIT ? W / 2 : W;
                    }
                    rotate();
                    main_part(g, buf);
                    next_inputs(g + CP, buf ^ 1);
                }
                __syncthreads();
                if (epi) epilogue(g - CP, buf ^ 1);
            } else {
                for (int g = 0; g < Gact; g += CP) {
                    __syncthreads();
                    rotate();
                    main_part(g, 0);
                    __syncthreads();
                    epilogue(g, 0);
                    next_inputs(g + CP, 0);
                }
            }
        }

        // ---- the tile's sums of dBm and dCm over this workgroup's channels
        // (the two halves hold different channels: summed by a swap that leaves the lower half with steps 0-3 of a lane, the
        // upper half with steps 4-7)
        const unsigned t0 = fresh(tid), q0 = ((t0 & 15) * 2 + (t0 >> 4 & 1)) * 2 + (t0 >> 5 & 1);      // four steps from step 4 q0 on
        auto halves = [&](float v, float v4) {
            const auto r = __builtin_amdgcn_permlane32_swap((unsigned)f2i(v), (unsigned)f2i(v4), false, false);
            return make_float2(i2f((int)r[0]), i2f((int)r[1]));
        };
        auto sums = [&](const float2 (&o)[T], int j) {                   // the sums' real (j = 0) and imaginary parts: conjugated back
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2 h = j ? halves(o[t].y, o[t + 4].y) : halves(o[t].x, o[t + 4].x);
                v[t] = j ? -h.x - h.y : h.x + h.y;
            }
            return make_float4(v[0], v[1], v[2], v[3]);
        };
        if (p.part) {
            // to this workgroup's own slot of the workspace; the sum over workgroups and the transposition to [L,N] are those of
            // the real backward pass with twice the states (k_ss_bwd_maps), so the slot is laid out as its kernel does
            float *pt = p.part + (((slot0 + tile_first + tile) * gridDim.x + blockIdx.x) * 4 * N + 2 * n0) * TILE + ((q0 & 1) << 7) + ((q0 >> 1) << 2);
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    *reinterpret_cast<float4 *>(pt + (2 * s + j) * TILE) = sums(dB[s], j);
                    *reinterpret_cast<float4 *>(pt + (2 * N + 2 * s + j) * TILE) = sums(dC[s], j);
                }
        } else {
            // without a workspace: float atomics, on consecutive addresses (the sums change their order in the maps' place; four
            // steps are a piece, whose place in a plane of the part is permuted against conflicts)
            float *bB = reinterpret_cast<float *>(sB), *bC = reinterpret_cast<float *>(sC);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int e = (n0 + s) * 2 + j, at = e * TILE + (q0 ^ (e & 15)) * 4;
                    *reinterpret_cast<float4 *>(bB + at) = sums(dB[s], j);
                    *reinterpret_cast<float4 *>(bC + at) = sums(dC[s], j);
                }
            __syncthreads();
            float *gB = reinterpret_cast<float *>(p.dBm + bc0 + l0 * N), *gC = reinterpret_cast<float *>(p.dCm + bc0 + l0 * N);
#pragma unroll 1
            for (int i = t0; i < rem * 2 * N; i += NT) {
                const int e = i % (2 * N), l = i / (2 * N), at = e * TILE + ((l >> 2) ^ (e & 15)) * 4 + (l & 3);
                unsafeAtomicAdd(gB + i, bB[at]);
                unsafeAtomicAdd(gC + i, bC[at]);
            }
        }
    }
    __syncthreads();
    // ---- per-channel results of this workgroup
    // (the parameters read again: held in scalar registers all through the kernel they would push others out)
    typedef const __attribute__((address_space(4))) CBwdParams KernArgs;
    KernArgs *args = (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    KernArgs &q = *args;
    const bool own = q.rows.sb >= 0;                 // see RowSums
    float *oA = reinterpret_cast<float *>(q.dA), *oD = q.dD, *ob = q.dbias;
    if (own) {
        const int64_t at = b * q.rows.sb;
        oA = q.rows.A + at; oD = oD ? q.rows.D + at : oD; ob = ob ? q.rows.b + at : ob;
    }
    auto leave = [&](float *at, float v) { if (own) *at = v; else unsafeAtomicAdd(at, v); };
    for (int i = tid; i < Gact * N; i += NT) {
        float *dst = oA + 2 * ((int64_t)d0 * N + i);
        leave(dst, sdA[i].x);
        leave(dst + 1, -sdA[i].y);
        if (q.dx0 && chunk == 0) q.dx0[((int64_t)b * q.D + d0) * N + i] = make_float2(sH[i].x, -sH[i].y);
    }
    for (int g = tid; g < Gact; g += NT) {
        if (oD) leave(oD + d0 + g, sdD[g]);
        if (ob) leave(ob + d0 + g, sdb[g]);
    }
}

// ---------------------------------------------------------------- launchers
template <typename IO, int N, int DISC>
static hipError_t launch_cbwd_n(const CBwdParams &p, hipStream_t s) {
    const dim3 grid(cbwd_grid_x(p), p.B, p.nchunks > 1 ? p.nchunks : 1), block(CBwdGeom<N>::NT);
    if (p.z) hipLaunchKernelGGL((k_ss_cbwd<IO, N, DISC, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((k_ss_cbwd<IO, N, DISC, false>), grid, block, 0, s, p);
    if (p.part) {
        BwdParams m{};
        m.B = p.B; m.D = p.D; m.N = 2 * N; m.L = p.L; m.G = p.G; m.bcg = p.bcg; m.dpg = p.dpg; m.cu = p.cu; m.nslots = p.nslots;
        m.dBm = reinterpret_cast<float *>(p.dBm); m.dCm = reinterpret_cast<float *>(p.dCm);
        m.wcap = p.wcap; m.gmin = p.gmin; m.part = p.part; m.part_tiles = p.part_tiles;
        m.rows = p.rows; m.dA = reinterpret_cast<float *>(p.dA); m.dD = p.dD; m.dbias = p.dbias;
        return launch_bwd_maps(m, (int)grid.x, s);
    }
    return hipGetLastError();
}

template <typename IO, int DISC>
static hipError_t launch_cbwd_disc(const CBwdParams &p, hipStream_t s) {
    switch (p.N) {
        case 1: return launch_cbwd_n<IO, 1, DISC>(p, s);
        case 2: return launch_cbwd_n<IO, 2, DISC>(p, s);
        case 4: return launch_cbwd_n<IO, 4, DISC>(p, s);
        case 8: return launch_cbwd_n<IO, 8, DISC>(p, s);
        case 16: return launch_cbwd_n<IO, 16, DISC>(p, s);
    }
    return hipErrorInvalidValue;
}

template <typename IO>
static hipError_t launch_cbwd_io(const CBwdParams &p, int disc, hipStream_t s) {
    switch (disc) {
        case DISC_ZOH_S6: return launch_cbwd_disc<IO, DISC_ZOH_S6>(p, s);
        case DISC_ZOH: return launch_cbwd_disc<IO, DISC_ZOH>(p, s);
        case DISC_BILINEAR: return launch_cbwd_disc<IO, DISC_BILINEAR>(p, s);
        case DISC_DIRAC: return launch_cbwd_disc<IO, DISC_DIRAC>(p, s);
    }
    return hipErrorInvalidValue;
}

// float32 and bfloat16 are compiled side by side: selective_cplx_bwd_f32.hip includes this file for the former.
hipError_t launch_ss_cbwd_f32(const CBwdParams &p, int disc, hipStream_t s);
#ifdef LRNNX_CBWD_F32
hipError_t launch_ss_cbwd_f32(const CBwdParams &p, int disc, hipStream_t s) { return launch_cbwd_io<float>(p, disc, s); }
#else
hipError_t launch_ss_cbwd(const CBwdParams &p, int io_dtype, int disc, hipStream_t s) {
    if (p.G > kMaxGc) return hipErrorInvalidValue;         // (more channels than the tables in LDS hold)
    return io_dtype == 1 ? launch_cbwd_io<bf16_t>(p, disc, s) : launch_ss_cbwd_f32(p, disc, s);
}

// Workgroups the chip holds at once: two wavefronts per SIMD are what the registers allow.
int cbwd_places(int N) { return 2048 / (N >= 2 ? N / 2 : 1); }

// channels per workgroup: as many as fit when every place of the chip has one, since the staging of the maps and the flush
// of dBm/dCm are paid once per (workgroup, tile)
int cbwd_channels_per_group(int B, int D, int N, bool balanced) {
    const int64_t full = cbwd_places(N);
    // packed sequences of unknown lengths: four times as many workgroups, so that the short ones fill in beside the long
    int64_t G = ((int64_t)B * D) / (balanced ? full : 4 * full);
    if (balanced) {
        // never a few workgroups more than a whole number of rounds (see channels_for in selective_bwd.hip)
        int64_t rounds = 1;
        while ((int64_t)B * ((D + kMaxGc - 1) / kMaxGc) > rounds * full && rounds < 64) ++rounds;
        const int64_t nb = rounds * full / B;
        if (nb >= 1) G = (D + nb - 1) / nb;
    }
    if (G < 8) G = 8;
    if (G > kMaxGc) G = kMaxGc;
    if (G > D) G = D;
    const int64_t groups = (D + G - 1) / G;
    G = (D + groups - 1) / groups;                     // even split
    return (int)(G + 1) / 2 * 2;                       // (walked in pairs)
}
void cbwd_packed_shape(int B, int D, int bcg, int N, int64_t L, int64_t max_seqlen, int *G, int *wcap, int *gmin) {
    packed_shape(B, D, D / bcg, L, max_seqlen, cbwd_channels_per_group(B * bcg, D / bcg, N, true), kMaxGc, 1.3, cbwd_places(N), G, wcap, gmin);
}

// Whether the tile sums of dBm and dCm, which take `bytes`, go through the workspace and a second launch instead of float atomics.
// Many small workgroups meet at the same addresses (2 x 771 rows, L = 1531, N = 16, bf16: 181 us with atomics, 162 through
// the workspace; 4 x 1024 rows in 4 groups, L = 1000: 218 and 205); rows of one tile are done before a second launch could start
// (64 x 512, L = 100, N = 4: 90 and 97; 4 x 1024, L = 256, N = 8: 50 and 55), and so are small calls altogether (512 rows, L = 512,
// N = 4: 45 and 48).  With one or two states there are more workgroups, and their atomics cost more.
bool cbwd_sums_pay(int N, int64_t tiles, bool packed, size_t bytes) {
    return bytes > ((size_t)4 << 20) && (packed || tiles > 1 || N < 4);
}
int cbwd_grid_x(const CBwdParams &p) {
    const int gmin = p.wcap > 0 ? p.gmin : p.G;                       // fewest channels a workgroup may take
    return p.bcg * ((p.dpg + gmin - 1) / gmin);
}

// launch shape incl. the chunked path for few rows and long sequences (selective_bwd_carry.hip)
BwdPlan cbwd_plan(int rowsg, int dpg, int N, int64_t L, int mode, bool balanced) {
    const int G = cbwd_channels_per_group(rowsg, dpg, N, balanced);
    BwdPlan pl = plan_time_chunks(rowsg, dpg, L, balanced ? mode : 1, G, cbwd_places(N), kMaxGc);
    pl.G = (pl.G + 1) / 2 * 2;
    return pl;
}
#endif

}  // namespace lrnnx
