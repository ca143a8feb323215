// attn_bwd_mfma.hip -- backward of the squared-error JAB loss through causal GQA attention
// for the 16-bit dtypes at head_dim 64 and 128: the dK/dV and dQ kernels with their
// operand tiles streamed into LDS by DMA.
//
// Paper: Method, "Joint fine-tuning through the quantizer" and the Appendix on its design
// decisions, (1) / eq. lsq: the gradient of the attention-output loss of eq. joint_loss
// reaches the weights through Q, K and V.  With G = a_hat - a_ref, P the causal softmax
// (recomputed from the forward's log-sum-exp), D_i = sum_c G_ic a_hat_ic:
//   dV_j = sum_i P_ij G_i   (summed over the query heads of a kv group)
//   dS_ij = P_ij (G_i . V_j - D_i)
//   dQ_i = sum_j dS_ij K_j / sqrt(dh),   dK_j = sum_i dS_ij Q_i / sqrt(dh)
//
// gfx950 design (no atomics, fixed summation order => deterministic)
//  * Operand tiles are 32 rows of Q, G (dK/dV) or K, V (dQ) in their row-major form, DMA'd
//    (global_load_lds_dwordx4) into a ring of LDS stages with one barrier per tile.  The
//    products that contract over tokens need the tiles transposed (G^T, Q^T, K^T): those
//    operands come from the same row-major tiles through transposed LDS reads
//    (ds_read_b64_tr_b16), so no transposed copy exists in memory or in LDS.
//  * Tiles are stored quad-major (TileLayout): 16-byte chunks in groups of four per row,
//    each group of 32 rows contiguous, the chunk inside a group rotated by row / 4.  Both
//    access patterns are then free of bank conflicts (16 rows reading one logical chunk;
//    4 consecutive rows reading 4 consecutive chunks), and every fragment of a wave is its
//    lane's base address plus a constant offset.
//  * dK/dV: a wave owns 32 keys of one kv head with K and V in registers as B operands and walks
//    32-query tiles of the group's query heads from the last tile down to its diagonal.  S = Q K^T
//    and dP = G V^T come out with one key per lane; P and dS go from registers into the B operand of
//    dV^T += G^T P and dK^T += Q^T dS.  With room for it in the workspace, each 32 x 32 dS tile is
//    also stored as that operand (2 KiB).  Two forms (run_bwd_dma_kl says where each is taken):
//    - attn_bwd_dkdv_pipe_kernel: one 128-, 64- or 32-key block per workgroup, the waves of a key
//      slice taking turns at its tiles, and in a wave the scores of one tile beside the softmax of the
//      one before; for grids that do not fill the chip twice, and the KL term at head_dim 128.
//    - attn_bwd_dkdv_dma_kernel: a workgroup takes the 128-key blocks p and nkb - 1 - p (the same
//      number of tiles for all), tile after tile, two workgroups per CU.
//    What bounds the paired form once the chip is full is not one unit (16 x 2048 tokens, head_dim 128, counters
//    of the launch): matrix cores 45 % busy, the LDS data path 29 % of its cycles, no bank conflicts, each
//    wave at a wait for 47 % of its time, two waves per SIMD.  Either form takes 1.2 us for four waves' tile.
//  * dQ from the stored dS: a wave owns 32 queries of one query head; the workgroup's waves
//    share a kv head and walk its 32-key tiles, each wave's dS tiles riding the same LDS ring
//    and read transposed into the B operand of dQ^T += K^T dS^T (5 products in all).
//  * dQ recomputing dS (no stored dS): a wave owns 32 queries of one query head (Q and G in
//    registers as B operands); the workgroup's waves share a kv head and walk its 32-key
//    tiles.  S^T = K Q^T and dP^T = V G^T come out with one query per lane, so lse and D are
//    per-lane scalars, and dQ^T += K^T dS^T (7 products in all).
//  * Rows past the sequence are read at the sequence's last row (finite values) and
//    removed by the masks; the results are written transposed, dY^T [R][tokens], the
//    operand layout of the weight-gradient GEMM.
#include "device_common.h"
#include "kernels.h"
#include "lds_pipe.h"

namespace jab {
namespace {

// Quad-major tile layout: chunk c (16 bytes) of row r of a 32-row tile is stored at chunk slot
//   (c / 4) * 128 + 4 r + ((c % 4) ^ ((r / 4) % 4)).
// Row reads (16 rows, one logical chunk) land on 16 distinct 16-byte bank slots: 4 (r % 4) plus
// a rotation by r / 4.  Transposed reads (rows 4x .. 4x + 3, chunks 4m .. 4m + 3) use one row
// group per 64 bytes and one rotation: 16 distinct slots as well.
__host__ __device__ constexpr int quad_slot(int r, int c) { return (c >> 2) * 128 + 4 * r + ((c & 3) ^ ((r >> 2) & 3)); }

template <int DT, int DH, int NW, bool KL = false>
struct BwdTiles {
    static constexpr int NKC = DH / 16;           // k-steps of 16 over the head dimension
    static constexpr int NDB = DH / 32;           // 32-row blocks of a transposed result
    static constexpr int CK = DH / 8;             // 16-byte chunks per row
    static constexpr int ROW = CK * 16;           // bytes per tile row
    static constexpr int TILE = 32 * ROW;         // one 32-row tile
    static constexpr int TI = TILE / 1024;        // DMA instructions per tile
    // dK/dV stage: Q tile | G tile (| teacher Q tile) | lse[32] | D[32] (| teacher lse[32] twice).
    // With the KL term the wave also keeps its keys' teacher K in registers: one wave per SIMD.
    static constexpr int NT_KV = KL ? 3 : 2;
    static constexpr int WPC_KV = KL && DH == 128 ? 1 : 2;          // workgroups per CU
    static constexpr int NS_KV = 4;                                 // ring stages
    static constexpr int KV_STAGE = NT_KV * TILE + (KL ? 512 : 256);
    static constexpr int KV_PW = NT_KV * TI / NW + (KL ? 2 : 1);   // DMA instructions per wave and tile
    // dQ stage: K tile | V tile (| teacher K tile)
    static constexpr int NT_Q = KL ? 3 : 2;
    static constexpr int WPC_Q = NW == 4 ? 2 : 1;
    static constexpr int NS_Q = KL ? 3 : 4;
    static constexpr int Q_STAGE = NT_Q * TILE;
    static constexpr int Q_PW = NT_Q * TI / NW;
    static_assert(TI % NW == 0, "each tile splits evenly over the waves");
    static_assert((size_t)NS_KV * KV_STAGE * WPC_KV <= 160 * 1024, "LDS ring (dK/dV)");
    static_assert((size_t)NS_Q * Q_STAGE * WPC_Q <= 160 * 1024, "LDS ring (dQ)");
};

// per-lane byte offsets inside a tile: the row read of k-step kc (logical chunk 2 kc + half of
// row lane % 32) is at rd[kc % 2] + (kc / 2) * 2048; the transposed read of k-step ks, part p
// (rows 16 ks + 8 p + 4 half .. + 3) and row block db is at tr[p] + db * 2048 + ks * 1024.
struct TileLanes {
    int rd[2], tr[2];
    __device__ TileLanes(int lane) {
        const int r = lane & 31, half = lane >> 5;
#pragma unroll
        for (int k = 0; k < 2; ++k) rd[k] = 16 * quad_slot(r, 2 * k + half);
        const int j = lane & 15, ta = j & 3, ts = j >> 2, tg = lane >> 4;
#pragma unroll
        for (int p = 0; p < 2; ++p)
            tr[p] = 16 * quad_slot(8 * p + 4 * (tg >> 1) + ts, 2 * (tg & 1) + (ta >> 1)) + 8 * (ta & 1);
    }
};

// A operand of k-step kc from a row-major tile: row (lane % 32), logical chunk 2 kc + half
template <int DT>
__device__ inline typename Mma<DT>::operand row_frag(const lds_u8 *tile, const TileLanes &tl, int kc) {
    return __builtin_bit_cast(typename Mma<DT>::operand,
                              *reinterpret_cast<const __attribute__((address_space(3))) u32x4 *>(
                                  tile + tl.rd[kc & 1] + (kc >> 1) * 2048));
}
// A operand of a product contracting over the tile's rows: row (lane % 32) of the transposed
// row block db, k-slots = the 8 tile rows 16 ks + 4 half + {0..3, 8..11}
template <int DT>
__device__ inline typename Mma<DT>::operand tr_frag(const lds_u8 *tile, const TileLanes &tl, int ks, int db) {
    const s16x4 lo = lds_read_tr16(tile + tl.tr[0] + db * 2048 + ks * 1024);
    const s16x4 hi = lds_read_tr16(tile + tl.tr[1] + db * 2048 + ks * 1024);
    return __builtin_bit_cast(typename Mma<DT>::operand, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// global source chunk of DMA piece idx (1 KiB) of a tile for this lane: row and element column
__device__ inline void quad_source(int idx, int lane, int &row, int &col) {
    const int P = idx * 64 + lane, rem = P & 127, r = rem >> 2;
    row = r;
    col = (4 * (P >> 7) + ((rem & 3) ^ ((r >> 2) & 3))) * 8;
}
// B operand of k-step ks from an accumulator tile: values 8 ks .. 8 ks + 7 rounded and packed
template <int DT>
__device__ inline typename Mma<DT>::operand acc_operand(const f32x16 &v, int ks) {
    const u32x4 w = u32x4{pack2<DT>(v[8 * ks], v[8 * ks + 1]), pack2<DT>(v[8 * ks + 2], v[8 * ks + 3]),
                          pack2<DT>(v[8 * ks + 4], v[8 * ks + 5]), pack2<DT>(v[8 * ks + 6], v[8 * ks + 7])};
    return __builtin_bit_cast(typename Mma<DT>::operand, w);
}

__device__ inline int xcd_remap(int lin, int nwg) {
    return (nwg & 7) == 0 ? (lin & 7) * (nwg >> 3) + (lin >> 3) : lin;
}

// ------------------------------------------------------------------ dK / dV
// A workgroup's four waves are KW key slices of 32 keys times QW = 4 / KW query ways: the QW waves of
// a slice take every QW-th 32-query tile and add their sums in LDS at the end (in the order of the
// ways, so the result does not depend on timing).
template <int DT, int DH, int KW, bool KL>
struct DkdvCfg {
    typedef BwdTiles<DT, DH, KW, KL> B;
    static constexpr int QW = 4 / KW;
    // a way's part of a stage: Q tile | G tile (| teacher Q tile) | lse[32] | D[32] (| teacher lse twice)
    static constexpr int NT = KL ? 3 : 2;
    static constexpr int SUB = NT * B::TILE + (KL ? 512 : 256);
    static constexpr int STAGE = QW * SUB;
    static constexpr int PW = NT * B::TI / KW + (KL ? 2 : 1);       // DMA instructions per wave and stage
    static constexpr int WPC = DH == 64 && KW > 1 && !KL ? 2 : 1;   // workgroups per CU
    static constexpr int NS = WPC * 4 * STAGE <= 160 * 1024 ? 4 : 3;                // ring stages
    static constexpr int LDS = NS * STAGE;
    static constexpr int ACC = 2 * B::NDB * 16 * 256;               // bytes of one wave's sums
    static_assert(WPC * LDS <= 160 * 1024 && (QW - 1) * KW * ACC <= LDS, "LDS ring and the exchange of the sums");
    static_assert(B::TI % KW == 0, "each tile splits evenly over a way's waves");
    static_assert(NS >= 3 && (NS - 2) * PW < 64, "the counted waits");
};

// KL: the gradient of the KL attention-map term rides along (kl_scale (P - P_t) added to each dS
// entry, P_t the teacher's map rebuilt from its projection and log-sum-exp); dS is then multiplied
// by grad_scale (a power of two that keeps fp16 in range; the scale-gradient kernel divides it out
// of the W_Q and W_K rows of the weight gradient).
// With room for it (AttnBwdArgs::ds) dS is stored for the dQ pass.
//
// The score products of tile u + 1 and the softmax of tile u are issued alternately: a wave's matrix
// instructions run while its vector instructions do, so one wave per SIMD keeps both busy, and the 512
// registers it may then use hold both tiles' scores beside the two outputs.
template <int DT, int DH, int KW, bool KL>
__global__ __launch_bounds__(256, (DkdvCfg<DT, DH, KW, KL>::WPC)) void attn_bwd_dkdv_pipe_kernel(
    AttnBwdArgs a, float scale_log2, float inv_sqrt, int nkb, uint32_t inv_g) {
    typedef DkdvCfg<DT, DH, KW, KL> C;
    typedef typename C::B B;
    typedef Mma<DT> MM;
    typedef typename MM::operand opnd;
    typedef uint16_t elem;
    constexpr int BK = 32 * KW;                        // keys per block
    constexpr int NS = C::NS, QW = C::QW, NKC = B::NKC, NDB = B::NDB, TI = B::TI;
    extern __shared__ __align__(16) unsigned char smem[];

    const int T = a.seq_len, Hq = a.n_heads, Hkv = a.n_kv_heads;
    const int G = Hq / Hkv;
    // one key block per workgroup, the longest first, so that the short ones fill what the long ones
    // leave idle; one kv head's workgroups on one XCD where the counts allow it
    const int heads = gridDim.x / nkb, per = heads & 7 ? heads : heads >> 3;
    const int xcd = heads & 7 ? 0 : blockIdx.x & 7, idx = heads & 7 ? blockIdx.x : blockIdx.x >> 3;
    const int kb = idx / per, head = xcd * per + idx % per;
    const int kvh = head % Hkv, b = head / Hkv;
    const int nq = (T - kb * BK + 31) / 32, n = G * nq;        // its tiles, QW per step
    const int U = (n + QW - 1) / QW;

    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int kw = wave % KW, qw = wave / KW;
    const int64_t row0 = (int64_t)b * T;
    const elem *Qs = static_cast<const elem *>(a.q) + row0 * a.ldq;
    const elem *Gs = static_cast<const elem *>(a.g) + row0 * Hq * DH;
    const elem *Qts = KL ? static_cast<const elem *>(a.qt) + row0 * a.ldq : nullptr;
    const int64_t ld_base = (int64_t)b * Hq * T;       // lse2 / D of (b, h, t): ld_base + h T + t

    // step u, this wave's way -> query head, first query (the group's heads for the last query tile,
    // then the tile below, down to the block's diagonal; past the last tile the last one again, which
    // is then not used)
    auto tile_of = [&](int u, int &h, int &q0) -> bool {
        const int v0 = QW * u + qw;
        const int v = min(v0, n - 1);
        const int vq = G == 1 ? v : (int)__umulhi((uint32_t)v, inv_g);     // v / G
        h = kvh * G + (v - vq * G);
        q0 = kb * BK + 32 * (nq - 1 - vq);
        return v0 < n;
    };

    // ---- DMA: instruction i of a wave loads 1 KiB piece kw + KW i of its way's tiles (pieces
    // [0, TI): Q, [TI, 2 TI): G, [2 TI, 3 TI): the teacher's Q), then lse and D (one 4-byte load per
    // lane: lanes below 32 lse, the others D) and with the KL term the teacher's lse (every lane; lanes
    // 32..63 repeat lanes 0..31).  A piece's row inside the tile depends on its parity alone and its
    // first column is wave-uniform, so a lane forms one offset per tensor and parity.  Steps past the
    // last load the last tile again: the waits below count the same loads in every step.
    constexpr int NP = C::NT * TI / KW, NPAR = KW == 1 ? 2 : 1;
    auto stage_ptr = [&](int s) { return smem + s * C::STAGE + qw * C::SUB; };
    const float *ldp = (lane < 32 ? a.lse2 : a.D) + ld_base;
    const int dcol = ((lane & 3) ^ ((lane >> 4) & 3)) * 8;             // quad_source at the lane
    struct Loads { uint32_t q[NPAR], g[NPAR]; int l; const elem *Q, *G, *Qt; unsigned char *st; int h; };
    auto plan = [&](int u, Loads &x) {
        int h, q0;
        tile_of(min(u, U - 1), h, q0);
#pragma unroll
        for (int p = 0; p < NPAR; ++p) {
            const int q = min(q0 + 16 * (KW == 1 ? p : kw & 1) + (lane >> 2), T - 1);
            x.q[p] = 2u * (uint32_t)(q * a.ldq + dcol);
            x.g[p] = 2u * (uint32_t)(q * Hq * DH + dcol);
        }
        x.l = min(q0 + (lane & 31), T - 1);
        x.Q = Qs + h * DH;
        x.G = Gs + h * DH;
        if constexpr (KL) x.Qt = Qts + h * DH;
        x.st = stage_ptr(u % NS);
        x.h = h;
    };
    auto issue_part = [&](const Loads &x, int i) {
        if (i < NP) {
            const int tix = (KW * i) / TI, idx = kw + (KW * i) % TI, par = KW == 1 ? i & 1 : 0;
            const elem *base = (tix == 0 ? x.Q : tix == 1 ? x.G : x.Qt) + 32 * (idx >> 1);
            lds_dma16_raw(base, tix == 1 ? x.g[par] : x.q[par], x.st + tix * B::TILE + idx * 1024);
        } else if (i == NP) {
            lds_dma4_raw(ldp + (int64_t)x.h * T + x.l, x.st + C::NT * B::TILE);
        } else if (KL && i == NP + 1) {
            lds_dma4_raw(a.lse_t + ld_base + (int64_t)x.h * T + x.l, x.st + C::NT * B::TILE + 256);
        }
    };
    auto sync = [&] {
        if constexpr (KW > 1) raw_barrier();
        else asm volatile("" ::: "memory");            // a way of one wave reads its own loads only
    };

    const int kw0 = kb * BK + 32 * kw;                 // first key of this wave
    const TileLanes tl(lane);
    opnd kf[NKC], vf[NKC], ktf[KL ? NKC : 1];
    f32x16 dkt[NDB], dvt[NDB];
    auto load_keys = [&] {
        const int kr = min(kw0 + (lane & 31), T - 1);
        const elem *kp = static_cast<const elem *>(a.k) + (row0 + kr) * a.ldq + kvh * DH + half * 8;
        const elem *vp = static_cast<const elem *>(a.v) + (row0 + kr) * a.ldv + kvh * DH + half * 8;
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
            kf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(kp + kc * 16));
            vf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(vp + kc * 16));
        }
        if constexpr (KL) {
            const elem *ktp = static_cast<const elem *>(a.kt) + (row0 + kr) * a.ldq + kvh * DH + half * 8;
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc)
                ktf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(ktp + kc * 16));
        }
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) { dkt[d][e] = 0.f; dvt[d][e] = 0.f; }
    };
    // dK^T, dV^T: lane -> key (a token column of dY^T), registers -> head-dimension rows
    auto store_sums = [&] {
        if constexpr (QW > 1) {                        // the ways' sums, exchanged through the (drained) ring
            typedef __attribute__((address_space(3))) float lds_f32;
            lds_f32 *ex = (lds_f32 *)smem;
            constexpr int WF = C::ACC / 4;
            wait_lgkm0();
            wait_vmcnt<0>();
            raw_barrier();
            if (qw > 0) {
                lds_f32 *o = ex + ((qw - 1) * KW + kw) * WF + lane;
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        o[(d * 16 + e) * 64] = dkt[d][e];
                        o[((NDB + d) * 16 + e) * 64] = dvt[d][e];
                    }
            }
            __syncthreads();
            if (qw > 0) return;
#pragma unroll 1
            for (int w = 1; w < QW; ++w) {
                const lds_f32 *o = ex + ((w - 1) * KW + kw) * WF + lane;
#pragma unroll
                for (int d = 0; d < NDB; ++d)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        dkt[d][e] += o[(d * 16 + e) * 64];
                        dvt[d][e] += o[((NDB + d) * 16 + e) * 64];
                    }
            }
        }
        const int key = kw0 + (lane & 31);
        if (key >= T) return;
        elem *dyt = static_cast<elem *>(a.dyt) + row0 + key;
        const int koff = Hq * DH + kvh * DH, voff = (Hq + Hkv) * DH + kvh * DH;
#pragma unroll
        for (int d = 0; d < NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                dyt[(int64_t)(koff + c) * a.ldt] = from_f32<DT>(dkt[d][e] * inv_sqrt);
                dyt[(int64_t)(voff + c) * a.ldt] = from_f32<DT>(dvt[d][e]);
            }
    };

    // The scores of a tile: S = Q K^T, dP = G V^T and the teacher's S_t = Q_t K_t^T; lane -> key,
    // registers -> queries 8 (e / 4) + 4 half + e % 4
    struct Scores { f32x16 s, dp, st; };
    auto clear = [&](Scores &x) {
#pragma unroll
        for (int e = 0; e < 16; ++e) { x.s[e] = 0.f; x.dp[e] = 0.f; if constexpr (KL) x.st[e] = 0.f; }
    };
    struct Frags { opnd q, g, t; };
    auto score_frags = [&](Frags &f, const lds_u8 *stq, int kc) {
        f.q = row_frag<DT>(stq, tl, kc);
        f.g = row_frag<DT>(stq + B::TILE, tl, kc);
        if constexpr (KL) f.t = row_frag<DT>(stq + 2 * B::TILE, tl, kc);
    };
    auto score_step = [&](Scores &x, const Frags &f, int kc) {
        x.s = MM::mma(f.q, kf[kc], x.s);
        x.dp = MM::mma(f.g, vf[kc], x.dp);
        if constexpr (KL) x.st = MM::mma(f.t, ktf[kc], x.st);
    };

    // step u: P and dS of tile u from its scores x, beside the scores y of tile u + 1; then the products
    auto step = [&](int u, Scores &x, Scores &y) {
        // this wave's part of tile u + 1 has landed (tiles issued after it may be pending), then every
        // wave's part; every wave is also done reading tile u - 1, whose stage is refilled.  The dS
        // stores in between only make a wait longer.
        wait_lgkm0();
        wait_vmcnt<(NS - 3) * C::PW>();
        sync();
        const lds_u8 *stq = (const lds_u8 *)stage_ptr(u % NS);
        const lds_u8 *stn = (const lds_u8 *)stage_ptr((u + 1) % NS);
        const lds_u8 *stg = stq + B::TILE;
        Frags fr[NKC];
        score_frags(fr[0], stn, 0);
        score_frags(fr[1], stn, 1);
        const __attribute__((address_space(3))) float *lsd =
            (const __attribute__((address_space(3))) float *)(stq + C::NT * B::TILE);
        f32x4 ls[4], dd[4], lt[4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int r0 = 8 * e4 + 4 * half;
            ls[e4] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + r0);
            dd[e4] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + 32 + r0);
            if constexpr (KL) lt[e4] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + 64 + r0);
        }
        Loads ld;
        plan(u + NS - 1, ld);
        int h, q0;
        const bool valid = tile_of(u, h, q0);
        clear(y);
        constexpr int EPK = 16 / NKC, IPK = (C::PW + NKC - 1) / NKC;   // softmax entries, loads per k-step
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) {
            if (kc + 2 < NKC) score_frags(fr[kc + 2], stn, kc + 2);
            score_step(y, fr[kc], kc);
#pragma unroll
            for (int i = kc * IPK; i < (kc + 1) * IPK; ++i) issue_part(ld, i);
#pragma unroll
            for (int i = 0; i < EPK; ++i) {
                const int e = kc * EPK + i;
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(x.s[e], scale_log2, -ls[e >> 2][e & 3]));
                float ds = p * (x.dp[e] - dd[e >> 2][e & 3]);
                if constexpr (KL) {
                    const float pt = __builtin_amdgcn_exp2f(__builtin_fmaf(x.st[e], scale_log2, -lt[e >> 2][e & 3]));
                    ds = (ds + a.kl_scale * (p - pt)) * a.grad_scale;
                }
                // kept here: the compiler would sink the whole softmax behind the branch below
                float pk = p, dk = ds;
                asm volatile("" : "+v"(pk), "+v"(dk));
                x.s[e] = pk;
                x.dp[e] = dk;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // the first operands of the products below
        opnd tg[2], tq[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            tg[d] = tr_frag<DT>(stg, tl, 0, d);
            tq[d] = tr_frag<DT>(stq, tl, 0, d);
        }
        if (!valid || q0 + 31 < kw0 || kw0 >= T) return;   // no query of the tile sees these keys
        // the diagonal and sequence-tail tiles (wave-uniform): entries above the diagonal or past the
        // sequence are zero; the other tiles take no compare and no select
        if (q0 < kw0 + 31 || q0 + 31 >= T) {
            const int key = kw0 + (lane & 31);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int q = q0 + 8 * (e >> 2) + 4 * half + (e & 3);
                const bool off = q < key || q >= T;
                x.s[e] = off ? 0.f : x.s[e];
                x.dp[e] = off ? 0.f : x.dp[e];
            }
        }
        // dV^T += G^T P, dK^T += Q^T dS (k = the tile's 32 queries in two steps); the operand of each
        // step is the dS tile that the dQ pass reads (2 KiB per tile: step ks, lane at ks KiB + 16
        // lane).  The tile's address is wave-uniform (a buffer resource in scalar registers); the store
        // is non-temporal (read once, by the dQ pass), so it does not push the Q and G tiles out of L2.
        const opnd sb[2] = {acc_operand<DT>(x.dp, 0), acc_operand<DT>(x.dp, 1)};
        if (a.ds) {
            const int qt = q0 / 32, kt = kw0 / 32, nt = (T + 31) / 32;
            const i32x4 rds = buffer_rsrc(static_cast<char *>(a.ds) +
                                          (((int64_t)b * Hq + h) * (nt * (nt + 1) / 2) + qt * (qt + 1) / 2 + kt) * 2048);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                buffer_store16_nt(rds, lane * 16, ks * 1024, __builtin_bit_cast(i32x4, sb[ks]));
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const opnd pb = acc_operand<DT>(x.s, ks);
#pragma unroll
            for (int d = 0; d < NDB; ++d) {
                const bool have = ks == 0 && d < 2;
                dvt[d] = MM::mma(have ? tg[d & 1] : tr_frag<DT>(stg, tl, ks, d), pb, dvt[d]);
                dkt[d] = MM::mma(have ? tq[d & 1] : tr_frag<DT>(stq, tl, ks, d), sb[ks], dkt[d]);
            }
        }
    };

#pragma unroll
    for (int t = 0; t < NS - 1; ++t) {
        Loads ld;
        plan(t, ld);
#pragma unroll
        for (int i = 0; i < C::PW; ++i) issue_part(ld, i);
    }
    load_keys();
    wait_vmcnt<0>();                                   // the keys and the first tiles
    sync();
    Scores x, y;
    clear(x);
    const lds_u8 *st0 = (const lds_u8 *)stage_ptr(0);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
        Frags f;
        score_frags(f, st0, kc);
        score_step(x, f, kc);
    }
    int u = 0;
    for (; u + 1 < U; u += 2) {
        step(u, x, y);
        step(u + 1, y, x);
    }
    if (u < U) step(u, x, y);
    store_sums();
    wait_vmcnt<0>();                                   // no load into LDS outlives the workgroup
}

// The same tile after tile, two key blocks per workgroup and two workgroups per CU, for grids that
// fill the chip twice.
template <int DT, int DH, int NW, bool KL, bool DS>
__global__ __launch_bounds__(64 * NW, (BwdTiles<DT, DH, NW, KL>::WPC_KV)) void attn_bwd_dkdv_dma_kernel(
    AttnBwdArgs a, float scale_log2, float inv_sqrt, int nkb, int npair) {
    typedef BwdTiles<DT, DH, NW, KL> C;
    typedef Mma<DT> MM;
    typedef typename MM::operand opnd;
    typedef uint16_t elem;
    constexpr int BK = 32 * NW;                        // keys per block
    constexpr int NS = C::NS_KV;
    extern __shared__ __align__(16) unsigned char smem[];
    const lds_u8 *sm = (const lds_u8 *)smem;

    const int T = a.seq_len, Hq = a.n_heads, Hkv = a.n_kv_heads;
    const int G = Hq / Hkv;
    const int lin = xcd_remap(blockIdx.x, gridDim.x);
    const int pr = lin % npair;
    const int kvh = (lin / npair) % Hkv;
    const int b = lin / (npair * Hkv);
    const int kbA = pr, kbB = nkb - 1 - pr;            // equal for the middle block of an odd count
    const int nqA = (T - kbA * BK + 31) / 32, nqB = (T - kbB * BK + 31) / 32;
    const int nA = G * nqA;
    const int U = nA + (kbB != kbA ? G * nqB : 0);     // tiles of this workgroup

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int64_t row0 = (int64_t)b * T;
    const elem *Qs = static_cast<const elem *>(a.q) + row0 * a.ldq;
    const elem *Gs = static_cast<const elem *>(a.g) + row0 * Hq * DH;
    const elem *Qts = KL ? static_cast<const elem *>(a.qt) + row0 * a.ldq : nullptr;
    const int64_t ld_base = (int64_t)b * Hq * T;       // lse2 / D of (b, h, t): ld_base + h T + t

    // tile u -> key block, query head, first query (tiles of a block: the group's heads for
    // the last query tile, then the tile below, down to the block's diagonal)
    auto tile_of = [&](int u, int &kb, int &h, int &q0) {
        const bool second = u >= nA;
        const int v = second ? u - nA : u;
        kb = second ? kbB : kbA;
        const int nq = second ? nqB : nqA;
        h = kvh * G + v % G;
        q0 = kb * BK + 32 * (nq - 1 - v / G);
    };

    // ---- DMA: instruction i of this wave loads 1 KiB piece wave + NW i of the stage's tiles
    // (pieces [0, TI): Q, [TI, 2 TI): G, [2 TI, 3 TI): the teacher's Q), then lse and D (one
    // 4-byte load per lane: lanes below 32 lse, the others D) and with the KL term the teacher's
    // lse (every lane; lanes 32..63 repeat lanes 0..31)
    constexpr int NP = C::NT_KV * C::TI / NW;
    auto stage_ptr = [&](int s) { return smem + s * C::KV_STAGE; };
    // piece wave + NW i lies in tile (NW i) / TI (TI is a multiple of NW); its LDS offset inside
    // that tile is wave KiB plus a constant
    const int wofs = __builtin_amdgcn_readfirstlane(wave * 1024);
    const float *ldp = (lane < 32 ? a.lse2 : a.D) + ld_base;
    auto issue = [&](int u) {
        if (u >= U) return;
        int kb, h, q0;
        tile_of(u, kb, h, q0);
        unsigned char *st = stage_ptr(u % NS) + wofs;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int tix = (NW * i) / C::TI;
            int drow, dcol;                            // formed per load: registers are scarce here
            quad_source((wave + NW * i) % C::TI, lane, drow, dcol);
            const int q = min(q0 + drow, T - 1);
            const elem *src = tix == 1 ? Gs + h * DH + (q * Hq * DH + dcol)
                                       : (tix == 0 ? Qs : Qts) + h * DH + (q * a.ldq + dcol);
            lds_dma16((const void *)src, st + tix * C::TILE + ((NW * i) % C::TI) * 1024);
        }
        const int q = min(q0 + (lane & 31), T - 1);
        lds_dma4((const void *)(ldp + (h * T + q)), stage_ptr(u % NS) + C::NT_KV * C::TILE);
        if constexpr (KL)
            lds_dma4((const void *)(a.lse_t + ld_base + (h * T + q)), stage_ptr(u % NS) + C::NT_KV * C::TILE + 256);
    };

    const TileLanes tl(lane);
    opnd kf[C::NKC], vf[C::NKC], ktf[KL ? C::NKC : 1];
    f32x16 dkt[C::NDB], dvt[C::NDB];
    auto begin_block = [&](int kb) {
        const int key = kb * BK + 32 * wave + (lane & 31);
        const int kr = min(key, T - 1);
        const elem *kp = static_cast<const elem *>(a.k) + (row0 + kr) * a.ldq + kvh * DH + half * 8;
        const elem *vp = static_cast<const elem *>(a.v) + (row0 + kr) * a.ldv + kvh * DH + half * 8;
#pragma unroll
        for (int kc = 0; kc < C::NKC; ++kc) {
            kf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(kp + kc * 16));
            vf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(vp + kc * 16));
        }
        if constexpr (KL) {
            const elem *ktp = static_cast<const elem *>(a.kt) + (row0 + kr) * a.ldq + kvh * DH + half * 8;
#pragma unroll
            for (int kc = 0; kc < C::NKC; ++kc)
                ktf[kc] = __builtin_bit_cast(opnd, *reinterpret_cast<const u32x4 *>(ktp + kc * 16));
        }
#pragma unroll
        for (int d = 0; d < C::NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) { dkt[d][e] = 0.f; dvt[d][e] = 0.f; }
    };
    // dK^T, dV^T: lane -> key (a token column of dY^T), registers -> head-dimension rows
    auto end_block = [&](int kb) {
        const int key = kb * BK + 32 * wave + (lane & 31);
        if (key >= T) return;
        elem *dyt = static_cast<elem *>(a.dyt) + row0 + key;
        const int koff = Hq * DH + kvh * DH, voff = (Hq + Hkv) * DH + kvh * DH;
#pragma unroll
        for (int d = 0; d < C::NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                dyt[(int64_t)(koff + c) * a.ldt] = from_f32<DT>(dkt[d][e] * inv_sqrt);
                dyt[(int64_t)(voff + c) * a.ldt] = from_f32<DT>(dvt[d][e]);
            }
    };

    // tiles [u0, u1) of key block kb
    auto run_block = [&](int kb, int u0, int u1) {
        begin_block(kb);
        for (int u = u0; u < u1; ++u) {
            // this wave's part of tile u has landed (the tiles issued after it may be pending),
            // then every wave's part; every wave is also done reading tile u - 1, whose stage is
            // refilled
            wait_vm_groups<C::KV_PW, NS - 2>(min(NS - 2, U - 1 - u));
            raw_barrier();
            issue(u + NS - 1);
            int kbu, h, q0;
            tile_of(u, kbu, h, q0);
            const int kw = kb * BK + 32 * wave;        // first key of this wave
            if (q0 + 31 < kw || kw >= T) continue;     // no query of the tile sees these keys
            const lds_u8 *stq = sm + (u % NS) * C::KV_STAGE;
            const lds_u8 *stg = stq + C::TILE;
            const __attribute__((address_space(3))) float *lsd =
                (const __attribute__((address_space(3))) float *)(stq + C::NT_KV * C::TILE);

            // S = Q K^T, dP = G V^T (and the teacher's S_t = Q_t K_t^T): lane -> key, registers ->
            // queries 8 (e / 4) + 4 half + e % 4
            f32x16 s, dp, st;
#pragma unroll
            for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; st[e] = 0.f; }
#pragma unroll
            for (int kc = 0; kc < C::NKC; ++kc) {
                s = MM::mma(row_frag<DT>(stq, tl, kc), kf[kc], s);
                dp = MM::mma(row_frag<DT>(stg, tl, kc), vf[kc], dp);
                if constexpr (KL) st = MM::mma(row_frag<DT>(stq + 2 * C::TILE, tl, kc), ktf[kc], st);
            }
            const int key = kw + (lane & 31);
            const bool diag = q0 < kw + 31, tail = q0 + 31 >= T;
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const int r0 = 8 * e4 + 4 * half;
                const f32x4 ls = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + r0);
                const f32x4 dd = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + 32 + r0);
                f32x4 lt;
                if constexpr (KL) lt = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>(lsd + 64 + r0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = 4 * e4 + i;
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2, -ls[i]));
                    float ds = p * (dp[e] - dd[i]);
                    if constexpr (KL) {
                        const float pt = __builtin_amdgcn_exp2f(__builtin_fmaf(st[e], scale_log2, -lt[i]));
                        ds = (ds + a.kl_scale * (p - pt)) * a.grad_scale;
                    }
                    s[e] = p;
                    dp[e] = ds;
                }
            }
            // the diagonal and sequence-tail tiles (wave-uniform): entries above the diagonal or
            // past the sequence are zero; the other tiles take no compare and no select
            if (diag || tail) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int q = q0 + 8 * (e >> 2) + 4 * half + (e & 3);
                    const bool off = q < key || q >= T;
                    s[e] = off ? 0.f : s[e];
                    dp[e] = off ? 0.f : dp[e];
                }
            }
            // dV^T += G^T P, dK^T += Q^T dS (k = the tile's 32 queries in two steps); with a dS store,
            // the operand of each step goes out before its products (2 KiB per tile: step ks, lane
            // at ks KiB + 16 lane), for the dQ pass.  The tile's address is wave-uniform (a buffer
            // resource in scalar registers); the store is non-temporal (read once, by the dQ pass),
            // so it does not push the Q and G tiles out of L2.
            i32x4 rds;
            if constexpr (DS) {
                const int qt = q0 / 32, kt = __builtin_amdgcn_readfirstlane(kw / 32), nq = (T + 31) / 32;
                rds = buffer_rsrc(static_cast<char *>(a.ds) +
                                  (((int64_t)b * Hq + h) * (nq * (nq + 1) / 2) + qt * (qt + 1) / 2 + kt) * 2048);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const opnd pb = acc_operand<DT>(s, ks), sb = acc_operand<DT>(dp, ks);
                if constexpr (DS) buffer_store16_nt(rds, lane * 16, ks * 1024, __builtin_bit_cast(i32x4, sb));
#pragma unroll
                for (int d = 0; d < C::NDB; ++d) {
                    dvt[d] = MM::mma(tr_frag<DT>(stg, tl, ks, d), pb, dvt[d]);
                    dkt[d] = MM::mma(tr_frag<DT>(stq, tl, ks, d), sb, dkt[d]);
                }
            }
        }
        end_block(kb);
    };

#pragma unroll
    for (int t = 0; t < NS - 1; ++t) issue(t);
    run_block(kbA, 0, nA);
    if (U > nA) run_block(kbB, nA, U);
}

// ------------------------------------------------------------------ dQ
template <int DT, int DH, int NW, bool KL>
__global__ __launch_bounds__(64 * NW, (BwdTiles<DT, DH, NW, KL>::WPC_Q)) void attn_bwd_dq_dma_kernel(
    AttnBwdArgs a, float scale_log2, float inv_sqrt, int hpw, int nqt, int n_ht) {
    typedef BwdTiles<DT, DH, NW, KL> C;
    typedef Mma<DT> MM;
    typedef typename MM::operand opnd;
    typedef uint16_t elem;
    constexpr int NS = C::NS_Q;
    extern __shared__ __align__(16) unsigned char smem[];
    const lds_u8 *sm = (const lds_u8 *)smem;

    const int T = a.seq_len, Hq = a.n_heads;
    const int G = Hq / a.n_kv_heads;
    const int QT = 32 * NW / hpw;                      // queries per workgroup
    const int lin = xcd_remap(blockIdx.x, gridDim.x);
    const int qt = nqt - 1 - lin % nqt;                // longest query tiles first
    const int ht = (lin / nqt) % n_ht;
    const int b = lin / (nqt * n_ht);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int h = ht * hpw + wave % hpw;
    const int kvh = h / G;
    const int q0 = qt * QT + (wave / hpw) * 32;        // first query of this wave
    const int qrow = q0 + (lane & 31);
    const int kend = min(T, qt * QT + QT);
    const int nblk = (kend + 31) / 32;
    const int jlast = q0 < T ? q0 / 32 : -1;           // the wave's diagonal block
    const int64_t row0 = (int64_t)b * T;
    const elem *Ks = static_cast<const elem *>(a.k) + row0 * a.ldq + kvh * DH;
    const elem *Vs = static_cast<const elem *>(a.v) + row0 * a.ldv + kvh * DH;
    const elem *Kts = KL ? static_cast<const elem *>(a.kt) + row0 * a.ldq + kvh * DH : nullptr;

    // this wave's queries as B operands of S^T = K Q^T and dP^T = V G^T (and of the teacher's
    // S_t^T = K_t Q_t^T)
    opnd qf[C::NKC], gf[C::NKC], qtf[KL ? C::NKC : 1];
    {
        const int qr = min(qrow, T - 1);
        const elem *qp = static_cast<const elem *>(a.q) + (row0 + qr) * a.ldq + h * DH + half * 8;
        const elem *gp = static_cast<const elem *>(a.g) + ((row0 + qr) * Hq + h) * DH + half * 8;
#pragma unroll
        for (int kc = 0; kc < C::NKC; ++kc) {
            u32x4 x = *reinterpret_cast<const u32x4 *>(qp + kc * 16);
            u32x4 y = *reinterpret_cast<const u32x4 *>(gp + kc * 16);
            if (qrow >= T) { x = u32x4{0u, 0u, 0u, 0u}; y = x; }
            qf[kc] = __builtin_bit_cast(opnd, x);
            gf[kc] = __builtin_bit_cast(opnd, y);
        }
        if constexpr (KL) {
            const elem *qtp = static_cast<const elem *>(a.qt) + (row0 + qr) * a.ldq + h * DH + half * 8;
#pragma unroll
            for (int kc = 0; kc < C::NKC; ++kc) {
                u32x4 x = *reinterpret_cast<const u32x4 *>(qtp + kc * 16);
                if (qrow >= T) x = u32x4{0u, 0u, 0u, 0u};
                qtf[kc] = __builtin_bit_cast(opnd, x);
            }
        }
    }
    const int64_t li = ((int64_t)b * Hq + h) * T + min(qrow, T - 1);
    const float lse = qrow < T ? a.lse2[li] : INFINITY;
    const float Dq = qrow < T ? a.D[li] : 0.f;
    const float lset = KL && qrow < T ? a.lse_t[li] : INFINITY;

    // ---- DMA: instruction i of this wave loads 1 KiB piece wave + NW i of the stage's K, V (and
    // teacher K) tiles (piece p lies in tile p / TI)
    constexpr int NP = C::Q_PW;
    int drow[NP], dcol[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        quad_source((wave + NW * i) % C::TI, lane, drow[i], dcol[i]);
    }
    const int wofs = __builtin_amdgcn_readfirstlane(wave * 1024);
    auto issue = [&](int j) {
        if (j >= nblk) return;
        unsigned char *st = smem + (j % NS) * C::Q_STAGE + wofs;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int tix = (NW * i) / C::TI;
            const int k = min(32 * j + drow[i], T - 1);
            const elem *src = tix == 1 ? Vs + (k * a.ldv + dcol[i]) : (tix == 0 ? Ks : Kts) + (k * a.ldq + dcol[i]);
            lds_dma16((const void *)src, st + tix * C::TILE + ((NW * i) % C::TI) * 1024);
        }
    };

    const TileLanes tl(lane);
    f32x16 dqt[C::NDB];
#pragma unroll
    for (int d = 0; d < C::NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) dqt[d][e] = 0.f;

#pragma unroll
    for (int t = 0; t < NS - 1; ++t) issue(t);
    for (int j = 0; j < nblk; ++j) {
        wait_vm_groups<C::Q_PW, NS - 2>(min(NS - 2, nblk - 1 - j));
        raw_barrier();
        issue(j + NS - 1);
        if (j > jlast) continue;                       // keys above every query of the wave
        const lds_u8 *stk = sm + (j % NS) * C::Q_STAGE;
        const lds_u8 *stv = stk + C::TILE;
        // S^T = K Q^T, dP^T = V G^T: lane -> query, registers -> keys 8 (e / 4) + 4 half + e % 4
        f32x16 s, dp, st;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; st[e] = 0.f; }
#pragma unroll
        for (int kc = 0; kc < C::NKC; ++kc) {
            s = MM::mma(row_frag<DT>(stk, tl, kc), qf[kc], s);
            dp = MM::mma(row_frag<DT>(stv, tl, kc), gf[kc], dp);
            if constexpr (KL) st = MM::mma(row_frag<DT>(stk + 2 * C::TILE, tl, kc), qtf[kc], st);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2, -lse));
            float ds = p * (dp[e] - Dq);
            if constexpr (KL) {
                const float pt = __builtin_amdgcn_exp2f(__builtin_fmaf(st[e], scale_log2, -lset));
                ds = (ds + a.kl_scale * (p - pt)) * a.grad_scale;
            }
            dp[e] = ds;
        }
        if (j == jlast) {                              // the diagonal tile (wave-uniform) alone is masked
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int key = 32 * j + 8 * (e >> 2) + 4 * half + (e & 3);
                dp[e] = key > qrow ? 0.f : dp[e];
            }
        }
        // dQ^T += K^T dS^T (k = the tile's 32 keys in two steps)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const opnd sb = acc_operand<DT>(dp, ks);
#pragma unroll
            for (int d = 0; d < C::NDB; ++d) dqt[d] = MM::mma(tr_frag<DT>(stk, tl, ks, d), sb, dqt[d]);
        }
    }
    if (qrow < T) {
        elem *dyt = static_cast<elem *>(a.dyt) + row0 + qrow;
#pragma unroll
        for (int d = 0; d < C::NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                dyt[(int64_t)(h * DH + c) * a.ldt] = from_f32<DT>(dqt[d][e] * inv_sqrt);
            }
    }
}

// ------------------------------------------------------------------ dQ from the stored dS
// dQ^T += K^T dS^T over the key tiles of the wave's queries, dS read back as the dK pass stored it
// (the operand of dK^T += Q^T dS: lane = key, eight queries per step).  The workgroup's waves share
// the kv head's key tiles (an LDS ring, as the recomputing kernel); each wave's dS tile rides the same
// stage and is read transposed (ds_read_b64_tr_b16) into the B operand of the dQ product: lane =
// query, keys 16 ks + 4 half + {0..3, 8..11}, the k-slots of tr_frag on the key tile.  The same
// product as the recomputing kernel, on the dK pass's dS.
template <int DT, int DH, int NW>
struct DqDsCfg {
    typedef BwdTiles<DT, DH, NW> B;
    static constexpr int NS = 3;                        // 48 KiB at head_dim 128: three workgroups per CU
    static constexpr int STAGE = B::TILE + NW * 2048;   // key tile | the waves' dS tiles
    static constexpr int PW = B::TI / NW + 2;            // DMA instructions per wave and stage
    static constexpr int WPC = NW == 4 ? 2 : 1;         // at least
    static_assert((size_t)NS * STAGE * WPC <= 160 * 1024, "LDS ring (dQ from dS)");
};

template <int DT, int DH, int NW>
__global__ __launch_bounds__(64 * NW, (DqDsCfg<DT, DH, NW>::WPC)) void attn_bwd_dq_ds_kernel(
    AttnBwdArgs a, float inv_sqrt, int hpw, int nqt, int n_ht) {
    typedef BwdTiles<DT, DH, NW> C;
    typedef DqDsCfg<DT, DH, NW> D;
    typedef Mma<DT> MM;
    typedef typename MM::operand opnd;
    typedef uint16_t elem;
    constexpr int NS = D::NS;
    extern __shared__ __align__(16) unsigned char smem[];
    const lds_u8 *sm = (const lds_u8 *)smem;

    const int T = a.seq_len, Hq = a.n_heads;
    const int G = Hq / a.n_kv_heads;
    const int QT = 32 * NW / hpw;                      // queries per workgroup
    const int lin = xcd_remap(blockIdx.x, gridDim.x);
    const int qt = nqt - 1 - lin % nqt;                // longest query tiles first
    const int ht = (lin / nqt) % n_ht;
    const int b = lin / (nqt * n_ht);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int h = ht * hpw + wave % hpw;
    const int kvh = h / G;
    const int q0 = qt * QT + (wave / hpw) * 32;        // first query of this wave
    const int qrow = q0 + (lane & 31);
    const int kend = min(T, qt * QT + QT);
    const int nblk = (kend + 31) / 32;
    const int jlast = q0 < T ? q0 / 32 : -1;           // the wave's diagonal block
    const int64_t row0 = (int64_t)b * T;
    const elem *Ks = static_cast<const elem *>(a.k) + row0 * a.ldq + kvh * DH;
    const int nq = (T + 31) / 32;
    // the wave's dS tiles: (sequence b, head h, query tile q0 / 32, key tile j)
    const char *dsw = static_cast<const char *>(a.ds) +
                      (((int64_t)b * Hq + h) * (nq * (nq + 1) / 2) + (jlast >= 0 ? jlast * (jlast + 1) / 2 : 0)) * 2048;

    // ---- DMA: instruction i < TI / NW of this wave loads key-tile piece wave + NW i; the last two load
    // the wave's dS tile (blocks past its diagonal re-load the diagonal's, never read), its 16-byte
    // chunk c placed at chunk c ^ 8 (c >> 5 & 1) ^ 4 (c >> 6 & 1) of the wave's LDS area (an
    // involution) so the transposed reads below are free of bank conflicts
    constexpr int NK = C::TI / NW;
    int drow[NK], dcol[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) quad_source(wave + NW * i, lane, drow[i], dcol[i]);
    const int wofs = __builtin_amdgcn_readfirstlane(wave * 1024);
    const int dofs = __builtin_amdgcn_readfirstlane(C::TILE + wave * 2048);
    int dsrc[2];                                       // byte of the dS tile lane `lane` of piece i loads
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int pc = 64 * i + lane;
        dsrc[i] = (pc ^ (((pc >> 5) & 1) << 3) ^ (((pc >> 6) & 1) << 2)) * 16;
    }
    auto issue = [&](int j) {
        if (j >= nblk) return;
        unsigned char *st = smem + (j % NS) * D::STAGE;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int k = min(32 * j + drow[i], T - 1);
            lds_dma16((const void *)(Ks + (k * a.ldq + dcol[i])), st + wofs + NW * i * 1024);
        }
        // dS is read once: non-temporal, so it does not push the key tiles out of L2
        const char *src = dsw + (int64_t)min(j, max(jlast, 0)) * 2048;
#pragma unroll
        for (int i = 0; i < 2; ++i) lds_dma16_nt((const void *)(src + dsrc[i]), st + dofs + i * 1024);
    };

    // transposed reads of the dS tile: read rr of k-step ks, lane a + 4 s of its 16-lane group g:
    // key 16 ks + 4 (g / 2) + 8 rr + s, queries 16 (g % 2) + 4 a .. + 3, stored as chunk
    // c = 64 (g % 2) + 32 (a % 2) + key (16 bytes, the query pairs at 8 (a / 2) within it), which
    // the DMA placed at chunk c ^ 8 (a % 2) ^ 4 (g % 2)
    const int jg = lane & 15, ta = jg & 3, ts = jg >> 2, tg = lane >> 4;
    int dsoff[2];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr)
        dsoff[rr] = (64 * (tg & 1) + 32 * (ta & 1) + 8 * ((ta & 1) ^ rr) + 4 * ((tg >> 1) ^ (tg & 1)) + ts) * 16 +
                    8 * (ta >> 1);
    const TileLanes tl(lane);
    f32x16 dqt[C::NDB];
#pragma unroll
    for (int d = 0; d < C::NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) dqt[d][e] = 0.f;

#pragma unroll
    for (int t = 0; t < NS - 1; ++t) issue(t);
    for (int j = 0; j < nblk; ++j) {
        wait_vm_groups<D::PW, NS - 2>(min(NS - 2, nblk - 1 - j));
        raw_barrier();
        issue(j + NS - 1);
        if (j > jlast) continue;                       // keys above every query of the wave
        const lds_u8 *stk = sm + (j % NS) * D::STAGE;
        const lds_u8 *std_ = stk + C::TILE + wave * 2048;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const s16x4 lo = lds_read_tr16(std_ + dsoff[0] + ks * 256);
            const s16x4 hi = lds_read_tr16(std_ + dsoff[1] + ks * 256);
            const opnd sb = __builtin_bit_cast(opnd, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int d = 0; d < C::NDB; ++d) dqt[d] = MM::mma(tr_frag<DT>(stk, tl, ks, d), sb, dqt[d]);
        }
    }
    if (qrow < T) {
        elem *dyt = static_cast<elem *>(a.dyt) + row0 + qrow;
#pragma unroll
        for (int d = 0; d < C::NDB; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                dyt[(int64_t)(h * DH + c) * a.ldt] = from_f32<DT>(dqt[d][e] * inv_sqrt);
            }
    }
}

}  // namespace

// dK/dV and dQ for the 16-bit dtypes at head_dim 64 / 128 (KL: with the KL term's gradient)
template <int DT, int DH, bool KL>
hipError_t run_bwd_dma_kl(const AttnBwdArgs &a, hipStream_t st) {
    constexpr int NW = 4;
    typedef BwdTiles<DT, DH, NW, KL> C;
    const int T = a.seq_len;
    // per-sequence element offsets are 32-bit
    if ((int64_t)T * a.ldq >= (1ll << 31) || (int64_t)T * a.ldv >= (1ll << 31) ||
        (int64_t)T * a.n_heads * DH >= (1ll << 31))
        return hipErrorInvalidValue;
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
    const float inv_sqrt = 1.f / sqrtf((float)DH);
    const size_t q_lds = (size_t)C::NS_Q * C::Q_STAGE;
    hipError_t e = hipFuncSetAttribute((const void *)attn_bwd_dq_dma_kernel<DT, DH, NW, KL>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)q_lds);
    if (e != hipSuccess) return e;
    const int G = a.n_heads / a.n_kv_heads;
    const uint32_t inv_g = (uint32_t)((1ull << 32) / (uint32_t)G + 1);
    // KW key slices per workgroup, one key block each
    auto dkdv = [&](auto kw_c) -> hipError_t {
        constexpr int KW = decltype(kw_c)::value;
        typedef DkdvCfg<DT, DH, KW, KL> CM;
        hipError_t err = hipFuncSetAttribute((const void *)attn_bwd_dkdv_pipe_kernel<DT, DH, KW, KL>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, CM::LDS);
        if (err != hipSuccess) return err;
        const int nkb = (T + 32 * KW - 1) / (32 * KW);
        attn_bwd_dkdv_pipe_kernel<DT, DH, KW, KL><<<dim3(nkb * a.n_kv_heads * a.batch), dim3(256), CM::LDS, st>>>(
            a, scale_log2, inv_sqrt, nkb, inv_g);
        return hipGetLastError();
    };
    auto dkdv_paired = [&](auto ds_c) -> hipError_t {
        constexpr bool DS = decltype(ds_c)::value;
        const size_t lds = (size_t)C::NS_KV * C::KV_STAGE;
        hipError_t err = hipFuncSetAttribute((const void *)attn_bwd_dkdv_dma_kernel<DT, DH, NW, KL, DS>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess) return err;
        const int nkb = (T + 32 * NW - 1) / (32 * NW), npair = (nkb + 1) / 2;
        attn_bwd_dkdv_dma_kernel<DT, DH, NW, KL, DS><<<dim3(npair * a.n_kv_heads * a.batch), dim3(64 * NW), lds, st>>>(
            a, scale_log2, inv_sqrt, nkb, npair);
        return hipGetLastError();
    };
    // Which form, by the number of pairs of 128-key blocks (the paired form's workgroups; it needs about
    // two per CU).  us of the dK/dV pass, KW = 1 / 2 / 4 / paired, on 256 CUs, bf16 or fp16:
    //   DH 128: 64 pairs - / 187 / 305 / 426, 128 - / 247 / 345 / 456, 192 - / 367 / 372 / 473,
    //   256 - / 498 / 452 / 546, 384 - / - / 649 / 618, 512 - / 977 / 912 / 721
    //   DH 128, KL term: 128 - / 124 / 137, 256 - / 709 / 570, 512 - / 1470 / 1174 (paired: one workgroup per
    //   CU, 256 781, 512 1588)
    //   DH 64: 32 16 / 20 / 33 / 57, 48 22 / 20 / 31 / 41, 128 105 / 75 / 120 / 150, 256 204 / 123 / 140 / 167,
    //   384 145 / 61 / 57 / 67, 768 300 / 127 / 109 / 127, 1536 - / - / 230 / 226
    //   DH 64, KL term: 64 41 / 50 / 83 / 97, 96 44 / 33 / 47 / 54, 192 - / 58 / - / -, 384 177 / 122 / 106 / 88,
    //   768 361 / 257 / 212 / 155
    // (the head grouping and length differ between the rows; KW = 1 runs one workgroup per CU and is
    // taken while its own blocks have a CU each).  The number of ways is the same with the KL term as
    // without, so lambda = 0 gives the squared error's gradients bit for bit.
    const int64_t heads = (int64_t)a.n_kv_heads * a.batch;
    const int64_t pairs = heads * (((T + 127) / 128 + 1) / 2);
    auto run_dkdv = [&]() -> hipError_t {
        if constexpr (DH == 64 || !KL) {
            if (pairs >= (DH == 128 ? 384 : KL ? 257 : 1024))
                return a.ds ? dkdv_paired(std::true_type()) : dkdv_paired(std::false_type());
        }
        if constexpr (DH == 128 || !KL) {
            if (pairs >= (DH == 128 ? 192 : 257)) return dkdv(std::integral_constant<int, 4>());
        }
        if constexpr (DH == 64) {
            if (heads * ((T + 31) / 32) <= 256) return dkdv(std::integral_constant<int, 1>());
        }
        return dkdv(std::integral_constant<int, 2>());
    };
    e = run_dkdv();
    if (e != hipSuccess) return e;
    const int hpw = G % NW == 0 ? NW : G;              // query heads per workgroup
    const int QT = 32 * NW / hpw;
    const int nqt = (T + QT - 1) / QT;
    const int n_ht = a.n_heads / hpw;
    if (a.ds) {   // dQ from the dS the dK pass stored
        typedef DqDsCfg<DT, DH, NW> DC;
        const size_t lds = (size_t)DC::NS * DC::STAGE;
        e = hipFuncSetAttribute((const void *)attn_bwd_dq_ds_kernel<DT, DH, NW>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attn_bwd_dq_ds_kernel<DT, DH, NW><<<dim3(nqt * n_ht * a.batch), dim3(64 * NW), lds, st>>>(
            a, inv_sqrt, hpw, nqt, n_ht);
        return hipGetLastError();
    }
    attn_bwd_dq_dma_kernel<DT, DH, NW, KL><<<dim3(nqt * n_ht * a.batch), dim3(64 * NW), q_lds, st>>>(
        a, scale_log2, inv_sqrt, hpw, nqt, n_ht);
    return hipGetLastError();
}

template <int DT, int DH>
hipError_t run_bwd_dma(const AttnBwdArgs &a, hipStream_t st) {
    if (a.qt) return run_bwd_dma_kl<DT, DH, true>(a, st);
    return run_bwd_dma_kl<DT, DH, false>(a, st);
}

template hipError_t run_bwd_dma<F16, 64>(const AttnBwdArgs &, hipStream_t);
template hipError_t run_bwd_dma<F16, 128>(const AttnBwdArgs &, hipStream_t);
template hipError_t run_bwd_dma<BF16, 64>(const AttnBwdArgs &, hipStream_t);
template hipError_t run_bwd_dma<BF16, 128>(const AttnBwdArgs &, hipStream_t);

}  // namespace jab
