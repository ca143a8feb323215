// gemm.hip -- projection GEMM of the fused QKV weight on the matrix cores.
//
// Paper: Method, "Layer-wise PTQ": y = x W with the QKV projection fused as
// W = [W_Q | W_K | W_V].  Here C[m][n] = sum_k A[m][k] B[n][k] with A = X
// [tokens][d_model] and B = W_hat [R][d_model] (one row per output channel), both
// k-contiguous, accumulated in fp32 and stored in the storage dtype.
//
// Two kernels (launch_project and the other launchers choose by the sizes, see persistent_pays):
//  * gemm_w4p_kernel (16-bit): persistent, 256 x 256 tiles, one workgroup of four waves per CU, each
//    wave 128 x 128 as 4 x 4 blocks of v_mfma_f32_32x32x16_{bf16,f16} (256 accumulator registers; per
//    k-step a wave reads 4 + 4 operand fragments for 16 MFMAs).
//  * gemm_small_kernel (every dtype): 128 x 128 or 64 x 64 tiles, two or three workgroups per CU, for
//    the shapes whose 256-tiles would leave CUs idle, for short K, and for fp32.
// Common to both:
//  * k-tiles go straight from global memory into LDS (buffer_load_dwordx4 ... lds: a scalar resource and
//    k offset, one fixed per-lane offset per instruction, so no vector address arithmetic).  The MUBUF
//    form keeps the LDS counter ordered, so each MFMA waits only for its own fragments.
//  * 16-byte chunks are XOR-swizzled per row so the 16 rows served per LDS cycle hit distinct banks.
//  * The MFMA operands are swapped (B first), so a lane's accumulators hold four consecutive output
//    columns of one row; outputs leave from registers, 16 bytes per lane.
//  * Workgroup ids are remapped so that each XCD (ids congruent mod 8 land on the same XCD) walks a
//    contiguous range of tiles, grouped 8 M-tiles at a time so that concurrently running tiles share A
//    and B panels in that XCD's L2.
//  * A projection's [Q|K] and value tiles go in one launch where that pays (the value tiles with the operands swapped),
//    so that neither part leaves the chip half empty: at 4 x 2048 tokens of d 4096 640 + 128 tiles took
//    3 + 1 rounds of the 256 CUs, together 3 (372 -> 308 us); at 1 x 1999 160 + 32 tiles 189 -> 92 us,
//    of which 54 us went into 2-byte stores of the ragged value tiles.
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "kernels.h"
#include "lds_pipe.h"


namespace jab {
namespace {

// Output modes:
//   OUT_DT : C[m][n] in the storage dtype
//   OUT_F32: C[m][n] = alpha * (A B^T) in fp32
//   OUT_VT : values transposed for the attention kernel, C[m][pos(n)] in the storage
//            dtype, where column n is the token index b*T + t of a batch of sequences of
//            length T; pos(n) = b*Tp + perm(t), Tp = T rounded up to 32, and perm swaps
//            bits 2 and 3 of t inside each block of 32 tokens (the key order in which an
//            MFMA lane consumes softmax probabilities, so each lane's eight keys are one
//            contiguous 16-byte read).
//   OUT_QKV: (persistent kernel) [Q|K] tiles as OUT_DT and value tiles as OUT_VT in one launch
enum { OUT_DT = 0, OUT_F32 = 1, OUT_VT = 2, OUT_QKV = 3 };

// XOR key of LDS row r (16-byte chunks of a row of CPR chunks): rotates the chunk index so the
// 16 rows one LDS cycle serves land on 16 distinct chunk slots
template <int CPR>
__device__ inline int w4_key(int r) {
    if constexpr (CPR == 8) return (r >> 1) & 7;
    else return (r >> 2) & 3;
}

// ---------------------------------------------------------------- small tiles
// One GEMM launch of the small-tile kernel: the product A B^T (rows of A and B k-contiguous) and,
// for a projection (OUT_DT with nv > 0), the transposed values from the nv rows of B that follow
// its first N: C2[r][pos] over the padded token positions of a batch of sequences.
struct SmallArgs {
    const void *A, *B;
    void *C, *C2;
    int M, N, K, lda, ldb, ldc;
    int nv, ldv, seq_T, seq_Tp, n_tok;   // values: rows, row stride, sequence length, padded, batch * padded
    float alpha;
    int pack;                            // OUT_VT: sequences per tile
    int ksplit;                          // OUT_F32: parts of K, part p > 0 at C2 + (p - 1) part_stride
    int64_t part_stride;
    int tiles_m, tiles_n, tiles_vm, tiles_vn;
    const float4 *rtab;                  // rotary embedding (RDH > 0): the transposed table
};

// Tiles of BT x BT, four waves in a 2 x 2 arrangement (BT / 2 square each), for every dtype; the
// shapes whose 256 x 256 tiles would leave CUs idle, the fp32 products, and k-tiles of 32 (CPR 4).
// A projection's [Q|K] tiles and value tiles are work items of one launch: a value tile has the
// weights as its A panel and the tokens as its B panel, in padded token positions, so every block
// of 32 positions lies in one sequence, leaves in 16-byte stores and holds its pad positions'
// zeros.
//
// The k-tiles (CPR 16-byte chunks per row) stream into a ring of NS stages by MUBUF DMA, one barrier
// per k-tile; two workgroups per CU cover each other's start-up, barriers and epilogues.  An operand
// chunk of 16 bytes is one 32x32x16 product of the 16-bit dtypes, and four 32x32x2 products of fp32
// (half h of the wave takes chunk 2 c + h, element s of both halves is step s: a permutation of k
// that A and B share), so fp32 reads LDS 16 bytes at a time too.  For the 16-bit dtypes the products
// and their order are gemm_w4p_kernel's, so the output bits are the same (but for the value tiles
// that kernel starts at another k-tile).
template <int DT, int BT, int CPR>
struct SmallCfg {
    typedef typename Mma<DT>::elem elem;
    static constexpr int ES = (int)sizeof(elem), EPC = 16 / ES, BK = CPR * EPC;
    static constexpr int U = CPR / 2;                      // chunk steps per k-tile
    static constexpr int FB = BT / 64;                     // 32-row blocks per wave and direction
    static constexpr int ROWB = CPR * 16, PANEL = BT * ROWB, STAGE = 2 * PANEL;
    // 64 KiB of stages for the 128-tile (two workgroups per CU), three stages for the 64-tile (three;
    // measured at 8 x 1024 x 768 x 2304 fp16: four stages 61 us, three 54; the 128-tile with two
    // stages of 128-byte rows 42 us, with four or five of 64-byte rows 49, with three of 128 51)
    static constexpr int NS = BT == 64 ? 3 : 65536 / STAGE;
    static constexpr int DPP = BT * CPR / 256, DPW = 2 * DPP;   // DMA instructions per wave: panel, k-tile
    static constexpr int RPI = 64 / CPR;                   // rows per DMA instruction
    static constexpr size_t LDS_BYTES = (size_t)NS * STAGE;
    static_assert(NS >= 2 && BT % 64 == 0 && DPP >= 1, "small-tile configuration");
};

template <int DT>
__device__ inline f32x16 mma_chunk(u32x4 a, u32x4 b, f32x16 c) {
    if constexpr (DT == F32) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t x = a[s], y = b[s];
            c = Mma<F32>::mma(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y), c);
        }
        return c;
    } else {
        typedef typename Mma<DT>::operand opnd;
        return Mma<DT>::mma(__builtin_bit_cast(opnd, a), __builtin_bit_cast(opnd, b), c);
    }
}

// RDH > 0 (128-tile, 16-bit, OUT_DT): the rotary embedding on the [Q|K] tiles, heads of RDH columns, as
// in gemm_w4p_kernel's epilogue.  A pair (c, c + RDH / 2) has to sit in one wave: at RDH 128 wave
// column wc takes the 32-column blocks wc and wc + 2 of the tile instead of 2 wc and 2 wc + 1.
// OUT_VT: the values alone, of sequences that fit in a tile's columns: a tile's columns are the tokens of `pack` whole
// sequences (as many as fit) instead of padded positions, and its outputs are spread to the padded
// positions, zeros between, through LDS.
// WIDE: rows of a panel more than 2^32 bytes apart (offsets_fit), so the loads take 64-bit addresses per lane.
template <int DT, int BT, int CPR, int OUT, int RDH, bool WIDE>
__global__ __launch_bounds__(256, 2) void gemm_small_kernel(SmallArgs g) {
    typedef SmallCfg<DT, BT, CPR> S;
    static_assert(RDH == 0 || (OUT == OUT_DT && BT == 128 && DT != F32 && (RDH == 64 || RDH == 128)), "rotary epilogue");
    constexpr int CB0 = RDH == 128 ? 1 : S::FB, CBJ = RDH == 128 ? 2 : 1;   // column block CB0 wc + CBJ j
    typedef typename S::elem elem;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = wave >> 1, wc = wave & 1, half = lane >> 5, l32 = lane & 31;

    // ---- work item: XCD x (ids congruent to x mod 8) takes a contiguous range; [Q|K] tiles (times
    // the parts of K) first, in groups of eight row tiles, then the value tiles
    const int n_items = gridDim.x, x = blockIdx.x & 7;
    int pid = x * (n_items >> 3) + min(x, n_items & 7) + (blockIdx.x >> 3);
    const int tiles = g.tiles_m * g.tiles_n;
    const bool val = OUT == OUT_VT || (OUT == OUT_DT && pid >= tiles);
    int part = 0, tm = g.tiles_m, tn = g.tiles_n;
    if (val) {
        pid -= OUT == OUT_VT ? 0 : tiles;
        tm = g.tiles_vm;
        tn = g.tiles_vn;
    } else if (OUT == OUT_F32) {
        part = pid / tiles;
        pid -= part * tiles;
    }
    const int group_tiles = 8 * tn;
    const int first_m = (pid / group_tiles) * 8;
    const int gsz = min(tm - first_m, 8);
    const int bm0 = (first_m + (pid % group_tiles) % gsz) * BT;
    const int bn0 = (pid % group_tiles) / gsz * (OUT == OUT_VT ? g.pack * g.seq_T : BT);   // OUT_VT: a token
    const int nkt = g.K / S::BK;
    const int kt0 = part * nkt / g.ksplit, nk = (part + 1) * nkt / g.ksplit - kt0;

    // ---- panels.  Value tile: A panel = rows bm0.. of the value weights, B panel = the tokens of
    // padded positions bn0..; rows past an edge (and pad positions) read a valid row, for outputs
    // that are not stored (or stored as zero)
    const int lda = val ? g.ldb : g.lda, ldb = val ? g.lda : g.ldb;
    const elem *Ap = static_cast<const elem *>(val ? g.B : g.A) + (val ? (int64_t)g.N * lda : 0);
    const elem *Bp = static_cast<const elem *>(val ? g.A : g.B);
    const int rows_a = val ? g.nv : g.M;
    const int n_pos = OUT == OUT_VT ? g.M : g.n_tok;
    auto token = [&](int n) -> int {          // source row of padded position n
        if constexpr (OUT == OUT_VT) return n;
        const int s = n / g.seq_Tp;
        return s * g.seq_T + min(n - s * g.seq_Tp, g.seq_T - 1);
    };
    const int rb0 = val ? token(min(bn0, n_pos - 1)) : bn0;
    const elem *Ab = Ap + (int64_t)bm0 * lda + (int64_t)kt0 * S::BK, *Bb = Bp + (int64_t)rb0 * ldb + (int64_t)kt0 * S::BK;
    const i32x4 rsA = buffer_rsrc(Ab), rsB = buffer_rsrc(Bb);
    typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type off_t;
    off_t voffA[S::DPP], voffB[S::DPP];
#pragma unroll
    for (int i = 0; i < S::DPP; ++i) {
        const int r = S::RPI * (wave + 4 * i) + lane / CPR, c = (lane % CPR) ^ w4_key<CPR>(r);
        const int ra = min(bm0 + r, rows_a - 1) - bm0;
        const int rb = (val ? token(min(bn0 + r, n_pos - 1)) : min(bn0 + r, g.N - 1)) - rb0;
        voffA[i] = (off_t)ra * (off_t)lda * (off_t)S::ES + (off_t)(c * 16);
        voffB[i] = (off_t)rb * (off_t)ldb * (off_t)S::ES + (off_t)(c * 16);
    }
    auto issue = [&](int kt, int slot) {      // k-tile kt (past the end: the last again, never read)
        const off_t kk = (off_t)min(kt, nk - 1) * (off_t)(S::BK * S::ES);
        unsigned char *st = smem + slot * S::STAGE;
#pragma unroll
        for (int i = 0; i < S::DPP; ++i) {
            if constexpr (WIDE) {
                lds_dma16(reinterpret_cast<const char *>(Ab) + voffA[i] + kk, st + (wave + 4 * i) * 1024);
                lds_dma16(reinterpret_cast<const char *>(Bb) + voffB[i] + kk, st + S::PANEL + (wave + 4 * i) * 1024);
            } else {
                buffer_dma16(rsA, voffA[i], (int)kk, st + (wave + 4 * i) * 1024);
                buffer_dma16(rsB, voffB[i], (int)kk, st + S::PANEL + (wave + 4 * i) * 1024);
            }
        }
    };

    // ---- fragment reads: row l32 of a 32-row block, logical chunk 2 u + half
    const int key = w4_key<CPR>(l32);
    uint32_t rda[S::U], rdb[S::U];
#pragma unroll
    for (int u = 0; u < S::U; ++u) {
        const int pc = (2 * u + half) ^ key;
        rda[u] = (uint32_t)((wr * (BT / 2) + l32) * S::ROWB + pc * 16);
        rdb[u] = (uint32_t)(S::PANEL + (wc * CB0 * 32 + l32) * S::ROWB + pc * 16);
    }
    f32x16 acc[S::FB][S::FB];
#pragma unroll
    for (int i = 0; i < S::FB; ++i)
#pragma unroll
        for (int j = 0; j < S::FB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll
    for (int s0 = 0; s0 < S::NS - 1; ++s0) issue(s0, s0);
    int slot = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // k-tile kt has landed for every wave, and every wave has read k-tile kt - 1, whose slot
        // takes k-tile kt + NS - 1
        wait_lgkm0();
        wait_vmcnt<(S::NS - 2) * S::DPW>();
        raw_barrier();
        issue(kt + S::NS - 1, slot == 0 ? S::NS - 1 : slot - 1);
        const unsigned char *st = smem + slot * S::STAGE;
        u32x4 fa[S::U][S::FB], fb[S::U][S::FB];
#pragma unroll
        for (int u = 0; u < S::U; ++u)
#pragma unroll
            for (int i = 0; i < S::FB; ++i) {
                fa[u][i] = *reinterpret_cast<const u32x4 *>(st + rda[u] + i * 32 * S::ROWB);
                fb[u][i] = *reinterpret_cast<const u32x4 *>(st + rdb[u] + i * CBJ * 32 * S::ROWB);
            }
#pragma unroll
        for (int u = 0; u < S::U; ++u)
#pragma unroll
            for (int i = 0; i < S::FB; ++i)
#pragma unroll
                for (int j = 0; j < S::FB; ++j) acc[i][j] = mma_chunk<DT>(fb[u][j], fa[u][i], acc[i][j]);
        slot = slot == S::NS - 1 ? 0 : slot + 1;
    }
    wait_vmcnt<0>();

    if constexpr (OUT == OUT_VT) {
        // the tile as [BT value rows][BT tokens] in LDS (16-byte chunks XOR-swizzled per row), then whole rows of
        // padded positions: positions 16 p + 8 h + 4 b + 0..3 of a sequence hold tokens 16 p + 8 b + 4 h + 0..3
        static_assert((size_t)BT * BT * S::ES <= S::LDS_BYTES, "the tile in the ring's LDS");
        constexpr int CB = BT / S::EPC;                    // chunks per row
        raw_barrier();                                     // every wave has left the ring
        auto at = [&](int row, int col) -> elem * {
            const int ch = (col / S::EPC) ^ (row & (CB < 16 ? CB - 1 : 15));
            return reinterpret_cast<elem *>(smem) + row * BT + ch * S::EPC + col % S::EPC;
        };
#pragma unroll
        for (int i = 0; i < S::FB; ++i)
#pragma unroll
            for (int j = 0; j < S::FB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    *at(wr * (BT / 2) + 32 * i + l32, 32 * (S::FB * wc + j) + 8 * (e >> 2) + 4 * half + (e & 3)) =
                        from_f32<DT>(acc[i][j][e]);
        __syncthreads();
        const int T = g.seq_T, seq0 = bn0 / T, ns = min(g.pack, g.M / T - seq0);
        const uint32_t cps = (uint32_t)g.seq_Tp / S::EPC;  // chunks of a sequence's positions
        for (int r = wave; r < min(BT, rows_a - bm0); r += 4) {
            elem *crow = static_cast<elem *>(g.C2) + (int64_t)(bm0 + r) * g.ldv + (int64_t)seq0 * g.seq_Tp;
            for (uint32_t c = lane; c < ns * cps; c += 64) {
                const int sq = (int)(c / cps), p0 = (int)(c % cps) * S::EPC;
                elem v[S::EPC];
#pragma unroll
                for (int k = 0; k < S::EPC; ++k) {
                    const int t = vt_perm(p0 + k);
                    v[k] = t < T ? *at(r, sq * T + t) : elem(0);
                }
                u32x4 o;
                __builtin_memcpy(&o, v, 16);
                *reinterpret_cast<u32x4 *>(crow + (int64_t)c * S::EPC) = o;
            }
        }
        return;
    }

    // ---- epilogue from registers: acc[i][j][4 q + t] = C[row][col + t], row = 32 i + l32, col =
    // 32 (CB0 wc + CBJ j) + 8 q + 4 half (tile coordinates); 16 bytes per lane and store
    if constexpr (RDH > 0) {
        if (!val) {
#pragma unroll
            for (int i = 0; i < S::FB; ++i) {
                const int t = min(bm0 + wr * (BT / 2) + 32 * i + l32, g.M - 1) % g.seq_T;
#pragma unroll
                for (int e2 = 0; e2 < 8; ++e2) {      // elements 2 e2 and 2 e2 + 1 of a block: one float4
                    const int q = (RDH == 128 ? 16 * wc : 0) + 4 * (e2 >> 1) + 2 * half + (e2 & 1);
                    const float4 cs = g.rtab[(int64_t)q * g.seq_T + t];
                    const float a0 = acc[i][0][2 * e2], b0 = acc[i][1][2 * e2];
                    const float a1 = acc[i][0][2 * e2 + 1], b1 = acc[i][1][2 * e2 + 1];
                    acc[i][0][2 * e2] = __builtin_fmaf(a0, cs.x, -(b0 * cs.y));
                    acc[i][1][2 * e2] = __builtin_fmaf(b0, cs.x, a0 * cs.y);
                    acc[i][0][2 * e2 + 1] = __builtin_fmaf(a1, cs.z, -(b1 * cs.w));
                    acc[i][1][2 * e2 + 1] = __builtin_fmaf(b1, cs.z, a1 * cs.w);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < S::FB; ++i) {
        const int row = bm0 + wr * (BT / 2) + 32 * i + l32;
        if (row >= rows_a) continue;
#pragma unroll
        for (int j = 0; j < S::FB; ++j) {
            const int colb = bn0 + 32 * (CB0 * wc + CBJ * j);
            if (val) {
                if constexpr (OUT == OUT_DT) {
                    if (colb >= g.n_tok) continue;
                    const int left = g.seq_T - colb % g.seq_Tp;      // tokens of the block
                    elem *crow = static_cast<elem *>(g.C2) + (int64_t)row * g.ldv + colb;
                    float v[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        v[e] = 8 * (e >> 2) + 4 * half + (e & 3) < left ? acc[i][j][e] : 0.f;
                    // bits 2 and 3 of the token exchanged: tokens 16 p + 8 b + 4 half + 0..3 sit at
                    // positions 16 p + 8 half + 4 b + 0..3
                    if constexpr (DT == F32) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<f32x4 *>(crow + 16 * (q >> 1) + 8 * half + 4 * (q & 1)) =
                                f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                    } else {
#pragma unroll
                        for (int p = 0; p < 2; ++p)
                            *reinterpret_cast<u32x4 *>(crow + 16 * p + 8 * half) =
                                u32x4{pack2<DT>(v[8 * p], v[8 * p + 1]), pack2<DT>(v[8 * p + 2], v[8 * p + 3]),
                                      pack2<DT>(v[8 * p + 4], v[8 * p + 5]), pack2<DT>(v[8 * p + 6], v[8 * p + 7])};
                    }
                }
            } else if constexpr (OUT == OUT_F32 || DT == F32) {
                const float al = OUT == OUT_F32 ? g.alpha : 1.f;
                float *base = static_cast<float *>(OUT == OUT_F32 && part ? g.C2 : g.C) +
                              (OUT == OUT_F32 && part ? (part - 1) * g.part_stride : 0) + (int64_t)row * g.ldc;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = colb + 8 * q + 4 * half;
                    const f32x4 v = f32x4{al * acc[i][j][4 * q], al * acc[i][j][4 * q + 1], al * acc[i][j][4 * q + 2],
                                          al * acc[i][j][4 * q + 3]};
                    if (col + 4 <= g.N) *reinterpret_cast<f32x4 *>(base + col) = v;
                }
            } else {
                elem *crow = static_cast<elem *>(g.C) + (int64_t)row * g.ldc;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    uint32_t a0 = pack2<DT>(acc[i][j][8 * p], acc[i][j][8 * p + 1]);
                    uint32_t a1 = pack2<DT>(acc[i][j][8 * p + 2], acc[i][j][8 * p + 3]);
                    uint32_t b0 = pack2<DT>(acc[i][j][8 * p + 4], acc[i][j][8 * p + 5]);
                    uint32_t b1 = pack2<DT>(acc[i][j][8 * p + 6], acc[i][j][8 * p + 7]);
                    // exchange halves: each lane then holds columns 16 p + 8 half + 0..7.  The lanes
                    // of a row (l32 of both halves) are active together
                    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\ts_nop 1"
                                 : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
                    const int col = colb + 16 * p + 8 * half;
                    if (col + 8 <= g.N) *reinterpret_cast<u32x4 *>(crow + col) = u32x4{a0, a1, b0, b1};
                }
            }
        }
    }
}

// The persistent kernel: one workgroup per CU walks the tiles blockIdx.x, + gridDim.x, ... (in the same remapped order).  The
// operand that streams the tokens has an LDS ring of three k-tiles, the weights one of two (160 KiB
// at k-tiles of 64).  The rings run on across tiles: the refills of a tile's last stages bring the
// next tile's first two k-tiles, and the last stage's fragment reads already fetch its first k-step, so
// between two tiles only the epilogue remains; it stores from registers (16 bytes per lane) while
// the next tile's loads are in flight.  A tile is always whole: the last tile of a ragged M (N) is
// moved back to end at M (N), so the per-lane load offsets are the same for every tile (rows or
// columns it shares with its neighbour are written twice with the same values, the same products
// summed in the same order).  Needs M, N >= 256, at least three k-tiles, and for OUT_VT T a multiple
// of 32.
// RDH > 0 (storage-dtype output only): every output column belongs to a query or key head of
// RDH columns, rotated by the rotary embedding in the epilogue (see below).
// OUT_F32: alpha (A B^T) in fp32, K split in ksplit equal parts (work item w: tile w mod tiles,
// part w / tiles, written to Cp for part 0 and Cp2 for part 1).
// queue (grid a multiple of 8, at least six k-tiles per work item; else null and the static order
// above): the work items after the first are taken at run time, so that the XCDs that run faster
// take more of them.  XCD x (workgroups congruent to x mod 8) owns the items congruent to x mod 8
// (the static order's, so the L2 of an XCD still sees its own panels) and takes them in order
// through the counter queue[x]; once its own are gone it takes another XCD's (queue[(x + k) % 8],
// k = 1 .. 7).  Lane 0 of wave 0 takes the item that follows the current one at the start of the
// current one; it reaches the other waves through queue[16 + 2 b + parity] (workgroup b), stored
// after stage 0 and read after stage 1's barrier, long before stage nk - 2 needs it.
// queue[8] counts the workgroups that are done: the last one resets the counters, so each launch
// starts from zero.  No wait depends on another workgroup.  A work item is computed whole by one
// workgroup, so the output does not depend on the order.
template <int DT, int OUT, int CPR, int RDH = 0>
__global__ __launch_bounds__(256, 1) void gemm_w4p_kernel(const void *__restrict__ Ap, const void *__restrict__ Bp,
                                                          void *__restrict__ Cp, int M, int N, int K, int lda,
                                                          int ldb, int ldc, int tiles_m, int tiles_n, int seq_T,
                                                          int seq_Tp, int n_work, const float4 *__restrict__ rtab,
                                                          float alpha, int ksplit, void *__restrict__ Cp2,
                                                          int *__restrict__ queue_arg, int nv, int ldv, int n_tok) {
    int *const queue = OUT == OUT_QKV ? nullptr : queue_arg;   // its launches have few items per workgroup
    static_assert(RDH == 0 || ((OUT == OUT_DT || OUT == OUT_QKV) && (RDH == 64 || RDH == 128)), "rotary epilogue");
    typedef typename Mma<DT>::elem elem;
    typedef typename Mma<DT>::operand opnd;
    constexpr int BK = CPR * 8;
    constexpr int U = BK / 16;
    constexpr int ROWB = CPR * 16;
    constexpr int HALF = 256 * ROWB;                  // one operand's k-tile
    constexpr int DPW = 2 * 256 * CPR / 64 / 4;
    constexpr int DPA = DPW / 2;
    constexpr int RPI = 64 / CPR;
    // The operand that streams the tokens (A = X for the row-major outputs, B = X for the transposed
    // value output) has a ring of three k-tiles, the other (the weights) one of two: LDS holds the
    // deep ring's slots 0..2, then the shallow ring's 0..1.
    constexpr bool DA = OUT != OUT_VT;
    constexpr int ABASE = DA ? 0 : 3 * HALF, BBASE = DA ? 3 * HALF : 0;
    static_assert(U >= 4 && DPW == 16, "refill schedule");
    extern __shared__ __align__(16) unsigned char smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wr = wave >> 1, wc = wave & 1;
    const int half = lane >> 5, l32 = lane & 31;
    const int nk = K / BK / ksplit;                   // k-tiles per work item

    // a work item: its tile's corner, its first k-tile, its output and the buffer resources of its
    // A and B panels (all wave-uniform)
    struct Tile {
        int bm0, bn0, k0, ks;
        bool val;                                     // OUT_QKV: a tile of the transposed values
        void *out;
        i32x4 rsA, rsB;
    };
    // OUT_QKV: the source row of padded token position n (a pad position reads a valid row)
    auto token = [&](int n) -> int {
        const int sq = n / seq_Tp;
        return sq * seq_T + min(n - sq * seq_Tp, seq_T - 1);
    };
    auto decode = [&](int work, Tile &t) {
        int pid = work;
        if ((n_work & 7) == 0) pid = (pid & 7) * (n_work >> 3) + (pid >> 3);
        t.val = OUT == OUT_QKV && pid >= tiles_m * tiles_n;
        if constexpr (OUT == OUT_QKV) {
            if (t.val) {                              // A: the value weights (rows N.. of B), B: the tokens
                pid -= tiles_m * tiles_n;
                const int tvm = (nv + 255) >> 8;
                t.bm0 = min((pid % tvm) * 256, nv - 256);
                t.bn0 = min((pid / tvm) * 256, n_tok - 256);
                t.k0 = t.ks = 0;
                t.out = Cp2;
                t.rsA = buffer_rsrc(static_cast<const char *>(Bp) + (int64_t)(N + t.bm0) * ldb * (int64_t)sizeof(elem));
                t.rsB = buffer_rsrc(static_cast<const char *>(Ap) + (int64_t)token(t.bn0) * lda * (int64_t)sizeof(elem));
                return;
            }
        }
        const int part = pid / (tiles_m * tiles_n);
        pid -= part * tiles_m * tiles_n;
        t.k0 = part * nk;
        t.out = part ? Cp2 : Cp;
        const int group_tiles = 8 * tiles_n;
        const int first_m = (pid / group_tiles) * 8;
        const int gsz = min(tiles_m - first_m, 8);
        const int pm = first_m + (pid % group_tiles) % gsz;
        const int pn = (pid % group_tiles) / gsz;
        // transposed value output: the k-loop of a tile starts at k-tile ks and wraps around, ks
        // different for the tiles of a set that share an A or a B panel (measured: 1.67 -> 1.62 ms
        // at 1024 x 262144 x 4096; no gain for the row-major output).  Only when every tile is
        // whole: a ragged last tile moved back over its neighbour must sum the shared elements in the
        // same order as the neighbour does (both write them).
        t.ks = OUT == OUT_VT && M % 256 == 0 && N % 256 == 0 ? ((pm & 7) + (pn & 3)) % nk : 0;
        t.bm0 = min(pm * 256, M - 256);
        t.bn0 = min(pn * 256, N - 256);
        t.rsA = buffer_rsrc(static_cast<const char *>(Ap) + (int64_t)t.bm0 * lda * (int64_t)sizeof(elem));
        t.rsB = buffer_rsrc(static_cast<const char *>(Bp) + (int64_t)t.bn0 * ldb * (int64_t)sizeof(elem));
    };
    // DMA instruction d < DPA fills rows RPI (wave + 4 d) .. + RPI - 1 of the A part (d >= DPA: of
    // the B part); lane i writes row + i / CPR, physical chunk i % CPR = logical chunk ^ key(row)
    uint32_t voffA[DPA], voffB[DPA];
#pragma unroll
    for (int i = 0; i < DPA; ++i) {
        const int r = RPI * (wave + 4 * i) + lane / CPR, pc = lane % CPR;
        const int c = pc ^ w4_key<CPR>(r);
        voffA[i] = (uint32_t)r * (uint32_t)lda * 2u + c * 16u;
        voffB[i] = (uint32_t)r * (uint32_t)ldb * 2u + c * 16u;
    }
    // OUT_QKV (lda == ldb) with sequences that are not whole blocks of 32 tokens: a value tile's rows
    // of X skip at the sequence ends, so its per-lane offsets are its own; they are set for the first
    // tile and then, inside stage nk - 2, for the next one (before its first B loads)
    const bool ragged = OUT == OUT_QKV && seq_T != seq_Tp;
    auto set_voffB = [&](const Tile &t) {
        if constexpr (OUT == OUT_QKV) {
            // row 8 wave + 32 i + lane / 8, whose chunk key does not depend on i.  The lane id goes
            // through an opaque copy, so that nothing here is kept in registers between the tiles
            static_assert(CPR == 8, "rows of eight chunks");
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int r0 = 8 * wave + (ln >> 3), c16 = ((ln & 7) ^ w4_key<CPR>(r0)) * 16;
            const int base = t.val ? token(t.bn0) : 0;
#pragma unroll
            for (int i = 0; i < DPA; ++i) {
                const int rr = t.val ? token(t.bn0 + r0 + 32 * i) - base : r0 + 32 * i;
                voffB[i] = (uint32_t)rr * (uint32_t)ldb * 2u + c16;
            }
        }
    };
    // DMA instruction d of k-tile ktile into the operand's ring slot `slot`
    auto issue = [&](const Tile &t, int d, int ktile, int slot) {
        int kx = ktile + t.ks;
        if (kx >= nk) kx -= nk;
        const int kk = (int)((uint32_t)(t.k0 + kx) * (BK * 2u));
        if (d < DPA) buffer_dma16(t.rsA, voffA[d], kk, smem + ABASE + slot * HALF + (wave + 4 * d) * 1024);
        else buffer_dma16(t.rsB, voffB[d - DPA], kk, smem + BBASE + slot * HALF + (wave + 4 * (d - DPA)) * 1024);
    };
    // the deep (D) and shallow (S) operands' instruction numbers
    auto dsn = [&](int i) { return DA ? i : DPA + i; };
    auto ssn = [&](int i) { return DA ? DPA + i : i; };

    const int key = w4_key<CPR>(l32);
    uint32_t rda[U], rdb[U];
#pragma unroll
    for (int ks = 0; ks < U; ++ks) {
        const int pc = (2 * ks + half) ^ key;
        rda[ks] = (uint32_t)((wr * 128 + l32) * ROWB + pc * 16);
        rdb[ks] = (uint32_t)((wc * 128 + l32) * ROWB + pc * 16);
    }
    opnd fa[2][4], fb[2][4];
    // fragment read r of k-step ks from the deep slot ds and the shallow slot ss
    auto rd = [&](int r, int ds, int ss, int ks, int buf) {
        const unsigned char *ab = smem + ABASE + (DA ? ds : ss) * HALF;
        const unsigned char *bb = smem + BBASE + (DA ? ss : ds) * HALF;
        if (r == 0) fa[buf][0] = __builtin_bit_cast(opnd, *(const u32x4 *)(ab + rda[ks]));
        else if (r <= 4) fb[buf][r - 1] = __builtin_bit_cast(opnd, *(const u32x4 *)(bb + rdb[ks] + (r - 1) * 32 * ROWB));
        else fa[buf][r - 4] = __builtin_bit_cast(opnd, *(const u32x4 *)(ab + rda[ks] + (r - 4) * 32 * ROWB));
    };

    const bool q0l0 = queue != nullptr && wave == 0 && lane == 0;
    // the next work item from the queue, or -1
    auto grab = [&]() -> int {
        const int x = blockIdx.x & 7, first = gridDim.x >> 3;   // first items of each XCD: static
        for (int k = 0; k < 8; ++k) {
            const int xx = (x + k) & 7;
            const int i = atomicAdd(queue + xx, 1) + first;
            if (i < ((n_work - xx + 7) >> 3)) return xx + 8 * i;
        }
        return -1;
    };
    auto finish = [&]() {
        if (q0l0 && atomicAdd(queue + 8, 1) == (int)gridDim.x - 1)
            for (int x = 0; x <= 8; ++x) atomicExch(queue + x, 0);
    };
    int work = blockIdx.x;
    if (work >= n_work) {
        finish();
        return;
    }
    Tile cur, nxt;
    decode(work, cur);
    bool has_next;
    if (queue) {                                      // resolved before stage 2
        has_next = false;
        nxt = cur;
    } else {
        has_next = work + (int)gridDim.x < n_work;
        // after the last tile the refills re-load its first k-tiles (in bounds, never read)
        if (has_next) decode(work + gridDim.x, nxt);
        else nxt = cur;
    }
    int par = 0;                                      // the queue's mailbox slot of this tile

    if (ragged) set_voffB(cur);
    // prologue, as a previous tile's last stages leave the rings: k-tile 0 of both operands, k-tile
    // 1 of the deep one and the first half of the shallow one's (its second half goes out in the
    // first k-step of stage 0); then k-tile 0 has landed
#pragma unroll
    for (int d = 0; d < DPW; ++d) issue(cur, d, 0, 0);
#pragma unroll
    for (int i = 0; i < DPA; ++i) issue(cur, dsn(i), 1, 1);
#pragma unroll
    for (int i = 0; i < DPA / 2; ++i) issue(cur, ssn(i), 1, 1);
    wait_vmcnt<DPA + DPA / 2>();
    raw_barrier();
#pragma unroll
    for (int r = 0; r < 8; ++r) rd(r, 0, 0, 0, 0);

    f32x16 acc[4][4];
    int dslot = 0, sslot = 0;                         // the stage's deep and shallow ring slots
    for (;;) {
        // Stage kt of the current tile (FIRST: kt = 0, whose first k-step starts the accumulators
        // from zero).  k-step u: 16 MFMAs, a fragment read of the next k-step every other MFMA slot, and
        // refill loads; one barrier per stage, before its last k-step, by when every wave has read (and
        // waited for) the stage's other fragments and the next stage has landed.  The refills past the
        // tile's last k-tile load the next tile's first ones.
        // Refills, one DMA instruction every fourth MFMA slot: k-step 0 sends the second half of
        // the shallow operand's k-tile kt + 1 (into the slot stage kt - 1 left), k-steps 1 and 2 the
        // deep operand's k-tile kt + 2 (into the deep slot stage kt - 1 left), the last k-step,
        // after the barrier, the first half of the shallow operand's k-tile kt + 2 (into this
        // stage's shallow slot).  The deep loads have about two stages to land, the shallow ones
        // one; the barrier's wait leaves the 8 deep loads of k-tile kt + 2 in flight.  (Measured at
        // [Q|K] 262144 x 5120 x 4096 on one box: two-stage rings with the refill spread over 2
        // k-steps 8.12 ms, this 7.93 ms.)
        auto stage = [&](int kt, auto first_c) {
            constexpr bool FIRST = decltype(first_c)::value;
            const int nd = dslot == 2 ? 0 : dslot + 1, ns = sslot ^ 1;
            const int rd_ = dslot == 0 ? 2 : dslot - 1;    // deep slot of k-tile kt + 2 (= kt - 1)
            const bool n2 = kt + 2 >= nk, n1 = kt + 1 >= nk;
            const Tile &t2 = n2 ? nxt : cur;
            const Tile &t1 = n1 ? nxt : cur;
            const int k2 = n2 ? kt + 2 - nk : kt + 2, k1 = n1 ? kt + 1 - nk : kt + 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int cb = u & 1;
                if constexpr (OUT == OUT_QKV && !FIRST)
                    if (u == 1 && ragged && kt == nk - 2) set_voffB(nxt);
                if (u == U - 1) {
                    wait_lgkm0();
                    wait_vmcnt<DPA>();
                    raw_barrier();
                }
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    const int i = m >> 2, j = m & 3;
                    if (FIRST && u == 0) acc[i][j] = Mma<DT>::mma(fb[cb][j], fa[cb][i], f32x16{});
                    else acc[i][j] = Mma<DT>::mma(fb[cb][j], fa[cb][i], acc[i][j]);
                    if ((m & 1) == 0) {
                        if (u < U - 1) rd(m >> 1, dslot, sslot, u + 1, cb ^ 1);
                        else rd(m >> 1, nd, ns, 0, cb ^ 1);
                    }
                    if ((m & 3) == 0) {
                        if (u == 0) issue(t1, ssn(DPA / 2 + (m >> 2)), k1, ns);
                        else if (u <= 2) issue(t2, dsn(4 * (u - 1) + (m >> 2)), k2, rd_);
                        else if (u == U - 1) issue(t2, ssn(m >> 2), k2, sslot);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            dslot = nd;
            sslot = ns;
        };
        // rotary epilogue: the table entries of step 2 i + jp (row block i, pairs jp of the wave's
        // columns): this lane's position and 16 of its head columns, tb[4 pp + k] holds the (cos, sin)
        // of columns (32 jp for RDH 128) + 16 pp + 8 (k / 2) + 4 half + 2 (k % 2) and + 1, from the
        // transposed table rtab[q][t], so a load's 32 positions are one contiguous run; step 0's are
        // loaded before the tile's last stage, each next step's while the previous one is rotated
        f32x4 tab[2][8];
        auto tload = [&](int st, f32x4 (&tb)[8]) {
            if constexpr (RDH > 0) {
                const int t = (cur.bm0 + wr * 128 + 32 * (st >> 1) + l32) % seq_T, jp = st & 1;
#pragma unroll
                for (int pp = 0; pp < 2; ++pp)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int q = (RDH == 128 ? 16 * jp : 0) + 8 * pp + 4 * (k >> 1) + 2 * half + (k & 1);
                        tb[4 * pp + k] = __builtin_bit_cast(f32x4, rtab[(int64_t)q * seq_T + t]);
                    }
            }
        };
        int taken = 0;
        if (q0l0) taken = grab();
        int *mbox = queue ? queue + 16 + 2 * blockIdx.x + par : nullptr;
        stage(0, std::integral_constant<bool, true>());
        // The grab's result has returned by stage 0's barrier wait (vector-memory operations
        // complete in issue order).  The store goes out before stage 1's refills, so the wait at
        // stage 1's barrier, which leaves only the last DPA of those in flight, has completed it.
        if (q0l0) __hip_atomic_store(mbox, taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // after stage 1's barrier: the next work item (an agent-scope load, past the CU's cache)
        auto next_item = [&]() {
            const int w = __builtin_amdgcn_readfirstlane(__hip_atomic_load(mbox, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            has_next = w >= 0;
            if (has_next) {
                work = w;
                decode(w, nxt);
            }
        };
        int kt = 1;                                   // nk >= 2
        if constexpr (RDH > 0) {
            while (kt < nk - 1) {
                if (queue && kt == 2) next_item();
                stage(kt++, std::integral_constant<bool, false>());
            }
            tload(0, tab[0]);
            stage(kt, std::integral_constant<bool, false>());
        } else {
            do {
                if (queue && kt == 2) next_item();
                stage(kt, std::integral_constant<bool, false>());
            } while (++kt < nk);
        }

        // ---- epilogue from registers.  acc[i][j][4 g + t] = C[row][col + t], row = wr*128 + 32 i +
        // l32, col = wc*128 + 32 j + 8 g + 4 half (tile coordinates).  Accumulators are read one
        // block at a time (explicit reads keep the compiler from copying all of them out at once).
        if constexpr (OUT == OUT_F32) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = cur.bm0 + wr * 128 + 32 * i + l32;
                float *crow = static_cast<float *>(cur.out) + (int64_t)row * ldc;
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[i][j][4 * g + e]));
                        const int col = cur.bn0 + wc * 128 + 32 * j + 8 * g + 4 * half;
                        *reinterpret_cast<f32x4 *>(crow + col) =
                            f32x4{alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]};
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
        } else {
            auto store_rope = [&]() {
              if constexpr (RDH > 0) {
            // Rotary embedding of the half-split pairs (column c of a head with c + RDH/2), token
            // row % seq_T.  A wave's 128 columns start on a head boundary (tiles start at multiples
            // of 256 or end at N, N a multiple of RDH), so a pair sits in one lane: blocks j and
            // j + 2 (RDH 128) or j and j + 1 (RDH 64), the same register.  The fp32 accumulators
            // turn by the fp32 (cos, sin) of the table (formed in fp64),
            // (a, b) -> (fma(a, cos, -b sin), fma(b, cos, a sin)), then round to the dtype once.
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = cur.bm0 + wr * 128 + 32 * i + l32;
                elem *crow = static_cast<elem *>(cur.out) + (int64_t)row * ldc;
#pragma unroll
                for (int jp = 0; jp < 2; ++jp) {
                    if (2 * i + jp + 1 < 8) tload(2 * i + jp + 1, tab[(jp + 1) & 1]);
                    const int j1 = RDH == 128 ? jp : 2 * jp, j2 = RDH == 128 ? jp + 2 : 2 * jp + 1;
#pragma unroll
                    for (int pp = 0; pp < 2; ++pp) {
                        // elements 8 pp + e: head columns (32 jp for RDH 128) + 16 pp + 8 (e / 4) +
                        // 4 half + e % 4; tq[e / 2] holds the (cos, sin) of elements 2 (e / 2) and + 1
                        const f32x4 *tq = &tab[jp][4 * pp];
                        float v1[8], v2[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v1[e]) : "a"(acc[i][j1][8 * pp + e]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v2[e]) : "a"(acc[i][j2][8 * pp + e]));
                        }
                        uint32_t o1[4], o2[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            float y1[2], y2[2];
#pragma unroll
                            for (int h2 = 0; h2 < 2; ++h2) {
                                const int e = 2 * k + h2;
                                const f32x4 q = tq[e >> 1];
                                const float cs = q[2 * (e & 1)], sn = q[2 * (e & 1) + 1];
                                y1[h2] = __builtin_fmaf(v1[e], cs, -(v2[e] * sn));
                                y2[h2] = __builtin_fmaf(v2[e], cs, v1[e] * sn);
                            }
                            o1[k] = pack2<DT>(y1[0], y1[1]);
                            o2[k] = pack2<DT>(y2[0], y2[1]);
                        }
                        // as the plain epilogue: exchange halves so each lane stores 8 consecutive columns
                        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\ts_nop 1"
                                     : "+v"(o1[0]), "+v"(o1[2]), "+v"(o1[1]), "+v"(o1[3]));
                        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\ts_nop 1"
                                     : "+v"(o2[0]), "+v"(o2[2]), "+v"(o2[1]), "+v"(o2[3]));
                        const int cb1 = cur.bn0 + wc * 128 + 32 * j1, cb2 = cur.bn0 + wc * 128 + 32 * j2;
                        *reinterpret_cast<u32x4 *>(crow + cb1 + 16 * pp + 8 * half) = u32x4{o1[0], o1[1], o1[2], o1[3]};
                        *reinterpret_cast<u32x4 *>(crow + cb2 + 16 * pp + 8 * half) = u32x4{o2[0], o2[1], o2[2], o2[3]};
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
              }
            };
            // the storage-dtype tile (TR false) or the transposed values (TR true)
            auto store_tile = [&](auto tr_c) {
                constexpr bool TR = decltype(tr_c)::value;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = cur.bm0 + wr * 128 + 32 * i + l32;
                    elem *crow = static_cast<elem *>(cur.out) + (int64_t)row * (TR && OUT == OUT_QKV ? ldv : ldc);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int colb = cur.bn0 + wc * 128 + 32 * j;
#pragma unroll
                        for (int pp = 0; pp < 2; ++pp) {
                            float v[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[i][j][8 * pp + e]));
                            if constexpr (TR && OUT == OUT_QKV) {
                                // pad positions hold zeros (colb is a padded position)
                                if (ragged) {
                                    const int left = seq_T - colb % seq_Tp - 16 * pp - 4 * half;
#pragma unroll
                                    for (int e = 0; e < 8; ++e) v[e] = 8 * (e >> 2) + (e & 3) < left ? v[e] : 0.f;
                                }
                            }
                            uint32_t a0 = pack2<DT>(v[0], v[1]), a1 = pack2<DT>(v[2], v[3]);
                            uint32_t b0 = pack2<DT>(v[4], v[5]), b1 = pack2<DT>(v[6], v[7]);
                            int64_t dcol;
                            if constexpr (!TR) {
                                // a lane holds columns 16 pp + 4 half + 0..3 (a) and 16 pp + 8 + 4 half +
                                // 0..3 (b); exchanging a of the upper half-wave with b of the lower one
                                // leaves each lane eight consecutive columns, 16 pp + 8 half + 0..7
                                asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\ts_nop 1"
                                             : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
                                dcol = colb + 16 * pp + 8 * half;
                            } else {
                                // tokens 16 pp + 4 half + 0..3 and 16 pp + 8 + 4 half + 0..3 of the
                                // 32-token block colb: with bits 2 and 3 exchanged they are the eight
                                // consecutive positions 16 pp + 8 half + 0..7 (the block lies in one
                                // sequence; OUT_QKV: colb is already the padded position)
                                if constexpr (OUT == OUT_QKV) {
                                    dcol = colb + 16 * pp + 8 * half;
                                } else {
                                    const int sb = colb / seq_T;
                                    dcol = (int64_t)sb * seq_Tp + (colb - sb * seq_T) + 16 * pp + 8 * half;
                                }
                            }
                            *reinterpret_cast<u32x4 *>(crow + dcol) = u32x4{a0, a1, b0, b1};
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            };
            if constexpr (OUT == OUT_QKV) {
                if (cur.val) store_tile(std::integral_constant<bool, true>());
                else if constexpr (RDH > 0) store_rope();
                else store_tile(std::integral_constant<bool, false>());
            } else if constexpr (RDH > 0) {
                store_rope();
            } else {
                store_tile(std::integral_constant<bool, OUT == OUT_VT>());
            }
        }
        if (!has_next) break;
        cur = nxt;
        if (queue) {
            par ^= 1;
        } else {
            work += gridDim.x;
            has_next = work + (int)gridDim.x < n_work;
            if (has_next) decode(work + gridDim.x, nxt);
        }
    }
    wait_vmcnt<0>();
    finish();
}


// the persistent GEMMs' tile queues: 4 KiB per (device, stream), allocated on the first launch on
// that stream and held until the process ends
constexpr size_t kQueueBytes = 4096;
std::mutex g_queue_mu;
std::map<std::pair<int, hipStream_t>, int *> g_queues;
thread_local int g_queue_noalloc = 0;

int *gemm_queue(int dev, hipStream_t st) {
    std::lock_guard<std::mutex> lock(g_queue_mu);
    const auto it = g_queues.find({dev, st});
    if (it != g_queues.end()) return it->second;
    if (g_queue_noalloc > 0) return nullptr;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return nullptr;
    int *q = nullptr;
    if (hipMalloc(&q, kQueueBytes) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (hipMemset(q, 0, kQueueBytes) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(q);
        return nullptr;
    }
    g_queues[{dev, st}] = q;
    return q;
}

constexpr int CUS = 256;          // MI355X; the shape rules use it, the persistent grid asks the device
int device_cus(int *dev) {
    int ncu = 0;
    if (hipGetDevice(dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, *dev) != hipSuccess)
        return 0;
    return ncu;
}

// One product A B^T (and, OUT_QKV, the transposed values that go with it) as the launchers below see it
struct Gemm {
    int dtype;
    const void *A, *B;
    void *C;
    int M, N, K, lda, ldb, ldc;
    float alpha = 1.f;
    int seq_T = 1, seq_Tp = 1;
    // OUT_F32: parts of K (part p > 0 at C2 + (p - 1) part_stride); OUT_QKV: C2 the values' output
    void *C2 = nullptr;
    int ksplit = 1;
    int64_t part_stride = 0;
    // values: rows of B after its first N, output row stride, padded token positions
    int nv = 0, ldv = 0, n_tok = 0;
    const float4 *rtab = nullptr;
};

// sequences whose tokens fit in a tile's columns (OUT_VT of the small-tile kernel)
int packed(const Gemm &g, int bt) { return bt / g.seq_T; }
int packed_tiles(const Gemm &g, int bt) {
    return (g.nv + bt - 1) / bt * ((g.M / g.seq_T + packed(g, bt) - 1) / packed(g, bt));
}

template <int DT, int OUT, int RDH = 0>
hipError_t run_gemm_w4p(const Gemm &g, hipStream_t st) {
    constexpr int CPR = 8;
    constexpr size_t LDS = 5 * 256 * CPR * 16;       // rings of three and two k-tiles
    int dev = 0;
    const int ncu = device_cus(&dev);
    if (ncu <= 0) return hipErrorInvalidDevice;
    const int tm = (g.M + 255) / 256, tn = (g.N + 255) / 256;
    const int n_work = tm * tn * g.ksplit + (OUT == OUT_QKV ? (g.nv + 255) / 256 * ((g.n_tok + 255) / 256) : 0);
    hipError_t e = hipFuncSetAttribute((const void *)gemm_w4p_kernel<DT, OUT, CPR, RDH>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS);
    if (e != hipSuccess) return e;
    // the queue pays where a workgroup has many work items (measured: 80 per workgroup, the [Q|K]
    // projection of 128 x 2048 tokens at d 4096, 8.22 -> 8.00 ms; 10 and 2 per workgroup, the
    // projections of 16 x 2048 tokens, 1.8 and 8 % slower than the static order)
    const int grid = min(n_work, ncu);
    int *queue = grid % 8 == 0 && n_work >= 32 * grid && g.K / (CPR * 8) / g.ksplit >= 6 &&
                         (int)(kQueueBytes / 4) >= 16 + 2 * grid
                     ? gemm_queue(dev, st) : nullptr;
    gemm_w4p_kernel<DT, OUT, CPR, RDH><<<dim3(grid), dim3(256), LDS, st>>>(
        g.A, g.B, g.C, g.M, g.N, g.K, g.lda, g.ldb, g.ldc, tm, tn, g.seq_T, g.seq_Tp, n_work, g.rtab, g.alpha,
        g.ksplit, g.C2, queue, g.nv, g.ldv, g.n_tok);
    return hipGetLastError();
}

// A tile's loads take 32-bit byte offsets from its panels' first rows: bt rows of A and of B, and the k
// range behind the last one, end below 2^32 bytes (the weight gradient's rows are as long as the batch has
// tokens: 8.4 M of 16 bits with the 256-tile).  The row strides of a split plan are its K, at most a line less
// than the launch's: a plan for the persistent kernel that then does not fit runs its parts in small tiles.
bool offsets_fit(const Gemm &g, int bt) {
    return (int64_t)bt * std::max(g.lda, g.ldb) * (g.dtype == F32 ? 4 : 2) < ((int64_t)1 << 32) - 256;
}

// The persistent kernel takes whole 256 x 256 tiles, 16-byte aligned output rows and at least three
// k-tiles; a split K (fp32 output) only in two and where the tiles are whole in both directions (no
// tile moved back over its neighbour: the two parts are summed by the caller); for the transposed
// value output, 32-token blocks inside one sequence (OUT_QKV works on padded positions instead).
template <int OUT>
bool persistent_fits(const Gemm &g) {
    if (g.dtype == F32 || g.M < 256 || g.N < 256 || g.K % 64 != 0 || g.K / 64 / g.ksplit < 3 || !offsets_fit(g, 256))
        return false;
    if (g.ksplit > 1 && (OUT != OUT_F32 || g.ksplit > 2 || g.K % 128 != 0 || g.M % 256 != 0 || g.N % 256 != 0))
        return false;
    if (OUT == OUT_F32) return g.ldc % 4 == 0 && g.N % 4 == 0;
    if (g.ldc % 8 != 0) return false;
    if (OUT == OUT_VT) return g.seq_T % 32 == 0;
    if (g.N % 8 != 0) return false;
    return OUT != OUT_QKV || (g.nv >= 256 && g.n_tok >= 256 && g.lda == g.ldb && g.ldv % 8 == 0);
}

template <int DT, int BT, int CPR, int OUT, int RDH = 0, bool WIDE = false>
hipError_t run_gemm_small_cfg(const Gemm &g, hipStream_t st) {
    typedef SmallCfg<DT, BT, CPR> S;
    SmallArgs a;
    a.A = g.A; a.B = g.B; a.C = g.C; a.C2 = g.C2;
    a.M = g.M; a.N = g.N; a.K = g.K; a.lda = g.lda; a.ldb = g.ldb; a.ldc = g.ldc;
    a.nv = g.nv; a.ldv = g.ldv; a.seq_T = g.seq_T; a.seq_Tp = g.seq_Tp; a.n_tok = g.n_tok;
    a.alpha = g.alpha; a.ksplit = g.ksplit; a.part_stride = g.part_stride;
    a.tiles_m = g.C ? (g.M + BT - 1) / BT : 0;
    a.tiles_n = g.C ? (g.N + BT - 1) / BT : 0;
    a.tiles_vm = (g.nv + BT - 1) / BT;
    a.tiles_vn = (g.n_tok + BT - 1) / BT;
    if (OUT == OUT_VT) {
        a.pack = packed(g, BT);
        a.tiles_vn = (g.M / g.seq_T + a.pack - 1) / a.pack;
    }
    a.rtab = g.rtab;
    hipError_t e = hipFuncSetAttribute((const void *)gemm_small_kernel<DT, BT, CPR, OUT, RDH, WIDE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS_BYTES);
    if (e != hipSuccess) return e;
    const int n = a.tiles_m * a.tiles_n * g.ksplit + (OUT == OUT_F32 ? 0 : a.tiles_vm * a.tiles_vn);
    if (n == 0) return hipSuccess;
    gemm_small_kernel<DT, BT, CPR, OUT, RDH, WIDE><<<dim3(n), dim3(256), S::LDS_BYTES, st>>>(a);
    return hipGetLastError();
}

int tiles_of(const Gemm &g, int bt) {
    auto up = [bt](int v) { return (v + bt - 1) / bt; };
    return (g.C ? up(g.M) * up(g.N) * g.ksplit : 0) + up(g.nv) * up(g.n_tok);
}

// The 128-tile from one tile per CU on for the 16-bit dtypes (measured, 64-tile against 128-tile, us:
// K 768, 144 tiles 13.0 / 13.0, 288 18.6 / 18.6, 342 21.4 / 19.1; K 4096, 192 41.5 / 42.0, 384 76 / 61;
// at 48 tiles of K 4096 20 / 39) and from eight per CU for fp32 (whose 64-tile fills the matrix cores
// too: 576 tiles 128 / 155, 2304 442 / 433); packed sequences of more than 32 tokens fit the 64-tile once, the
// 128-tile up to three times
template <int DT, int OUT, int RDH>
hipError_t run_gemm_small(const Gemm &g, hipStream_t st) {
    if (g.K % 32 != 0) return hipErrorInvalidValue;
    if constexpr (RDH > 0) {                          // at least 192 rows of weights: K is below 11.2 M
        return g.K % 64 == 0 ? run_gemm_small_cfg<DT, 128, 8, OUT, RDH>(g, st)
                             : run_gemm_small_cfg<DT, 128, 4, OUT, RDH>(g, st);
    } else {
        if constexpr (OUT != OUT_VT)
            if (!offsets_fit(g, 64)) return run_gemm_small_cfg<DT, 64, 4, OUT, 0, true>(g, st);
        const int tiles = OUT == OUT_VT ? packed_tiles(g, 128) : tiles_of(g, 128);
        const bool big = (tiles >= (DT == F32 ? 8 : 1) * CUS || (OUT == OUT_VT && g.seq_T > 32)) && offsets_fit(g, 128);
        if constexpr (DT != F32)
            if (g.K % 64 != 0)
                return big ? run_gemm_small_cfg<DT, 128, 4, OUT>(g, st) : run_gemm_small_cfg<DT, 64, 4, OUT>(g, st);
        return big ? run_gemm_small_cfg<DT, 128, 8, OUT>(g, st) : run_gemm_small_cfg<DT, 64, 8, OUT>(g, st);
    }
}

template <int OUT, int RDH = 0>
hipError_t small(const Gemm &g, hipStream_t st) {
    if constexpr (RDH == 0)
        if (g.dtype == F32) return run_gemm_small<F32, OUT, 0>(g, st);
    if (g.dtype == F32) return hipErrorInvalidValue;
    return g.dtype == F16 ? run_gemm_small<F16, OUT, RDH>(g, st) : run_gemm_small<BF16, OUT, RDH>(g, st);
}
template <int OUT, int RDH = 0>
hipError_t persistent(const Gemm &g, hipStream_t st) {
    return g.dtype == F16 ? run_gemm_w4p<F16, OUT, RDH>(g, st) : run_gemm_w4p<BF16, OUT, RDH>(g, st);
}

// Where the 256-tiles fill their rounds of one workgroup per CU to at least 70 %, and K is long enough to
// carry a tile's start and end.  Measured (persistent against 128-tiles, us): K 4096, 75 % of one round
// 92 / 103, 75 % of two 186 / 194, 38 % of one 80 / 61; K 768, 88 % of one 32 / 33, 56 % of two 47 / 42,
// 75 % of three 71 / 70, 90 % of five 122 / 142; K 256, three whole rounds 59 / 52.
bool persistent_pays(const Gemm &g) {
    const int64_t t = tiles_of(g, 256);
    return g.K / g.ksplit >= 512 && 10 * t >= 7 * ((t + CUS - 1) / CUS) * CUS;
}

}  // namespace

GemmQueueNoAlloc::GemmQueueNoAlloc() { ++g_queue_noalloc; }
GemmQueueNoAlloc::~GemmQueueNoAlloc() { --g_queue_noalloc; }

hipError_t launch_gemm_nt(int dtype, const void *A, const void *B, void *C, int M, int N, int K,
                          int lda, int ldb, int ldc, hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    Gemm g{dtype, A, B, C, M, N, K, lda, ldb, ldc};
    return persistent_fits<OUT_DT>(g) && persistent_pays(g) ? persistent<OUT_DT>(g, st) : small<OUT_DT>(g, st);
}

namespace {
// An fp32 product whose K may be split: 256-tiles in one part or two where they pay, else small tiles
// in as many parts as fill the CUs (two 128-tiles each, three 64-tiles for fp32), each part keeping 512
// (fp32: 256) of K and the parts' sums at most 6 M values more to write and read.  Measured at 2304 x 768 x
// 8192 fp16, 27 256-tiles: two parts of them 82 us, four parts of 108 128-tiles
Gemm f32_plan(int dtype, int M, int N, int K, int ldc, bool split) {
    Gemm g{dtype, nullptr, nullptr, nullptr, M, N, K, K, K, ldc};
    char some = 0;
    g.C = &some;                                      // tiles count where there is an output
    if (split && K % 128 == 0) {
        const int t = tiles_of(g, 256);
        const double e1 = (double)t / (((t + CUS - 1) / CUS) * CUS);
        const double e2 = (double)(2 * t) / (((2 * t + CUS - 1) / CUS) * CUS);
        if (e2 > e1 + 0.05) g.ksplit = 2;
        if (persistent_fits<OUT_F32>(g) && persistent_pays(g)) return g;
        g.ksplit = 1;
    }
    if (!split || (persistent_fits<OUT_F32>(g) && persistent_pays(g))) return g;
    const int64_t t = tiles_of(g, dtype == F32 ? 64 : 128), slots = dtype == F32 ? 3 * CUS : 2 * CUS;
    const int64_t most = std::min<int64_t>({slots / t, K / (dtype == F32 ? 256 : 512), 1 + 6000000 / ((int64_t)M * N), 16});
    g.ksplit = (int)std::max<int64_t>(1, most);
    return g;
}
}  // namespace

int gemm_f32_parts(int dtype, int M, int N, int K) {
    return M > 0 && N > 0 && K > 0 ? f32_plan(dtype, M, N, K, N, true).ksplit : 1;
}

hipError_t launch_gemm_nt_f32out(int dtype, const void *A, const void *B, float *C, int M, int N, int K,
                                 int lda, int ldb, int ldc, float alpha, hipStream_t st, float *C2) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    Gemm g = f32_plan(dtype, M, N, K, ldc, C2 != nullptr);
    g.A = A; g.B = B; g.C = C; g.lda = lda; g.ldb = ldb;
    g.alpha = alpha;
    g.C2 = C2;
    g.part_stride = (int64_t)M * ldc;
    return persistent_fits<OUT_F32>(g) && persistent_pays(g) ? persistent<OUT_F32>(g, st) : small<OUT_F32>(g, st);
}

bool gemm_rope_fuses(int dtype, int head_dim) { return dtype != F32 && (head_dim == 64 || head_dim == 128); }

namespace {
Gemm projection(int dtype, const void *x, const void *w, void *qk, void *vt, int batch, int seq_T, int nqk, int nv,
                int K, int ldv, const float4 *rope_tab_t) {
    Gemm g{dtype, x, w, qk, batch * seq_T, nqk, K, K, K, nqk};
    g.seq_T = seq_T; g.seq_Tp = (seq_T + 31) / 32 * 32;
    g.C2 = vt; g.nv = nv; g.ldv = ldv; g.n_tok = vt ? batch * g.seq_Tp : 0;
    g.rtab = rope_tab_t;
    return g;
}
// a projection whose [Q|K] part goes to the persistent kernel
bool qk_persistent(const Gemm &g) { return persistent_fits<OUT_DT>(g) && persistent_pays(g); }
// ... and its values with it: one round less where both leave one part empty, and no second launch; a
// launch of its own keeps the values' k-tile rotation and the [Q|K] tile queue (from 32 rounds on).
// Measured, one launch / two, us, at d 4096, 5120 + 1024 columns: 8 K tokens 307 / 371, 16 K 611 / 612,
// 32 K 1203 / 1212, 64 K (24 rounds) 2450 / 2510.  Sequences that are not whole blocks of 32 tokens
// go together where this form takes them (256 value rows); else their values go to the small tiles
bool qkv_persistent(const Gemm &g) {
    return qk_persistent(g) && persistent_fits<OUT_QKV>(g) &&
           (g.seq_Tp != g.seq_T || tiles_of(g, 256) <= 24 * CUS);
}
}  // namespace

namespace {
// Values of very short sequences over their tokens, several sequences per tile, instead of over padded positions:
// in a launch of their own, whose tiles run at a little over half of the 256-tile's rate (fp32: four fifths of
// the 128-tile's).  Where the products left out (with that factor) are worth 20 us: 24 GFLOP at 1.2 PFLOP/s, fp32 a tenth.  Measured,
// us of the projection, padded / packed (and the 256-tiles over tokens, single stores and a zeroing pass that padded
// positions replaced): d 4096, 1024 value rows, 8192 x 1 token 1912 / 430 (1109), 4096 x 8 1814 / 1402 (1529),
// 2048 x 16 1445 / 1395 (1364), 2048 x 20 1728 / 1806, 256 x 1 97 / 62, 64 x 1 42 / 55; d 768, 4096 x 8 229 / 166,
// 2048 x 16 158 / 176; in fp32 4096 x 1 1347 / 180 (412), 1024 x 16 597 / 486 (537), 1000 x 33 1285 / 1151 (1190),
// 64 x 1 31 / 56.
bool pack_pays(const Gemm &g) {
    if (g.seq_T > 64 || g.nv == 0 || !offsets_fit(g, 128)) return false;
    const int64_t tiles = (g.M / g.seq_T + packed(g, 128) - 1) / packed(g, 128);
    const double saved = ((double)g.n_tok - (g.dtype == F32 ? 1.25 : 1.75) * 128 * (double)tiles) * 2.0 * g.nv * g.K;
    return saved >= (g.dtype == F32 ? 2.4e9 : 2.4e10);
}
}  // namespace

bool project_is_one_launch(int dtype, int batch, int seq_T, int nqk, int nv, int K, int ldv) {
    char some = 0;                                    // tiles count where there is an output
    const Gemm g = projection(dtype, nullptr, nullptr, &some, &some, batch, seq_T, nqk, nv, K, ldv, nullptr);
    if (pack_pays(g)) return false;
    return qk_persistent(g) ? qkv_persistent(g) : true;
}

hipError_t launch_project(int dtype, const void *x, const void *w, void *qk, void *vt, int batch, int seq_T, int nqk,
                          int nv, int K, int ldv, int head_dim, const float4 *rope_tab_t, hipStream_t st) {
    if (qk == nullptr) {
        // V^T = W_V X^T: the operands swapped
        const int M = batch * seq_T;
        Gemm t{dtype, static_cast<const char *>(w) + (size_t)nqk * K * (dtype == F32 ? 4 : 2), x, vt, nv, M, K, K, K, ldv};
        t.seq_T = seq_T; t.seq_Tp = (seq_T + 31) / 32 * 32;
        if (persistent_fits<OUT_VT>(t) && persistent_pays(t)) return persistent<OUT_VT>(t, st);
        const Gemm g = projection(dtype, x, w, nullptr, vt, batch, seq_T, nqk, nv, K, ldv, nullptr);
        return pack_pays(g) ? small<OUT_VT>(g, st) : small<OUT_DT>(g, st);
    }
    const bool rope = rope_tab_t != nullptr;
    if (rope && (!gemm_rope_fuses(dtype, head_dim) || nqk % head_dim != 0)) return hipErrorInvalidValue;
    Gemm g = projection(dtype, x, w, qk, vt, batch, seq_T, nqk, nv, K, ldv, rope_tab_t);
    if (!qk_persistent(g)) {
        if (!rope) return small<OUT_DT>(g, st);
        return head_dim == 64 ? small<OUT_DT, 64>(g, st) : small<OUT_DT, 128>(g, st);
    }
    if (vt != nullptr) {
        if (!qkv_persistent(g)) return hipErrorInvalidValue;
        if (!rope) return persistent<OUT_QKV>(g, st);
        return head_dim == 64 ? persistent<OUT_QKV, 64>(g, st) : persistent<OUT_QKV, 128>(g, st);
    }
    g.nv = 0;
    if (!rope) return persistent<OUT_DT>(g, st);
    return head_dim == 64 ? persistent<OUT_DT, 64>(g, st) : persistent<OUT_DT, 128>(g, st);
}

}  // namespace jab
