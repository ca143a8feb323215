// attn_bwd_f32.hip -- backward of the JAB loss through causal GQA attention in fp32: the dK/dV and dQ
// kernels (the formulas are those of attn_bwd_mfma.hip's header).
//
// What bounds it: the fp32 matrix instructions (32x32x2, 64 cycles for 2 k-steps): a 32 x 32 tile at
// head_dim 64 takes 128 of them for dK/dV, 3.5 us in one wave, so the length of a wave's chain of tiles
// decides at the sizes fp32 is used at.  A workgroup therefore owns one 32-row block (keys of a kv head, or
// queries of a head) and its NW waves (four, or one: one_wave) take every NW-th tile that block meets; the sums
// are added in LDS at the end, in wave order.  A wave stages its own tiles, row-major, with the next tile's global loads
// in registers while it computes: no barrier in the loop.  The products that contract over tokens read
// the same tiles column by column (one float per lane, 32 consecutive addresses), so no transposed copy is kept.
// The teacher's tile of the KL term enters one score product alone, so it stays in registers as that product's
// operand: with it in LDS, head_dim 128 had room for two waves per CU (8 x 2048 tokens of 32 / 8 heads of 128,
// dK/dV and dQ 14.8 and 11.2 ms against 9.0 and 6.2 with four).
// MI355X, us, dK/dV and dQ, with 128-row workgroups whose waves shared staged tiles / here: 3 x 333 tokens
// of 12 heads of 64 76 and 55 / 39 and 24, 8 x 512 191 and 149 / 125 and 71; with the KL term 2 x 512 124 and
// 99 / 43 and 35.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace jab {
namespace {

template <int DH, bool KL>
struct F32Cfg {
    static constexpr int RST = DH + 4;                 // floats per tile row
    static constexpr int NDB = DH < 32 ? 1 : DH / 32;  // 32-row blocks of a transposed result
    // head_dim 16 reads 32 columns (the upper 16 rows of the result are not used): 16 floats of slack
    static constexpr int TILE = 32 * RST + (DH < 32 ? 16 : 0);
    static constexpr int WAVE = 2 * TILE + 96;         // Q, G (K, V); lse, D and the teacher's lse of the 32 queries
    static constexpr int LD = DH / 8;                  // 16-byte loads per lane and tile
    static constexpr bool AHEAD = !(DH == 128 && KL);  // the next tile's loads in registers (else they spill)
};

typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

// a wave's own LDS writes are done before its reads (the lanes exchange data)
__device__ inline void wave_lds_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ inline f32x16 mma32(float x, float y, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, c, 0, 0, 0); }

template <int N>
__device__ inline void clear(f32x16 (&v)[N]) {
#pragma unroll
    for (int d = 0; d < N; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) v[d][e] = 0.f;
}

// rows r0 .. r0 + 31 (rows past T as zeros) of a matrix with row stride ld, column c0: lane -> 16-byte
// chunk 64 i + lane
template <int DH>
__device__ inline void load_rows(f32x4 (&v)[DH / 8], const float *base, int64_t ld, int r0, int T, int lane) {
    constexpr int CPR = DH / 4;
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        const int p = 64 * i + lane, r = p / CPR, c = p % CPR;
        v[i] = r0 + r < T ? *reinterpret_cast<const f32x4 *>(base + (int64_t)(r0 + r) * ld + 4 * c) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
}
template <int DH>
__device__ inline void store_rows(lds_f32 *t, const f32x4 (&v)[DH / 8], int lane) {
    constexpr int CPR = DH / 4;
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        const int p = 64 * i + lane, r = p / CPR, c = p % CPR;
        *(lds_f32x4 *)(t + r * (DH + 4) + 4 * c) = v[i];
    }
}
// operand of a product over the head dimension: row `row` (nullptr: zeros), k-steps 4 i + t at columns
// 8 i + 4 half + t
template <int DH>
__device__ inline void row_operand(f32x4 (&v)[DH / 8], const float *row, int half) {
#pragma unroll
    for (int i = 0; i < DH / 8; ++i)
        v[i] = row ? *reinterpret_cast<const f32x4 *>(row + 8 * i + 4 * half) : f32x4{0.f, 0.f, 0.f, 0.f};
}
// c += (tile rows) x (operand b): lane -> column (b's row), registers -> tile rows
template <int DH>
__device__ inline f32x16 scores(const lds_f32 *t, const f32x4 (&b)[DH / 8], int lane) {
    f32x16 c;
#pragma unroll
    for (int e = 0; e < 16; ++e) c[e] = 0.f;
#pragma unroll
    for (int i = 0; i < DH / 8; ++i) {
        const f32x4 x = *(const lds_f32x4 *)(t + (lane & 31) * (DH + 4) + 8 * i + 4 * (lane >> 5));
#pragma unroll
        for (int k = 0; k < 4; ++k) c = mma32(x[k], b[i][k], c);
    }
    return c;
}
// the same from the tile's rows in registers (row_operand of row lane % 32), with the same products in the same
// order: equal maps give equal scores
template <int DH>
__device__ inline f32x16 scores(const f32x4 (&t)[DH / 8], const f32x4 (&b)[DH / 8]) {
    f32x16 c;
#pragma unroll
    for (int e = 0; e < 16; ++e) c[e] = 0.f;
#pragma unroll
    for (int i = 0; i < DH / 8; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) c = mma32(t[i][k], b[i][k], c);
    return c;
}
// acc (transposed: registers -> head dimension) += tile^T x s, contracted over the tile's 32 rows
template <int DH, int NDB>
__device__ inline void accumulate(f32x16 (&acc)[NDB], const lds_f32 *t, const f32x16 &s, int lane) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int r = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
#pragma unroll
        for (int d = 0; d < NDB; ++d) acc[d] = mma32(t[r * (DH + 4) + d * 32 + (lane & 31)], s[e], acc[d]);
    }
}
// the waves' sums, into wave 0 (in wave order)
template <int NW, int N>
__device__ inline void add_waves(f32x16 (&acc)[N], lds_f32 *ex, int wave, int lane) {
    __syncthreads();                                   // every wave is done with its tiles
    if (wave > 0) {
#pragma unroll
        for (int d = 0; d < N; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) ex[(((wave - 1) * N + d) * 16 + e) * 64 + lane] = acc[d][e];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll 1
    for (int w = 0; w < NW - 1; ++w)
#pragma unroll
        for (int d = 0; d < N; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[d][e] += ex[((w * N + d) * 16 + e) * 64 + lane];
}
// workgroup -> (row block in launch order, head), the heads of an XCD its own where they divide evenly
__device__ inline void block_and_head(int nblocks, int &blk, int &head) {
    const int heads = gridDim.x / nblocks, per = heads & 7 ? heads : heads >> 3;
    const int x = heads & 7 ? 0 : blockIdx.x & 7, i = heads & 7 ? blockIdx.x : blockIdx.x >> 3;
    blk = i / per;
    head = x * per + i % per;
}

template <int DH, bool KL, int NW>
constexpr size_t f32_lds_bytes(int sums) {
    typedef F32Cfg<DH, KL> C;
    const size_t tiles = (size_t)NW * C::WAVE, ex = (size_t)(NW - 1) * sums * C::NDB * 1024;
    return (tiles > ex ? tiles : ex) * sizeof(float);
}

// dK^T and dV^T of the 32 keys of block kb of one kv head
template <int DH, bool KL, int NW>
__global__ __launch_bounds__(64 * NW, 1) void attn_bwd_dkdv_f32_kernel(AttnBwdArgs a, float scale_log2, float inv_sqrt,
                                                                      int nkb) {
    typedef F32Cfg<DH, KL> C;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = a.seq_len, Hq = a.n_heads, Hkv = a.n_kv_heads, G = Hq / Hkv;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int kb, head;
    block_and_head(nkb, kb, head);                     // the block of the most query tiles first
    const int kvh = head % Hkv, b = head / Hkv;
    const int k0 = 32 * kb, key = k0 + (lane & 31);
    const int64_t row0 = (int64_t)b * T;
    const float *Q = static_cast<const float *>(a.q) + row0 * a.ldq;
    const float *Gr = static_cast<const float *>(a.g) + row0 * Hq * DH;
    const float *Qt = KL ? static_cast<const float *>(a.qt) + row0 * a.ldq : nullptr;
    lds_f32 *tq = (lds_f32 *)smem + wave * C::WAVE, *tg = tq + C::TILE, *st = tq + 2 * C::TILE;

    f32x4 kf[C::LD], vf[C::LD], ktf[KL ? C::LD : 1];
    const bool live = key < T;
    row_operand<DH>(kf, live ? static_cast<const float *>(a.k) + (row0 + key) * a.ldq + kvh * DH : nullptr, half);
    row_operand<DH>(vf, live ? static_cast<const float *>(a.v) + (row0 + key) * a.ldv + kvh * DH : nullptr, half);
    if constexpr (KL)
        row_operand<DH>(ktf, live ? static_cast<const float *>(a.kt) + (row0 + key) * a.ldq + kvh * DH : nullptr, half);
    f32x16 acc[2 * C::NDB];                            // dV^T, then dK^T
    clear(acc);
    f32x16(&dvt)[C::NDB] = *reinterpret_cast<f32x16(*)[C::NDB]>(&acc[0]);
    f32x16(&dkt)[C::NDB] = *reinterpret_cast<f32x16(*)[C::NDB]>(&acc[C::NDB]);

    const int nq = (T - k0 + 31) / 32, n = G * nq;     // tile v: head kvh G + v / nq, query tile v % nq
    f32x4 rq[C::LD], rg[C::LD], rt[KL ? C::LD : 1];
    float rs = 0.f, rl = 0.f;
    auto load = [&](int v) {
        const int h = kvh * G + v / nq, i0 = k0 + 32 * (v % nq);
        load_rows<DH>(rq, Q + h * DH, a.ldq, i0, T, lane);
        load_rows<DH>(rg, Gr + h * DH, (int64_t)Hq * DH, i0, T, lane);
        const int q = i0 + (lane & 31);
        const int64_t li = ((int64_t)b * Hq + h) * T + q;
        rs = q < T ? (half ? a.D[li] : a.lse2[li]) : (half ? 0.f : INFINITY);
        if constexpr (KL) rl = q < T ? a.lse_t[li] : INFINITY;
    };
    auto load_teacher = [&](int v) {
        const int h = kvh * G + v / nq, q = k0 + 32 * (v % nq) + (lane & 31);
        if constexpr (KL) row_operand<DH>(rt, q < T ? Qt + (int64_t)q * a.ldq + h * DH : nullptr, half);
    };
    if (C::AHEAD && wave < n) {
        load(wave);
        load_teacher(wave);
    }
    for (int v = wave; v < n; v += NW) {
        if (!C::AHEAD) {
            load(v);
            load_teacher(v);
        }
        wave_lds_fence();                              // the last tile's reads are done
        store_rows<DH>(tq, rq, lane);
        store_rows<DH>(tg, rg, lane);
        st[lane] = rs;
        if (KL && half == 0) st[64 + lane] = rl;
        wave_lds_fence();
        const int i0 = k0 + 32 * (v % nq);
        if (C::AHEAD && v + NW < n) load(v + NW);
        f32x16 sc;
        if constexpr (KL) sc = scores<DH>(rt, ktf);
        if (C::AHEAD && v + NW < n) load_teacher(v + NW);
        f32x16 s = scores<DH>(tq, kf, lane), dp = scores<DH>(tg, vf, lane);
        const bool diag = i0 == k0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * half + (e & 3);
            const bool off = diag && i0 + r < key;
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2, -st[r]));
            if (off) p = 0.f;
            float ds = p * (dp[e] - st[32 + r]);
            if constexpr (KL) {
                float pt = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], scale_log2, -st[64 + r]));
                if (off) pt = 0.f;
                ds = (ds + a.kl_scale * (p - pt)) * a.grad_scale;
            }
            s[e] = p;
            dp[e] = ds;
        }
        accumulate<DH>(dvt, tg, s, lane);
        accumulate<DH>(dkt, tq, dp, lane);
    }
    add_waves<NW>(acc, (lds_f32 *)smem, wave, lane);
    if (wave > 0 || !live) return;
    float *dyt = static_cast<float *>(a.dyt) + row0 + key;
    const int koff = Hq * DH + kvh * DH, voff = (Hq + Hkv) * DH + kvh * DH;
#pragma unroll
    for (int d = 0; d < C::NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
            if (DH < 32 && c >= DH) continue;
            dyt[(int64_t)(koff + c) * a.ldt] = dkt[d][e] * inv_sqrt;
            dyt[(int64_t)(voff + c) * a.ldt] = dvt[d][e];
        }
}

// dQ^T of the 32 queries of one block of one head
template <int DH, bool KL, int NW>
__global__ __launch_bounds__(64 * NW, 1) void attn_bwd_dq_f32_kernel(AttnBwdArgs a, float scale_log2, float inv_sqrt,
                                                                    int nqb) {
    typedef F32Cfg<DH, KL> C;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = a.seq_len, Hq = a.n_heads, Hkv = a.n_kv_heads, G = Hq / Hkv;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int blk, head;
    block_and_head(nqb, blk, head);
    const int qb = nqb - 1 - blk;                      // the block of the most key tiles first
    const int h = head % Hq, b = head / Hq, kvh = h / G;
    const int qrow = 32 * qb + (lane & 31);
    const int64_t row0 = (int64_t)b * T;
    const float *K = static_cast<const float *>(a.k) + row0 * a.ldq + kvh * DH;
    const float *V = static_cast<const float *>(a.v) + row0 * a.ldv + kvh * DH;
    const float *Kt = KL ? static_cast<const float *>(a.kt) + row0 * a.ldq + kvh * DH : nullptr;
    lds_f32 *tk = (lds_f32 *)smem + wave * C::WAVE, *tv = tk + C::TILE;

    f32x4 qf[C::LD], gf[C::LD], qtf[KL ? C::LD : 1];
    const bool live = qrow < T;
    row_operand<DH>(qf, live ? static_cast<const float *>(a.q) + (row0 + qrow) * a.ldq + h * DH : nullptr, half);
    row_operand<DH>(gf, live ? static_cast<const float *>(a.g) + ((row0 + qrow) * Hq + h) * DH : nullptr, half);
    if constexpr (KL)
        row_operand<DH>(qtf, live ? static_cast<const float *>(a.qt) + (row0 + qrow) * a.ldq + h * DH : nullptr, half);
    const int64_t li = ((int64_t)b * Hq + h) * T + qrow;
    const float lse = live ? a.lse2[li] : INFINITY, Dq = live ? a.D[li] : 0.f;
    const float lset = KL && live ? a.lse_t[li] : INFINITY;
    f32x16 dqt[C::NDB];
    clear(dqt);

    f32x4 rk[C::LD], rv[C::LD], rt[KL ? C::LD : 1];
    auto load = [&](int j) {
        load_rows<DH>(rk, K, a.ldq, 32 * j, T, lane);
        load_rows<DH>(rv, V, a.ldv, 32 * j, T, lane);
    };
    auto load_teacher = [&](int j) {
        const int k = 32 * j + (lane & 31);
        if constexpr (KL) row_operand<DH>(rt, k < T ? Kt + (int64_t)k * a.ldq : nullptr, half);
    };
    if (C::AHEAD && wave <= qb) {
        load(wave);
        load_teacher(wave);
    }
    for (int j = wave; j <= qb; j += NW) {
        if (!C::AHEAD) {
            load(j);
            load_teacher(j);
        }
        wave_lds_fence();                              // the last tile's reads are done
        store_rows<DH>(tk, rk, lane);
        store_rows<DH>(tv, rv, lane);
        wave_lds_fence();
        if (C::AHEAD && j + NW <= qb) load(j + NW);
        f32x16 sc;
        if constexpr (KL) sc = scores<DH>(rt, qtf);
        if (C::AHEAD && j + NW <= qb) load_teacher(j + NW);
        f32x16 s = scores<DH>(tk, qf, lane), dp = scores<DH>(tv, gf, lane);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const bool off = j == qb && 32 * j + 8 * (e >> 2) + 4 * half + (e & 3) > qrow;
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2, -lse));
            if (off) p = 0.f;
            float ds = p * (dp[e] - Dq);
            if constexpr (KL) {
                float pt = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], scale_log2, -lset));
                if (off) pt = 0.f;
                ds = (ds + a.kl_scale * (p - pt)) * a.grad_scale;
            }
            dp[e] = ds;
        }
        accumulate<DH>(dqt, tk, dp, lane);
    }
    add_waves<NW>(dqt, (lds_f32 *)smem, wave, lane);
    if (wave > 0 || !live) return;
    float *dyt = static_cast<float *>(a.dyt) + row0 + qrow;
#pragma unroll
    for (int d = 0; d < C::NDB; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int c = d * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
            if (DH < 32 && c >= DH) continue;
            dyt[(int64_t)(h * DH + c) * a.ldt] = dqt[d][e] * inv_sqrt;
        }
}

// the arguments of sequences b0 .. b0 + n - 1
template <bool KL>
AttnBwdArgs sequences(const AttnBwdArgs &a, int b0, int n) {
    AttnBwdArgs s = a;
    const int64_t row = (int64_t)b0 * a.seq_len, map = (int64_t)b0 * a.n_heads * a.seq_len;
    auto rows = [row](const void *p, int64_t ld) { return static_cast<const float *>(p) + row * ld; };
    s.batch = n;
    s.q = rows(a.q, a.ldq);
    s.k = rows(a.k, a.ldq);
    s.v = rows(a.v, a.ldv);
    s.g = rows(a.g, (int64_t)a.n_heads * a.head_dim);
    s.lse2 = a.lse2 + map;
    s.D = a.D + map;
    s.dyt = static_cast<float *>(a.dyt) + row;
    if (KL) {
        s.qt = rows(a.qt, a.ldq);
        s.kt = rows(a.kt, a.ldq);
        s.lse_t = a.lse_t + map;
    }
    return s;
}

// Whether a block's tiles go to one wave, in a workgroup of its own, or to four: one where the blocks fill the
// chip's waves (one per SIMD) anyway, since four leave waves without a tile at each block's end and in every block
// of few tiles, and add their sums.  In times of a tile: the longest block, or all tiles over 4 x 256 waves
// (0.8 of a tile per block for its start and end); four waves' steps over 256 workgroups (1.3 per block).  shared:
// the kernel's registers let two such workgroups share a CU (dQ below head_dim 128), which hides more of theirs.
// The same with the KL term as without, so lambda = 0 gives the squared error's gradients bit for bit.
// us, four waves / one (and 128-row workgroups before): dK/dV GPT-2 1000 x 33 tokens 1207 / 319 (707), 100 x 100
// 244 / 100 (156), 8 x 512 132 / 99 (196), 3 x 333 39 / 62 (76); 32 / 8 heads of 128 64 x 33 117 / 89 (173),
// 16 x 100 83 / 159 (181), 8 x 512 403 / 637 (695).  dQ GPT-2 1000 x 33 480 / 225 (536), 20 x 333 103 / 83
// (152), 8 x 512 76 / 94 (152); heads of 128 64 x 33 222 / 80 (128), 16 x 100 122 / 56 (97)
bool one_wave(int nb, int G, int64_t heads, bool shared) {
    const double n = nb, tiles = G * n * (n + 1) / 2, part = G % 4 == 0 ? 0.0 : G == 2 ? 0.25 : 0.375;
    const double one = std::max(G * n + 0.8, heads * (tiles + 0.8 * n) / (shared ? 1.25 * 1024 : 1024));
    const double four = std::max(G * n / 4 + 1.3, heads * (tiles / 4 + (part + 1.3) * n) / (shared ? 1.9 * 256 : 256));
    return one < 0.9 * four;
}

template <int DH, bool KL>
hipError_t run(const AttnBwdArgs &a, hipStream_t st) {
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
    const float inv_sqrt = 1.f / sqrtf((float)DH);
    const int nb = (a.seq_len + 31) / 32;
    // (a grid holds below 2^32 threads, so many heads of many sequences go in several launches)
    auto launch = [&](auto kernel, int waves, int heads, size_t lds) -> hipError_t {
        hipError_t err = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        const int64_t most = (((int64_t)1 << 32) - 1) / (64 * waves);
        const int step = (int)std::max<int64_t>(1, most / ((int64_t)nb * heads));
        for (int b0 = 0; err == hipSuccess && b0 < a.batch; b0 += std::min(step, a.batch - b0)) {
            const int n = std::min(step, a.batch - b0);
            kernel<<<dim3(nb * heads * n), dim3(64 * waves), lds, st>>>(sequences<KL>(a, b0, n), scale_log2, inv_sqrt, nb);
            err = hipGetLastError();
        }
        return err;
    };
    static_assert(f32_lds_bytes<DH, KL, 4>(2) <= 160 * 1024, "LDS");
    const int G = a.n_heads / a.n_kv_heads;
    const hipError_t e =
        one_wave(nb, G, (int64_t)a.n_kv_heads * a.batch, false)
            ? launch(attn_bwd_dkdv_f32_kernel<DH, KL, 1>, 1, a.n_kv_heads, f32_lds_bytes<DH, KL, 1>(2))
            : launch(attn_bwd_dkdv_f32_kernel<DH, KL, 4>, 4, a.n_kv_heads, f32_lds_bytes<DH, KL, 4>(2));
    if (e != hipSuccess) return e;
    return one_wave(nb, 1, (int64_t)a.n_heads * a.batch, DH < 128)
               ? launch(attn_bwd_dq_f32_kernel<DH, KL, 1>, 1, a.n_heads, f32_lds_bytes<DH, KL, 1>(1))
               : launch(attn_bwd_dq_f32_kernel<DH, KL, 4>, 4, a.n_heads, f32_lds_bytes<DH, KL, 4>(1));
}

}  // namespace

hipError_t launch_attn_bwd_f32(const AttnBwdArgs &a, hipStream_t st) {
    switch (a.head_dim) {
    case 16: return a.qt ? run<16, true>(a, st) : run<16, false>(a, st);
    case 64: return a.qt ? run<64, true>(a, st) : run<64, false>(a, st);
    default: return a.qt ? run<128, true>(a, st) : run<128, false>(a, st);
    }
}

}  // namespace jab
