// quant.hip -- per-(output row, group) quantizer of the fused QKV weight.
//
// Paper: Method, eq. quant (grid and clipping), Appendix "Joint STE fine-tuning"
// (1) (one scale per (output row, group)).  Asymmetric variant: scale and integer
// zero-point from the group's min-max range with 0 included.
//
// Work decomposition: one thread owns 8 consecutive weights of one row.  A group
// of g weights is g/8 consecutive lanes (g in {32, 64, 128} -> 4, 8, 16 lanes),
// so min/max reductions are lane shuffles inside one wavefront.  Loads and
// stores are 16-byte (32-byte for fp32) per thread and fully coalesced.  Every
// fp32 operation is IEEE-rounded (correctly rounded division, no contraction,
// no flush of denormals) so codes are bit-identical to an fp32 reference.
#include "device_common.h"
#include "kernels.h"

namespace jab {
namespace {

template <int DT> struct Chunk8;
template <> struct Chunk8<BF16> {
    u16x8 v;
    __device__ float get(int i) const { return bf16_bits_to_f32(v[i]); }
};
template <> struct Chunk8<F16> {
    u16x8 v;
    __device__ float get(int i) const { return f16_bits_to_f32(v[i]); }
};
template <> struct Chunk8<F32> {
    f32x4 a, b;
    __device__ float get(int i) const { return i < 4 ? a[i] : b[i - 4]; }
};

template <int DT>
__device__ inline void load8(const void *w, int64_t e, float out[8]) {
    if constexpr (DT == F32) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(static_cast<const float *>(w) + e);
        Chunk8<F32> c{p[0], p[1]};
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = c.get(i);
    } else {
        Chunk8<DT> c{*reinterpret_cast<const u16x8 *>(static_cast<const uint16_t *>(w) + e)};
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = c.get(i);
    }
}

template <int DT>
__device__ inline void store8(void *dst, int64_t e, const float v[8]) {
    if constexpr (DT == F32) {
        f32x4 *p = reinterpret_cast<f32x4 *>(static_cast<float *>(dst) + e);
        p[0] = f32x4{v[0], v[1], v[2], v[3]};
        p[1] = f32x4{v[4], v[5], v[6], v[7]};
    } else {
        u16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = from_f32<DT>(v[i]);
        *reinterpret_cast<u16x8 *>(static_cast<uint16_t *>(dst) + e) = o;
    }
}

__device__ inline int matrix_of_row(int r, int row_k, int row_v) {
    return r < row_k ? 0 : (r < row_v ? 1 : 2);
}

// ------------------------------------------------------------------ quant-init
// A thread takes QCPT chunks of 8 weights, 256 chunks apart, all loads before the arithmetic, with 32-bit
// row and column indexing (rows * cols is at most 2^31 - 1).  Bound by HBM: 50 MB of a Mistral layer in
// 17 us with one chunk per thread, 64-bit divisions and a scale per chunk, 13 us so (16 layers at once 239 / 148, 5.4 TB/s).
constexpr int QCPT = 4;

template <int DT>
__global__ __launch_bounds__(256) void quant_init_kernel(QuantShape sh, const void *__restrict__ w,
                                                         float *__restrict__ scale,
                                                         uint8_t *__restrict__ zero) {
    const uint32_t nchunks = (uint32_t)((int64_t)sh.rows * sh.cols / 8);
    const uint32_t c0 = blockIdx.x * (256u * QCPT) + threadIdx.x;
    const int lpg = sh.group / 8;                     // lanes per group (power of two)
    // Threads past the end still take part in the shuffles (their lanes hold
    // neutral values); chunks never straddle groups since g is a multiple of 8.
    float v[QCPT][8];
#pragma unroll
    for (int i = 0; i < QCPT; ++i) {
        const uint32_t c = c0 + 256u * i;             // a group is past the end as a whole
        load8<DT>(w, (int64_t)(c < nchunks ? c : 0) * 8, v[i]);
    }
    // every lane of a group gets the group's range; lane i of the group keeps chunk i's, so the divisions
    // run once for all chunks
    const int gl = threadIdx.x & (lpg - 1);
    float lo = 0.f, hi = 0.f;                         // symmetric: hi = max |w|
#pragma unroll
    for (int i = 0; i < QCPT; ++i) {
        float l = 0.f, h = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            l = fminf(l, v[i][k]);
            h = fmaxf(h, sh.scheme == 0 ? v[i][k] : fabsf(v[i][k]));
        }
        for (int off = lpg / 2; off >= 1; off >>= 1) {
            l = fminf(l, __shfl_xor(l, off, 64));
            h = fmaxf(h, __shfl_xor(h, off, 64));
        }
        if (gl == i) {
            lo = l;
            hi = h;
        }
    }
    const uint32_t c = c0 + 256u * gl;                // a chunk of lane gl's group (the group's first is below it)
    if (gl >= QCPT || c - gl >= nchunks) return;
    const uint32_t gi = c / lpg;                      // groups are contiguous in memory
    const int r = (int)(gi / (uint32_t)(sh.cols / sh.group));
    const int bits = sh.bits[matrix_of_row(r, sh.row_k, sh.row_v)];
    float s = 1.f;
    int z = 0;
    if (bits != 0) {
        if (sh.scheme == 0) {
            const float levels = (float)((1 << bits) - 1);
            const float range = hi - lo;
            s = range / levels;
            if (s == 0.f) s = 1.f;
            float zf = rintf(-lo / s);
            zf = fminf(fmaxf(zf, 0.f), levels);
            z = (int)zf;
        } else {
            const float qmax = (float)((1 << (bits - 1)) - 1);
            s = hi / qmax;
            if (s == 0.f) s = 1.f;
        }
    }
    scale[gi] = s;
    if (zero) zero[gi] = (uint8_t)z;
}

// ------------------------------------------------------------------ fake quant
// Writes any of: codes (u8), w_hat (fp32), w_op (dtype; the projection operand),
// and per-block partial sums of (w_hat - w)^2 and w^2 for each matrix.  A thread takes
// QCPT chunks of 8 weights, 256 chunks apart (each of the block's QCPT passes reads 4 KiB
// (bf16) contiguously); all of its loads are issued before the arithmetic.  Bound by HBM with codes, fp32
// weights and weight errors (175 MB of a Mistral layer: 40 us with the errors selected per weight, 35.4 us
// = 4.95 TB/s per chunk, a copy's rate).

template <int DT>
__device__ inline void quant_chunk(const QuantShape &sh, int64_t e, const float v[8], const float *__restrict__ scale,
                                   const uint8_t *__restrict__ zero, uint8_t *__restrict__ codes,
                                   float *__restrict__ w_hat, void *__restrict__ w_op, bool want_err, double err[3],
                                   double nrm[3]) {
    // rows * cols fits 32 bits (problem validation) and the group size is a power of two
    const uint32_t eu = (uint32_t)e, cols = (uint32_t)sh.cols;
    const int r = (int)(eu / cols);
    const uint32_t col = eu - (uint32_t)r * cols;
    const int m = matrix_of_row(r, sh.row_k, sh.row_v);
    const int bits = sh.bits[m];
    float wh[8];
    uint8_t q8[8];
    if (bits == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { wh[i] = v[i]; q8[i] = 0; }
    } else {
        const int gsh = __builtin_ctz((unsigned)sh.group);
        const uint32_t gi = (uint32_t)r * (cols >> gsh) + (col >> gsh);
        const float s = scale[gi];
        float u[8];                                    // round half to even of fp32(v / s)
        if (s >= 0x1p-60f && s <= 0x1p60f) {
            // One correctly rounded reciprocal per chunk instead of eight divisions: with rs the
            // correctly rounded 1/s and q0 = fp32(v rs) (within one ulp of v / s), the remainder
            // v - q0 s is exact in one fma and q0 + rem rs, rounded once, is the correctly rounded
            // quotient (Markstein's theorem on division by a refined reciprocal, IBM J. Res. Dev.
            // 34(1), 1990).  The range of s keeps the remainder clear of underflow wherever the
            // quotient can round to a non-zero integer; an overflowing q0 is kept (infinite, as the
            // quotient is).
            const float rs = 1.f / s;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float q0 = v[i] * rs;
                const float rem = __builtin_fmaf(-q0, s, v[i]);
                u[i] = rintf(__builtin_isinf(q0) ? q0 : __builtin_fmaf(rem, rs, q0));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) u[i] = rintf(v[i] / s);
        }
        if (sh.scheme == 0) {
            const float levels = (float)((1 << bits) - 1);
            const float zf = (float)zero[gi];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float q = fminf(fmaxf(u[i] + zf, 0.f), levels);
                q8[i] = (uint8_t)q;
                wh[i] = (q - zf) * s;
            }
        } else {
            const float qmax = (float)((1 << (bits - 1)) - 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float q = fminf(fmaxf(u[i], -qmax), qmax);
                q8[i] = (uint8_t)(int)(q + qmax);
                wh[i] = q * s;
            }
        }
    }
    if (codes) {
        uint32_t lo = q8[0] | (q8[1] << 8) | (q8[2] << 16) | ((uint32_t)q8[3] << 24);
        uint32_t hi = q8[4] | (q8[5] << 8) | (q8[6] << 16) | ((uint32_t)q8[7] << 24);
        *reinterpret_cast<uint2 *>(codes + e) = make_uint2(lo, hi);
    }
    if (w_hat) store8<F32>(w_hat, e, wh);
    if (w_op) store8<DT>(w_op, e, wh);
    if (want_err) {
        double e2 = 0, n2 = 0;                         // the chunk's sums, then into the matrix's
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double x = (double)v[i], d = (double)wh[i] - x;
            e2 = __builtin_fma(d, d, e2);
            n2 = __builtin_fma(x, x, n2);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            err[k] += k == m ? e2 : 0.0;
            nrm[k] += k == m ? n2 : 0.0;
        }
    }
}

template <int DT>
__global__ __launch_bounds__(256) void quantize_kernel(QuantShape sh, const void *__restrict__ w,
                                                       const float *__restrict__ scale,
                                                       const uint8_t *__restrict__ zero,
                                                       uint8_t *__restrict__ codes,
                                                       float *__restrict__ w_hat,
                                                       void *__restrict__ w_op,
                                                       double *__restrict__ werr_part,
                                                       int *__restrict__ clear, int n_clear) {
    const int64_t nchunks = (int64_t)sh.rows * sh.cols / 8;
    const int64_t c0 = (int64_t)blockIdx.x * (256 * QCPT) + threadIdx.x;
    double err[3] = {0, 0, 0}, nrm[3] = {0, 0, 0};
    float v[QCPT][8];
#pragma unroll
    for (int i = 0; i < QCPT; ++i)
        if (c0 + i * 256 < nchunks) load8<DT>(w, (c0 + i * 256) * 8, v[i]);
#pragma unroll
    for (int i = 0; i < QCPT; ++i)
        if (c0 + i * 256 < nchunks)
            quant_chunk<DT>(sh, (c0 + i * 256) * 8, v[i], scale, zero, codes, w_hat, w_op, werr_part != nullptr, err,
                            nrm);
    if (clear && blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_clear; i += 256) clear[i] = 0;
    if (!werr_part)
        return;
    // block reduction in a fixed order: wave sums, then the waves in order
    __shared__ double red[4][6];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a = wave_sum_f64(err[k]);
        const double b = wave_sum_f64(nrm[k]);
        if (lane == 0) { red[wave][2 * k] = a; red[wave][2 * k + 1] = b; }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        double t = 0;
        for (int i = 0; i < 4; ++i) t += red[i][threadIdx.x];
        werr_part[(int64_t)blockIdx.x * 6 + threadIdx.x] = t;
    }
}

// Sum of the per-block [6] partials in a fixed order, in two stages: workgroup g of at most kWerrGroups - 1
// sums the blocks g L .. g L + L - 1 (thread t every 256th from t, then the waves
// in order) into stage[g][6]; one workgroup then sums the groups (thread t group t).
constexpr int kWerrGroups = 256;

// Workgroup g sums its share of the quantizer's partials; the workgroup that finishes last sums all
// workgroups' sums (whichever it is: the order is fixed).  The sums go past the XCDs' caches and have
// arrived before the count is raised.  One launch instead of two of 5 us.
__global__ __launch_bounds__(256) void werr_reduce_kernel(const double *__restrict__ part, int nblocks, int per,
                                                          double *__restrict__ stage, int *__restrict__ ticket,
                                                          double *__restrict__ out) {
    const int g = blockIdx.x, lane = lane_id(), wave = threadIdx.x >> 6;
    __shared__ double red[4][6];
    __shared__ int last;
    auto block_sum = [&](const double (&acc)[6], auto put) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double t = wave_sum_f64(acc[k]);
            if (lane == 0) red[wave][k] = t;
        }
        __syncthreads();
        if (threadIdx.x < 6) {
            double t = 0;
            for (int i = 0; i < 4; ++i) t += red[i][threadIdx.x];
            put(t);
        }
    };
    const int b0 = g * per, b1 = min(nblocks, b0 + per);
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int i = b0 + (int)threadIdx.x; i < b1; i += 256)
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[k] += part[(int64_t)i * 6 + k];
    block_sum(acc, [&](double t) {
        __hip_atomic_store(stage + g * 6 + threadIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    });
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    const bool mine = threadIdx.x < gridDim.x;          // at most 256 workgroups
#pragma unroll
    for (int k = 0; k < 6; ++k)
        acc[k] = mine ? __hip_atomic_load(stage + threadIdx.x * 6 + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    block_sum(acc, [&](double t) { out[threadIdx.x] = t; });
}

}  // namespace

int quant_blocks(const QuantShape &sh) {
    const int64_t nchunks = (int64_t)sh.rows * sh.cols / 8;
    return (int)((nchunks + 256 * QCPT - 1) / (256 * QCPT));
}

size_t werr_scratch_doubles(const QuantShape &sh) { return (size_t)(quant_blocks(sh) + kWerrGroups) * 6; }

// the reduction's workgroups leave kWerrGroups - 1 sums at most; the last slot holds their count
static int *werr_ticket(const QuantShape &sh, double *scratch) {
    return reinterpret_cast<int *>(scratch + (size_t)(quant_blocks(sh) + kWerrGroups - 1) * 6);
}

hipError_t launch_quant_init(const QuantShape &sh, int dtype, const void *w, float *scale,
                             uint8_t *zero, hipStream_t st) {
    const dim3 grid(quant_blocks(sh)), block(256);
    switch (dtype) {
    case F32: quant_init_kernel<F32><<<grid, block, 0, st>>>(sh, w, scale, zero); break;
    case F16: quant_init_kernel<F16><<<grid, block, 0, st>>>(sh, w, scale, zero); break;
    default: quant_init_kernel<BF16><<<grid, block, 0, st>>>(sh, w, scale, zero); break;
    }
    return hipGetLastError();
}

hipError_t launch_quantize(const QuantShape &sh, int dtype, const void *w, const float *scale,
                           const uint8_t *zero, uint8_t *codes, float *w_hat, void *w_op,
                           double *werr_part, hipStream_t st, int *clear, int n_clear) {
    const dim3 grid(quant_blocks(sh)), block(256);
    if (werr_part) {                                   // launch_werr_reduce's count
        clear = werr_ticket(sh, werr_part);
        n_clear = 1;
    }
    switch (dtype) {
    case F32: quantize_kernel<F32><<<grid, block, 0, st>>>(sh, w, scale, zero, codes, w_hat, w_op, werr_part, clear, n_clear); break;
    case F16: quantize_kernel<F16><<<grid, block, 0, st>>>(sh, w, scale, zero, codes, w_hat, w_op, werr_part, clear, n_clear); break;
    default: quantize_kernel<BF16><<<grid, block, 0, st>>>(sh, w, scale, zero, codes, w_hat, w_op, werr_part, clear, n_clear); break;
    }
    return hipGetLastError();
}

hipError_t launch_werr_reduce(const QuantShape &sh, double *scratch, double *out, hipStream_t st) {
    const int nblocks = quant_blocks(sh);
    const int per = (nblocks + kWerrGroups - 2) / (kWerrGroups - 1);
    double *stage = scratch + (size_t)nblocks * 6;
    werr_reduce_kernel<<<(nblocks + per - 1) / per, 256, 0, st>>>(scratch, nblocks, per, stage, werr_ticket(sh, scratch),
                                                                 out);
    return hipGetLastError();
}

}  // namespace jab
