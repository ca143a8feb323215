// reduce.hip -- deterministic reduction of the fused squared-error partials.
//
// Paper: eq. joint_loss (the Frobenius sum, reported as sse) and the Appendix on
// the effective weight of the KL term (the implementation's element-wise mean,
// reported as mse = sse / (B T n_heads d_head)); Appendix "Evaluation metrics in
// full", M4 (eps^A needs the teacher's sum of squares, reported alongside).
//
// Each attention wavefront leaves one (sse, sum a^2) pair in fp64.  One wavefront
// per (set, sequence) sums its pairs with a lane-strided loop and a butterfly in a
// fixed order; then one wavefront per set sums the set's sequences in a fixed order:
// the one that finishes last, whichever it is, from what all of them stored, or for
// many sequences a second launch's.  The only atomic is the count of finished
// wavefronts, so the result is bitwise reproducible.
#include "device_common.h"
#include "kernels.h"

namespace jab {
namespace {

// What the sequences of a set leave for its last wavefront goes past the XCDs' caches (agent scope)
// and has arrived before the count is raised: the wait is on the wavefront's own stores.
__device__ inline void store_agent(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double load_agent(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the sequences' sums q [batch][2] of one set (every lane of a wavefront)
__device__ inline void finish_set(const double *q, int batch, int set, int lane, const ReduceOut &r) {
    double *o = r.out + set * r.out_stride, *ps = r.per_seq ? r.per_seq + set * r.seq_stride : nullptr;
    double s0 = 0, s1 = 0;
    int k = lane;
    for (; k + 7 * 64 < batch; k += 8 * 64) {
        double x[8], y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            x[i] = load_agent(q + 2 * (k + 64 * i));
            y[i] = load_agent(q + 2 * (k + 64 * i) + 1);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s0 += x[i];
            s1 += y[i];
            if (ps) ps[k + 64 * i] = x[i];
        }
    }
    for (; k < batch; k += 64) {
        const double x = load_agent(q + 2 * k), y = load_agent(q + 2 * k + 1);
        s0 += x;
        s1 += y;
        if (ps) ps[k] = x;
    }
    s0 = wave_sum_f64(s0);
    s1 = wave_sum_f64(s1);
    if (lane == 0) {
        o[0] = s0;
        if (r.stats) {
            o[1] = s0 * r.inv[set];
            o[2] = s1;
        }
    }
}

// Bound by latency: at 16 x 2048 tokens of 32 heads a wavefront sums 2048 pairs, eight loads in flight.
// One launch (tickets) instead of two of 5 us while the wavefronts are few: their counts go one after the
// other, 11 ns each, whichever set they belong to.  us, one launch / two: 16 sequences of 2048 tokens 6 / 20 (the second
// launch with its loads one by one), 300 of 97 8.0 / 8.5, 1024 of 33 20.7 / 8.7, 2730 of 24
// 51 / 11, 8192 of 1 143 / 16, 64 sets of 4096 2770 / 64.
constexpr int kOneLaunchWaves = 512;

__global__ __launch_bounds__(64) void reduce_kernel(const double *__restrict__ part, int batch, int per_seq,
                                                    double *__restrict__ seq_sums, int *__restrict__ tickets,
                                                    ReduceOut r) {
    const int b = blockIdx.x, set = blockIdx.y, lane = lane_id();
    const double2 *p = reinterpret_cast<const double2 *>(part) + ((int64_t)set * batch + b) * per_seq;
    double s0 = 0, s1 = 0;
    int i = lane;
    for (; i + 7 * 64 < per_seq; i += 8 * 64) {
        double2 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = p[i + 64 * k];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            s0 += v[k].x;
            s1 += v[k].y;
        }
    }
    for (; i < per_seq; i += 64) {
        const double2 v = p[i];
        s0 += v.x;
        s1 += v.y;
    }
    s0 = wave_sum_f64(s0);
    s1 = wave_sum_f64(s1);
    double *q = seq_sums + (int64_t)set * batch * 2;
    int last = 0;
    if (lane == 0) {
        store_agent(q + 2 * b, s0);
        store_agent(q + 2 * b + 1, s1);
        if (tickets) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            last = __hip_atomic_fetch_add(tickets + set, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == batch - 1;
        }
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    asm volatile("" ::: "memory");
    finish_set(q, batch, set, lane, r);
}

__global__ __launch_bounds__(64) void reduce_sets_kernel(const double *__restrict__ seq_sums, int batch, ReduceOut r) {
    finish_set(seq_sums + (int64_t)blockIdx.x * batch * 2, batch, blockIdx.x, lane_id(), r);
}

}  // namespace

hipError_t launch_reduce(const double *partials, int n_sets, int batch, int per_seq, double *seq_sums, int *tickets,
                         const ReduceOut &r, hipStream_t st) {
    const bool one = (int64_t)batch * n_sets <= kOneLaunchWaves;
    reduce_kernel<<<dim3(batch, n_sets), dim3(64), 0, st>>>(partials, batch, per_seq, seq_sums, one ? tickets : nullptr, r);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || one) return e;
    reduce_sets_kernel<<<dim3(n_sets), dim3(64), 0, st>>>(seq_sums, batch, r);
    return hipGetLastError();
}

namespace {
constexpr int SUMSQ_BLOCKS = 256;   // partial sums per unit

// stage 1: block (b, u) sums the squares of its contiguous chunk of unit u's elements
// (float4 loads, fp64 accumulation, fixed lane and wave order)
__global__ __launch_bounds__(256) void unit_sumsq_kernel(const float *__restrict__ a, int64_t d, UnitRows rows,
                                                         double *__restrict__ part) {
    const int u = blockIdx.y, b = blockIdx.x, tid = threadIdx.x;
    const int64_t n4 = (rows.r[u + 1] - rows.r[u]) * d / 4;
    const float4 *src = reinterpret_cast<const float4 *>(a + rows.r[u] * d);
    const int64_t chunk = (n4 + SUMSQ_BLOCKS - 1) / SUMSQ_BLOCKS;
    const int64_t i0 = (int64_t)b * chunk, i1 = i0 + chunk < n4 ? i0 + chunk : n4;
    double acc = 0.0;
    for (int64_t i = i0 + tid; i < i1; i += 256) {
        const float4 v = src[i];
        acc += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
    }
    acc = wave_sum_f64(acc);
    __shared__ double wsum[4];
    if (lane_id() == 0) wsum[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) part[u * SUMSQ_BLOCKS + b] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// stage 2: one wavefront per unit sums its partials
__global__ __launch_bounds__(64) void unit_sumsq_final_kernel(const double *__restrict__ part,
                                                              double *__restrict__ out) {
    const int u = blockIdx.x, lane = lane_id();
    double acc = 0.0;
    for (int i = lane; i < SUMSQ_BLOCKS; i += 64) acc += part[u * SUMSQ_BLOCKS + i];
    acc = wave_sum_f64(acc);
    if (lane == 0) out[u] = acc;
}
}  // namespace

size_t unit_sumsq_part_bytes(int n_units) { return (size_t)n_units * SUMSQ_BLOCKS * sizeof(double); }

hipError_t launch_unit_sumsq(const float *a, int64_t d, const UnitRows &rows, int n_units, double *part,
                             double *out, hipStream_t st) {
    if (n_units < 1 || n_units > 3 || d % 4) return hipErrorInvalidValue;
    unit_sumsq_kernel<<<dim3(SUMSQ_BLOCKS, n_units), dim3(256), 0, st>>>(a, d, rows, part);
    unit_sumsq_final_kernel<<<dim3(n_units), dim3(64), 0, st>>>(part, out);
    return hipGetLastError();
}

}  // namespace jab
