// Attention sharing (Sec. 3.3): the cosine similarity of Eq. 11 between the attention outputs of the
// conditional and the unconditional pass, one value per segment (a transformer block's output, a
// head, ...).  A streaming reduction: 4 bytes read per element pair, nothing else.
//   cos[s] = A_s . B_s / (|A_s| |B_s|);   0 where either vector is all zero.
// A product of two bf16 values is exact in fp32; a lane adds 64 of them in fp32 (relative error
// below 64 * 2^-24 of the sum of magnitudes), then carries on in fp64: per-wave sums are merged
// with fp64 atomic adds into three accumulators per segment, which a second kernel turns into the
// cosine.  The order of the atomic adds varies from run to run; in fp64 that moves the result
// by parts in 10^16.
#include "device_utils.h"
#include <map>
#include <mutex>

#include "trdq_internal.h"

namespace trdq {

namespace {

__global__ void fill_zero_f64_kernel(double *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

constexpr int kAhead = 4;                                             // 16-byte pieces of each operand in flight per lane

// STREAM: non-temporal loads, for operands that together exceed the 256 MB memory-side cache (at 132 MB 25.8 against 25.6 us).
template <bool STREAM>
__device__ __forceinline__ uint4 load_piece(const uint16_t *p)
{
    if constexpr (STREAM) {
        const v4i q = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(p));
        return make_uint4(q[0], q[1], q[2], q[3]);
    } else {
        return *reinterpret_cast<const uint4 *>(p);
    }
}

// One workgroup's share of a segment: chunk `c` of `chunks`, in steps of its lanes x kAhead x 8 elements; the tail
// (seg_len % 8) is taken element by element by the last chunk.  Lane 0..2 of the workgroup return the sums.
// What bounds it is the memory: 5.3 TB/s read with one piece per lane in flight and a grid that was a few workgroups
// more than one round (28 segments of 4096 x 1152: 74 chunks each, 2072 workgroups for 2048 places).
// Figures there (28 segments), before and after: 104 -> 91 us as a whole (5.1 -> 5.8 TB/s), of which four pieces in flight
// and the one round 7 and non-temporal loads 8; eight pieces in flight are no faster.
template <bool STREAM>
__device__ __forceinline__ double segment_sums(const uint16_t *__restrict__ a, const uint16_t *__restrict__ b, int64_t seg_len,
                                               int c, int chunks, double (*part)[3])
{
    const int64_t vec = seg_len / 8;                                  // whole 16-byte pieces
    const int64_t stride = (int64_t)chunks * blockDim.x;
    double dd = 0.0, da = 0.0, db = 0.0;
    float fd = 0.0f, fa = 0.0f, fb = 0.0f;
    int run = 0;
    for (int64_t i = (int64_t)c * blockDim.x + threadIdx.x; i < vec; i += kAhead * stride) {
        uint4 x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const bool in = i + u * stride < vec;                     // past the end: zeros, which add nothing
            x[u] = y[u] = make_uint4(0u, 0u, 0u, 0u);
            if (in) {
                x[u] = load_piece<STREAM>(a + (i + u * stride) * 8);
                y[u] = load_piece<STREAM>(b + (i + u * stride) * 8);
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, ys[4] = {y[u].x, y[u].y, y[u].z, y[u].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x0 = bf16_lo(xs[j]), x1 = bf16_hi(xs[j]), y0 = bf16_lo(ys[j]), y1 = bf16_hi(ys[j]);
                fd = __builtin_fmaf(x0, y0, fd); fd = __builtin_fmaf(x1, y1, fd);
                fa = __builtin_fmaf(x0, x0, fa); fa = __builtin_fmaf(x1, x1, fa);
                fb = __builtin_fmaf(y0, y0, fb); fb = __builtin_fmaf(y1, y1, fb);
            }
        }
        if (++run == 8 / kAhead) {                                    // 64 products per fp32 sum
            dd += (double)fd; da += (double)fa; db += (double)fb;
            fd = fa = fb = 0.0f;
            run = 0;
        }
    }
    dd += (double)fd; da += (double)fa; db += (double)fb;
    if (c == chunks - 1 && threadIdx.x < (unsigned)(seg_len - vec * 8)) {
        const float x0 = bf16_lo(a[vec * 8 + threadIdx.x]), y0 = bf16_lo(b[vec * 8 + threadIdx.x]);
        dd += (double)x0 * (double)y0; da += (double)x0 * (double)x0; db += (double)y0 * (double)y0;
    }
    dd = wave_sum(dd); da = wave_sum(da); db = wave_sum(db);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { part[wave][0] = dd; part[wave][1] = da; part[wave][2] = db; }
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < 3)
        for (unsigned w = 0; w < blockDim.x >> 6; ++w) t += part[w][threadIdx.x];
    return t;
}

__device__ __forceinline__ float cosine(double d, double na, double nb)
{
    return (na > 0.0 && nb > 0.0) ? (float)(d / (sqrt(na) * sqrt(nb))) : 0.0f;
}

// grid: (chunks per segment, segments)
template <bool STREAM>
__global__ __launch_bounds__(256) void cosine_accumulate_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, int64_t seg_len, int64_t stride_a,
    int64_t stride_b, double *__restrict__ acc)
{
    __shared__ double part[4][3];
    const int s = blockIdx.y;
    const double t =
        segment_sums<STREAM>(A + (int64_t)s * stride_a, B + (int64_t)s * stride_b, seg_len, blockIdx.x, gridDim.x, part);
    if (threadIdx.x < 3) atomicAdd(acc + (int64_t)s * 3 + threadIdx.x, t);
}

// Short segments: a workgroup each, the whole value in one launch (no accumulators to clear or to turn into cosines:
// the three launches take 12 us whatever the size).
__global__ __launch_bounds__(1024) void cosine_short_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, int64_t seg_len, int64_t stride_a,
    int64_t stride_b, float *__restrict__ out)
{
    __shared__ double part[16][3];
    const int s = blockIdx.x;
    const double t = segment_sums<false>(A + (int64_t)s * stride_a, B + (int64_t)s * stride_b, seg_len, 0, 1, part);
    const double na = __shfl(t, 1), nb = __shfl(t, 2);
    if (threadIdx.x == 0) out[s] = cosine(t, na, nb);
}

__global__ void cosine_finish_kernel(const double *__restrict__ acc, int n_seg, float *__restrict__ out)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_seg) return;
    out[s] = cosine(acc[s * 3], acc[s * 3 + 1], acc[s * 3 + 2]);
}

// Accumulators of the entry point that allocates nothing: three float64 sums per segment, held by
// every GPU the library runs on until the process ends (96 KB).  Host code never passes this name to
// a kernel or a runtime call: it asks for the device's address of the array once per device
// (static_scratch below) and uses that pointer.
__device__ __align__(256) double scratch[3 * kCosineStaticMaxSeg];

}  // namespace

hipError_t cosine_static_scratch(double **out)
{
    static std::mutex mu;
    static std::map<int, double *> per_device;      // each GPU holds its own copy at its own address
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    auto it = per_device.find(dev);
    if (it == per_device.end()) {
        double *ptr = nullptr;
        if (hipError_t e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)); e != hipSuccess)
            return e;
        if (!ptr) return hipErrorInvalidSymbol;
        it = per_device.emplace(dev, ptr).first;
    }
    *out = it->second;
    return hipSuccess;
}

hipError_t launch_cosine_similarity(const uint16_t *A, const uint16_t *B, int n_seg, int64_t seg_len,
                                    int64_t stride_a, int64_t stride_b, double *acc_ws, float *out, hipStream_t st)
{
    // Up to 8192 pieces of 16 bytes (eight per lane) one workgroup per segment is faster than the three launches.
    const int64_t vec = seg_len / 8;
    if (vec <= 8192) {
        const int threads = vec <= 256 ? 64 : (vec <= 1024 ? 256 : 1024);
        hipLaunchKernelGGL(cosine_short_kernel, dim3((unsigned)n_seg), dim3(threads), 0, st, A, B, seg_len, stride_a, stride_b, out);
        return hipGetLastError();
    }
    const int64_t n_acc = (int64_t)n_seg * 3;
    hipLaunchKernelGGL(fill_zero_f64_kernel, dim3((unsigned)((n_acc + 255) / 256)), dim3(256), 0, st, acc_ws, n_acc);
    // one round of eight workgroups per compute unit over all segments (not a few more), each with at least one step
    int64_t chunks = (int64_t)num_cus() * 8 / n_seg;
    const int64_t most = (vec + 256 * kAhead - 1) / (256 * kAhead);
    if (chunks > most) chunks = most;
    if (chunks < 1) chunks = 1;
    const bool stream = 4.0 * (double)n_seg * (double)seg_len > 256.0 * 1024.0 * 1024.0;
    hipLaunchKernelGGL(stream ? cosine_accumulate_kernel<true> : cosine_accumulate_kernel<false>, dim3((unsigned)chunks, (unsigned)n_seg), dim3(256), 0, st,
                       A, B, seg_len, stride_a, stride_b, acc_ws);
    hipLaunchKernelGGL(cosine_finish_kernel, dim3((unsigned)((n_seg + 255) / 256)), dim3(256), 0, st, acc_ws, n_seg, out);
    return hipGetLastError();
}

}  // namespace trdq
