// prepare_weights: H_t(W) = R^T . (Delta_t^-1 . W) of Eq. 10 and the symmetric weight
// quantiser (per output channel for int8, per 128-row group and output channel for int4).
// Offline, once per time-step group.
//
// What bounds it: W is read (4 bytes an element) and the codes are written twice (row-major and
// block-tiled), 6 bytes an element, 32 MB for a 1152 x 4608 set; the rest of a set's preparation is the
// host's: device allocations and the final synchronisation.  So one Hadamard rotation goes without the
// float32 scratch matrix that used to carry the rotated weights from one kernel to the next: int4 codes
// need the maximum of their own 128-row block only and take one kernel, int8 codes need the maximum of
// the whole column, which a first pass finds and a second one, rotating again from W (which the
// memory-side cache still holds), uses.  The quantising kernel also writes the block-tiled codes and the
// column sums, which were kernels of their own.
#include "device_utils.h"
#include "trdq_internal.h"

namespace trdq {

namespace {

constexpr int kCols = 64;          // output channels per workgroup
constexpr int kPrepThreads = 256;

// A workgroup holds one 128-row block of 64 columns: wave q the rows 32 q .. 32 q + 31, a lane one column.
// Loads the block into v, row k through perm (clamped to the matrix) when a permutation is given -- the
// P^T factor of Eq. 9 in front of the second rotation --, divided by the diagonal.
__device__ __forceinline__ void load_block(const float *__restrict__ W, int K, int N, const float *__restrict__ diag,
                                           const int32_t *__restrict__ perm, int b, int q, int n, bool col_ok,
                                           float (&v)[32])
{
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        int row = b * kBlock + 32 * q + i;
        if (perm) {
            row = perm[row];
            row = row < 0 ? 0 : (row >= K ? K - 1 : row);
        }
        v[i] = col_ok ? W[(size_t)row * N + n] : 0.0f;
    }
    if (diag) {
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = v[i] / diag[b * kBlock + 32 * q + i];
    }
}

// Unnormalised H_128 down the column: five butterfly stages inside the lane, the last two across the four
// waves through LDS (one exchange: a lane reads the other waves' values of its row numbers and forms its
// own of the four results).
__device__ __forceinline__ void rotate_block(float (&v)[32], int q, int c, float (&tile)[kBlock][kCols])
{
#pragma unroll
    for (int h = 1; h < 32; h <<= 1) {
#pragma unroll
        for (int i0 = 0; i0 < 32; i0 += 2 * h) {
#pragma unroll
            for (int i = i0; i < i0 + h; ++i) {
                const float a = v[i], bb = v[i + h];
                v[i] = a + bb;
                v[i + h] = a - bb;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) tile[32 * q + i][c] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const float t0 = tile[i][c], t1 = tile[32 + i][c], t2 = tile[64 + i][c], t3 = tile[96 + i][c];
        const float lo = (q & 1) ? t0 - t1 : t0 + t1, hi = (q & 1) ? t2 - t3 : t2 + t3;
        v[i] = (q & 2) ? lo - hi : lo + hi;
    }
}

// Rotation of the whole matrix into a scratch matrix (in front of a permutation, or of the asymmetric quantiser):
//   Wrot[b*128 + j, n] = sum_k H[k][j] * W[b*128 + k, n] / d[b*128 + k]      (unnormalised H)
__global__ __launch_bounds__(kPrepThreads) void prepare_rotate_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, float *__restrict__ Wrot)
{
    __shared__ float tile[kBlock][kCols];
    const int b = blockIdx.y, c = threadIdx.x % kCols, q = __builtin_amdgcn_readfirstlane(threadIdx.x / kCols);
    const int n = blockIdx.x * kCols + c;
    const bool col_ok = n < N;
    float v[32];
    load_block(W, K, N, diag, nullptr, b, q, n, col_ok, v);
    rotate_block(v, q, c, tile);
    if (!col_ok) return;
#pragma unroll
    for (int i = 0; i < 32; ++i) Wrot[(size_t)(b * kBlock + 32 * q + i) * N + n] = v[i];
}

// First pass of the int8 quantiser: amax[b, n] = the largest magnitude of the rotated block.  Also clears the
// column sums that the second pass adds to, and copies the diagonal for a handle that keeps one.
__global__ __launch_bounds__(kPrepThreads) void prepare_absmax_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag,
    const int32_t *__restrict__ perm, float *__restrict__ amax, int32_t *__restrict__ colsum,
    float *__restrict__ diag_copy)
{
    __shared__ float tile[kBlock][kCols];
    __shared__ float part[4][kCols];
    const int b = blockIdx.y, c = threadIdx.x % kCols, q = __builtin_amdgcn_readfirstlane(threadIdx.x / kCols);
    const int n = blockIdx.x * kCols + c;
    const bool col_ok = n < N;
    float v[32];
    load_block(W, K, N, diag, perm, b, q, n, col_ok, v);
    if (diag_copy && blockIdx.x == 0 && threadIdx.x < kBlock)
        diag_copy[b * kBlock + threadIdx.x] = diag[b * kBlock + threadIdx.x];
    rotate_block(v, q, c, tile);
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) m = fmaxf(m, fabsf(v[i]));
    part[q][c] = m;
    __syncthreads();
    if (q == 0 && col_ok) {
        amax[(size_t)b * N + n] = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
        if (b == 0) colsum[n] = 0;
    }
}

// The rotation with a dense block in place of the butterflies (H_t(W) = R^T (Delta^-1 W) with
// the blocks of the BlockDiag equation as arbitrary orthogonal matrices):
//   Wrot[b*128 + j, n] = sum_k R_b[k][j] * W[b*128 + k, n] / d[b*128 + k]
// Wave q of the workgroup produces rows j = 32 q .. 32 q + 31 of 64 columns; the row of R_b it
// needs at step k is the same for all its lanes (scalar loads), the column of W comes from LDS.
__global__ __launch_bounds__(kPrepThreads) void prepare_rotate_dense_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, const int32_t *__restrict__ perm,
    const float *__restrict__ R, float *__restrict__ Wrot, float *__restrict__ amax)
{
    __shared__ float tile[kBlock][kCols + 1];
    __shared__ float part[4][kCols];
    const int b = blockIdx.y;
    const int n0 = blockIdx.x * kCols;
    const int c = threadIdx.x % kCols;
    const int q = __builtin_amdgcn_readfirstlane(threadIdx.x / kCols);     // 0..3, one wave each
    const int n = n0 + c;
    const bool col_ok = n < N;
    for (int k = q; k < kBlock; k += 4) {
        float w = 0.0f;
        if (col_ok) {
            int row = b * kBlock + k;
            if (perm) {                                  // the P^T factor in front of a second rotation
                row = perm[row];
                row = row < 0 ? 0 : (row >= K ? K - 1 : row);
            }
            w = W[(size_t)row * N + n];
            if (diag) w = w / diag[b * kBlock + k];
        }
        tile[k][c] = w;
    }
    __syncthreads();
    float acc[32];
#pragma unroll
    for (int jj = 0; jj < 32; ++jj) acc[jj] = 0.0f;
    const float *Rb = R + (size_t)b * kBlock * kBlock + 32 * q;
    for (int k = 0; k < kBlock; ++k) {
        const float w = tile[k][c];
#pragma unroll
        for (int jj = 0; jj < 32; ++jj) acc[jj] = __builtin_fmaf(Rb[k * kBlock + jj], w, acc[jj]);
    }
    float m = 0.0f;
#pragma unroll
    for (int jj = 0; jj < 32; ++jj) {
        m = fmaxf(m, fabsf(acc[jj]));
        if (col_ok) Wrot[(size_t)(b * kBlock + 32 * q + jj) * N + n] = acc[jj];
    }
    part[q][c] = m;
    __syncthreads();
    if (q == 0 && col_ok)
        amax[(size_t)b * N + n] = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
}

// Quantises one 128-row block of 64 columns into the layouts the product kernels read (see Weights in
// trdq_internal.h): K-contiguous rows, and where `tiled` is given the block-tiled copy.
//   wbits 8: scale[n]    = max_b amax[b, n] * norm / 127   (qmax = 31 in the same layout: 6-bit codes)
//   wbits 4: scale[b, n] = max over the block * norm / 7
// norm undoes the unnormalised butterflies: 1/sqrt(128) after one rotation, 1/128 after two.
//   code = rint(w * qmax / amax)   (ties to even; amax == 0 -> 0)
// ROTATE: W is rotated here (int4 codes then find their maximum here, too); otherwise W holds rotated
// values and amax their block maxima.  A lane ends with 32 consecutive codes of one channel: two
// 16-byte pieces of its row (a 128-byte line per channel from the four waves), 256 consecutive bytes
// over 16 lanes in the tiled form.  Measured, average over the four int8 linears of a block of width 1152: 9 us
// for the maxima and 10 us here, against 34 + 17 + 7 + 6 us for rotation, quantiser, column sums and
// second copy as kernels of their own with float32 values between them.
template <int WBITS, bool ROTATE>
__global__ __launch_bounds__(kPrepThreads) void prepare_quant_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, const int32_t *__restrict__ perm,
    const float *__restrict__ amax, float norm, float qmax, void *__restrict__ codes, void *__restrict__ tiled,
    float *__restrict__ scales, int32_t *__restrict__ colsum, float *__restrict__ diag_copy)
{
    __shared__ float tile[kBlock][kCols];
    __shared__ float part[4][kCols];
    const int nb = K / kBlock;
    const int b = blockIdx.y, c = threadIdx.x % kCols, q = __builtin_amdgcn_readfirstlane(threadIdx.x / kCols);
    const int n = blockIdx.x * kCols + c;
    const bool col_ok = n < N;
    float v[32];
    load_block(W, K, N, ROTATE ? diag : nullptr, ROTATE ? perm : nullptr, b, q, n, col_ok, v);
    float a = 0.0f;
    if (WBITS == 8) {
        if (col_ok)
            for (int bb = q; bb < nb; bb += 4) a = fmaxf(a, amax[(size_t)bb * N + n]);
    } else {
        if (diag_copy && blockIdx.x == 0 && threadIdx.x < kBlock)
            diag_copy[b * kBlock + threadIdx.x] = diag[b * kBlock + threadIdx.x];
        if (!ROTATE && col_ok) a = amax[(size_t)b * N + n];
    }
    if (ROTATE) rotate_block(v, q, c, tile);
    if (WBITS == 4 && ROTATE) {
#pragma unroll
        for (int i = 0; i < 32; ++i) a = fmaxf(a, fabsf(v[i]));
    }
    part[q][c] = a;
    __syncthreads();
    a = fmaxf(fmaxf(part[0][c], part[1][c]), fmaxf(part[2][c], part[3][c]));
    if (q == 0 && col_ok) {
        if (WBITS == 4) scales[(size_t)b * N + n] = a * (norm / qmax);
        else if (b == 0) scales[n] = a * (norm / qmax);
    }
    const float inv = a > 0.0f ? qmax / a : 0.0f;
    uint32_t u[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) u[i] = quant_bits(v[i], inv);
    const int k0 = b * kBlock + 32 * q;                // the lane's first input channel
    if (WBITS == 8) {
        if (colsum) {
            int t = 0;
#pragma unroll
            for (int i = 0; i < 32; ++i) t += (int)(int8_t)(u[i] & 0xFF);
            __syncthreads();
            part[q][c] = __int_as_float(t);
            __syncthreads();
            if (q == 0 && col_ok)
                atomicAdd(colsum + n, __float_as_int(part[0][c]) + __float_as_int(part[1][c]) +
                                          __float_as_int(part[2][c]) + __float_as_int(part[3][c]));
        }
        if (!col_ok) return;
        int8_t *const out = static_cast<int8_t *>(codes) + (size_t)n * K + k0;
        int8_t *const blk = static_cast<int8_t *>(tiled) + ((size_t)(n >> 4) * (K >> 6) + (k0 >> 6)) * 1024 +
                            ((k0 & 63) >> 4) * 256 + (n & 15) * 16;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                w[j] = pack4_low_bytes(u[16 * p + 4 * j], u[16 * p + 4 * j + 1], u[16 * p + 4 * j + 2], u[16 * p + 4 * j + 3]);
            const uint4 piece = make_uint4(w[0], w[1], w[2], w[3]);
            *reinterpret_cast<uint4 *>(out + 16 * p) = piece;
            if (tiled) *reinterpret_cast<uint4 *>(blk + 256 * p) = piece;
        }
    } else {
        if (!col_ok) return;
        // 8 consecutive k -> 4 bytes: byte j = code(k0+j) & 0xF | (code(k0+4+j) & 0xF) << 4
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t lo = pack4_low_bytes(u[8 * j], u[8 * j + 1], u[8 * j + 2], u[8 * j + 3]);
            const uint32_t hi = pack4_low_bytes(u[8 * j + 4], u[8 * j + 5], u[8 * j + 6], u[8 * j + 7]);
            w[j] = (lo & 0x0F0F0F0Fu) | ((hi << 4) & 0xF0F0F0F0u);
        }
        *reinterpret_cast<uint4 *>(static_cast<uint8_t *>(codes) + (size_t)n * (K / 2) + k0 / 2) =
            make_uint4(w[0], w[1], w[2], w[3]);
        if (tiled) {
            // units of 16 input channels (8 bytes), see qgemm_tiled.hip
            uint8_t *const blk = static_cast<uint8_t *>(tiled) + ((size_t)(n >> 4) * (K >> 6) + (k0 >> 6)) * 512 +
                                 ((k0 & 63) >> 4) * 128 + (n & 15) * 8;
            *reinterpret_cast<uint2 *>(blk) = make_uint2(w[0], w[1]);
            *reinterpret_cast<uint2 *>(blk + 128) = make_uint2(w[2], w[3]);
        }
    }
}

// Asymmetric weights (Eq. 1-3 on H_t(W), one range per output channel).  Kernel A: lo[n] = min(min_k Wrot[k,n], 0),
// hi[n] = max(max_k Wrot[k,n], 0) over the whole column, one thread per channel.
__global__ __launch_bounds__(kPrepThreads) void column_minmax_kernel(const float *__restrict__ Wrot, int K, int N,
                                                                      float *__restrict__ lo, float *__restrict__ hi)
{
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float a = 0.0f, b = 0.0f;
    for (int k = 0; k < K; ++k) {
        const float w = Wrot[(size_t)k * N + n];
        a = fminf(a, w);
        b = fmaxf(b, w);
    }
    lo[n] = a;
    hi[n] = b;
}

// Kernel B: s[n] = (hi - lo) * norm / 255, z[n] = -rint(lo * 255 / (hi - lo)), code = clamp(rint(w * 255 / (hi - lo)) + z,
// 0, 255), stored as code - 128 (the operand type of the int8 matrix instruction) in the [N, K] layout; zcw[n] = 128 - z,
// so that q - z = stored + zcw.  The integer offset rides in the rounding constant of one fused multiply-add.
__global__ __launch_bounds__(kPrepThreads) void prepare_quant_asym_kernel(
    const float *__restrict__ Wrot, const float *__restrict__ lo, const float *__restrict__ hi, int K, int N, float norm,
    int8_t *__restrict__ codes, float *__restrict__ scales, int32_t *__restrict__ zcw)
{
    __shared__ int8_t q8[kCols][kBlock + 16];
    __shared__ float inv_s[kCols], magic_s[kCols];
    const int b = blockIdx.y;
    const int n0 = blockIdx.x * kCols;
    if (threadIdx.x < kCols) {
        const int n = n0 + threadIdx.x;
        float inv = 0.0f, z = 0.0f;
        if (n < N) {
            const float range = hi[n] - lo[n];
            inv = range > 0.0f ? 255.0f / range : 0.0f;
            z = -rintf(lo[n] * inv);
            if (b == 0) {
                scales[n] = range * (norm / 255.0f);
                zcw[n] = 128 - (int)z;
            }
        }
        inv_s[threadIdx.x] = inv;
        magic_s[threadIdx.x] = kRoundMagic + (z - 128.0f);
    }
    __syncthreads();
    const int c = threadIdx.x % kCols;
    const int q = threadIdx.x / kCols;
    const int n = n0 + c;
    for (int k = q; k < kBlock; k += 4) {
        const float w = n < N ? Wrot[(size_t)(b * kBlock + k) * N + n] : 0.0f;
        const float t = __builtin_fmaf(w, inv_s[c], magic_s[c]);
        q8[c][k] = (int8_t)(__float_as_uint(__builtin_amdgcn_fmed3f(t, kRoundMagic - 128.0f, kRoundMagic + 127.0f)) & 0xFF);
    }
    __syncthreads();
    for (int ch = threadIdx.x; ch < kCols * (kBlock / 16); ch += kPrepThreads) {
        const int cc = ch / (kBlock / 16), kk = (ch % (kBlock / 16)) * 16;
        if (n0 + cc < N)
            *reinterpret_cast<uint4 *>(codes + (size_t)(n0 + cc) * K + b * kBlock + kk) =
                *reinterpret_cast<const uint4 *>(&q8[cc][kk]);
    }
}

// colsum[n] = sum_k codes[n][k]: one wave per output channel (the zero-point term of asymmetric
// activations needs it in the product's epilogue)
__global__ __launch_bounds__(64) void weight_colsum_kernel(const int8_t *__restrict__ codes, int K, int N,
                                                           int32_t *__restrict__ colsum)
{
    const int n = blockIdx.x;
    const int8_t *row = codes + (size_t)n * K;
    int t = 0;
    for (int k = threadIdx.x * 16; k < K; k += 64 * 16) {
        const int4 v = *reinterpret_cast<const int4 *>(row + k);
        const int wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            t += (int)(int8_t)(wv[u] & 0xFF) + (int)(int8_t)((wv[u] >> 8) & 0xFF) +
                 (int)(int8_t)((wv[u] >> 16) & 0xFF) + (wv[u] >> 24);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if (threadIdx.x == 0) colsum[n] = t;
}

}  // namespace

hipError_t launch_prepare_quant_asym(const float *Wrot, float *lohi, int K, int N, float norm, void *codes, float *scales,
                                     int32_t *zcw, hipStream_t st)
{
    float *lo = lohi, *hi = lohi + N;
    hipLaunchKernelGGL(column_minmax_kernel, dim3((N + kPrepThreads - 1) / kPrepThreads), dim3(kPrepThreads), 0, st, Wrot, K, N,
                       lo, hi);
    dim3 grid((N + kCols - 1) / kCols, K / kBlock);
    hipLaunchKernelGGL(prepare_quant_asym_kernel, grid, dim3(kPrepThreads), 0, st, Wrot, lo, hi, K, N, norm,
                       static_cast<int8_t *>(codes), scales, zcw);
    return hipGetLastError();
}

// rowsum[i] = sum_k Xq[i][k]: one wave per token (the zero-point term of asymmetric weights needs it)
__global__ __launch_bounds__(256) void xq_rowsum_kernel(const int8_t *__restrict__ Xq, int64_t M, int K,
                                                        int32_t *__restrict__ rowsum)
{
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= M) return;
    const int lane = threadIdx.x & 63;
    const int8_t *row = Xq + i * K;
    int t = 0;
    for (int k = lane * 16; k < K; k += 64 * 16) {
        const int4 v = *reinterpret_cast<const int4 *>(row + k);
        const int wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            t += (int)(int8_t)(wv[u] & 0xFF) + (int)(int8_t)((wv[u] >> 8) & 0xFF) +
                 (int)(int8_t)((wv[u] >> 16) & 0xFF) + (wv[u] >> 24);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if (lane == 0) rowsum[i] = t;
}

hipError_t launch_xq_rowsum(const int8_t *Xq, int64_t M, int K, int32_t *rowsum, hipStream_t st)
{
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(xq_rowsum_kernel, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, st, Xq, M, K, rowsum);
    return hipGetLastError();
}

hipError_t launch_weight_colsum(const void *codes, int K, int N, int32_t *colsum, hipStream_t st)
{
    hipLaunchKernelGGL(weight_colsum_kernel, dim3(N), dim3(64), 0, st, static_cast<const int8_t *>(codes), K, N, colsum);
    return hipGetLastError();
}

hipError_t launch_prepare_rotate(const float *W, int K, int N, const float *diag, float *Wrot, hipStream_t st)
{
    dim3 grid((N + kCols - 1) / kCols, K / kBlock);
    hipLaunchKernelGGL(prepare_rotate_kernel, grid, dim3(kPrepThreads), 0, st, W, K, N, diag, Wrot);
    return hipGetLastError();
}

// int4 weights: colsumw[n] = 16 * sum_g s_w[g][n] * (sum over the 128 codes of group g), one wave per
// output channel; a lane sums two packed bytes (four codes) per group.
__global__ __launch_bounds__(64) void weight_colsumw4_kernel(const uint8_t *__restrict__ codes, const float *__restrict__ scales,
                                                             int K, int N, float *__restrict__ colsumw)
{
    const int n = blockIdx.x, lane = threadIdx.x;
    const uint8_t *row = codes + (size_t)n * (K / 2);
    float t = 0.0f;
    for (int g = 0; g < K / kBlock; ++g) {
        // 64 bytes per group; lane takes byte `lane`: two codes as signed nibbles
        const uint32_t b = row[g * 64 + lane];
        int s = (int)((b & 0xF) ^ 8) - 8 + (int)(((b >> 4) & 0xF) ^ 8) - 8;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        t += scales[(size_t)g * N + n] * (float)s;
    }
    if (lane == 0) colsumw[n] = 16.0f * t;
}

hipError_t launch_prepare_rotate_dense(const float *W, int K, int N, const float *diag, const int32_t *perm,
                                       const float *R, float *Wrot, float *amax, hipStream_t st)
{
    dim3 grid((N + kCols - 1) / kCols, K / kBlock);
    hipLaunchKernelGGL(prepare_rotate_dense_kernel, grid, dim3(kPrepThreads), 0, st, W, K, N, diag, perm, R, Wrot, amax);
    return hipGetLastError();
}

hipError_t launch_prepare_quant(const float *W, const float *diag, const int32_t *perm, bool rotate, float norm,
                                const Weights &w, float *amax, float *diag_copy, hipStream_t st)
{
    const int K = w.K, N = w.N;
    const dim3 grid((N + kCols - 1) / kCols, K / kBlock), threads(kPrepThreads);
    if (!diag) diag_copy = nullptr;
    if (w.wbits == 4) {
        auto kern = rotate ? prepare_quant_kernel<4, true> : prepare_quant_kernel<4, false>;
        hipLaunchKernelGGL(kern, grid, threads, 0, st, W, K, N, diag, perm, amax, norm, 7.0f, w.codes, w.codes_tiled,
                           w.scales, nullptr, diag_copy);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        hipLaunchKernelGGL(weight_colsumw4_kernel, dim3(N), dim3(64), 0, st, static_cast<const uint8_t *>(w.codes), w.scales,
                           K, N, w.colsumw);
        return hipGetLastError();
    }
    const float qmax = w.qbits == 6 ? 31.0f : 127.0f;
    if (rotate) {
        hipLaunchKernelGGL(prepare_absmax_kernel, grid, threads, 0, st, W, K, N, diag, perm, amax, w.colsum, diag_copy);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        hipLaunchKernelGGL((prepare_quant_kernel<8, true>), grid, threads, 0, st, W, K, N, diag, perm, amax, norm, qmax,
                           w.codes, w.codes_tiled, w.scales, w.colsum, nullptr);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((prepare_quant_kernel<8, false>), grid, threads, 0, st, W, K, N, diag, perm, amax, norm, qmax,
                       w.codes, w.codes_tiled, w.scales, nullptr, nullptr);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    return launch_weight_colsum(w.codes, K, N, w.colsum, st);
}

}  // namespace trdq
