// prepare_weights: H_t(W) = R^T . (Delta_t^-1 . W) of Eq. 10 and the symmetric weight
// quantiser (per output channel for int8, per 128-row group and output channel for int4).
// Offline, once per time-step group.
//
// What bounds it: W is read (4 bytes an element) and the codes are written twice (row-major and
// block-tiled; int4 a third time, widened), 6 bytes an element, 32 MB for a 1152 x 4608 set; the rest of a set's preparation is the
// host's: device allocations and the final synchronisation.  One Hadamard rotation goes without a float32 scratch matrix:
// one kernel reads W, rotates, finds the maxima, and writes codes, scales and column sums (two for some sets: prepare_takes_pair).
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
                                           const int32_t *__restrict__ perm, int b, int q, int n, bool col_ok, float (&v)[32])
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

// The rotation with a dense block in place of the butterflies (H_t(W) = R^T (Delta^-1 W) with
// the blocks of the BlockDiag equation as arbitrary orthogonal matrices):
//   Wrot[b*128 + j, n] = sum_k R_b[k][j] * W[b*128 + k, n] / d[b*128 + k]
// Wave q of the workgroup produces rows j = 32 q .. 32 q + 31 of 64 columns; the row of R_b it
// needs at step k is the same for all its lanes (scalar loads), the column of W comes from LDS.
__global__ __launch_bounds__(kPrepThreads) void prepare_rotate_dense_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, const int32_t *__restrict__ perm,
    const float *__restrict__ R, float *__restrict__ Wrot)
{
    __shared__ float tile[kBlock][kCols + 1];
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
    if (!col_ok) return;
#pragma unroll
    for (int jj = 0; jj < 32; ++jj) Wrot[(size_t)(b * kBlock + 32 * q + jj) * N + n] = acc[jj];
}

// The symmetric quantiser as a kernel for the block maxima (8 bits) and one for the codes, a workgroup to 128 rows of 64
// columns: for the rows and sets that the one kernel below is slower for (prepare_takes_pair).
// First pass of the 8-bit quantiser: amax[b, n] = the largest magnitude of the rotated block.  Also clears the
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

// Codes of one 128-row block of 64 columns, in the layouts and by the rounding of the kernel below; int4 codes find their maximum here.
// A lane ends with 32 consecutive codes of one channel: two 16-byte pieces of its row (a 128-byte line per channel from the
// four waves), 256 consecutive bytes over 16 lanes in the tiled form.
template <int WBITS, bool ROTATE>
__global__ __launch_bounds__(kPrepThreads) void prepare_quant_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, const int32_t *__restrict__ perm,
    const float *__restrict__ amax, float norm, float qmax, void *__restrict__ codes, void *__restrict__ tiled, void *__restrict__ wide,
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
    } else if (diag_copy && blockIdx.x == 0 && threadIdx.x < kBlock) {
        diag_copy[b * kBlock + threadIdx.x] = diag[b * kBlock + threadIdx.x];
    }
    if (ROTATE) rotate_block(v, q, c, tile);
    if (WBITS == 4) {
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
    const size_t block = (size_t)(n >> 4) * (K >> 6) + (k0 >> 6);
    if (WBITS == 8) {
        int t = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) t += (int)(int8_t)(u[i] & 0xFF);
        __syncthreads();
        part[q][c] = __int_as_float(t);
        __syncthreads();
        if (q == 0 && col_ok)
            atomicAdd(colsum + n, __float_as_int(part[0][c]) + __float_as_int(part[1][c]) +
                                      __float_as_int(part[2][c]) + __float_as_int(part[3][c]));
        if (!col_ok) return;
        int8_t *const out = static_cast<int8_t *>(codes) + (size_t)n * K + k0;
        int8_t *const blk = static_cast<int8_t *>(tiled) + block * 1024 + ((k0 & 63) >> 4) * 256 + (n & 15) * 16;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                w[j] = pack4_low_bytes(u[16 * p + 4 * j], u[16 * p + 4 * j + 1], u[16 * p + 4 * j + 2], u[16 * p + 4 * j + 3]);
            const uint4 piece = make_uint4(w[0], w[1], w[2], w[3]);
            *reinterpret_cast<uint4 *>(out + 16 * p) = piece;
            *reinterpret_cast<uint4 *>(blk + 256 * p) = piece;
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
        uint8_t *const blk = static_cast<uint8_t *>(tiled) + block * 512 + ((k0 & 63) >> 4) * 128 + (n & 15) * 8;
        uint8_t *const bytes = static_cast<uint8_t *>(wide) + block * 1024 + ((k0 & 63) >> 4) * 256 + (n & 15) * 16;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            *reinterpret_cast<uint2 *>(blk + 128 * p) = make_uint2(w[2 * p], w[2 * p + 1]);
            if (wide)
                *reinterpret_cast<uint4 *>(bytes + 256 * p) = make_uint4((w[2 * p] << 4) & 0xF0F0F0F0u, w[2 * p] & 0xF0F0F0F0u,
                                                                         (w[2 * p + 1] << 4) & 0xF0F0F0F0u, w[2 * p + 1] & 0xF0F0F0F0u);
        }
    }
}

// int4 weights: colsumw[n] = 16 * sum_g s_w[g][n] * (sum over the 128 codes of group g), one wave per
// output channel; a lane sums the two codes of a byte per group.
__global__ __launch_bounds__(64) void weight_colsumw4_kernel(const uint8_t *__restrict__ codes, const float *__restrict__ scales,
                                                             int K, int N, float *__restrict__ colsumw)
{
    const int n = blockIdx.x, lane = threadIdx.x;
    const uint8_t *row = codes + (size_t)n * (K / 2);
    float t = 0.0f;
    for (int g = 0; g < K / kBlock; ++g) {
        const uint32_t b = row[g * 64 + lane];
        int s = (int)((b & 0xF) ^ 8) - 8 + (int)(((b >> 4) & 0xF) ^ 8) - 8;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        t += scales[(size_t)g * N + n] * (float)s;
    }
    if (lane == 0) colsumw[n] = 16.0f * t;
}

// The symmetric quantiser, rotation included.  A workgroup owns eight output channels for the whole K: a wave takes a
// 128-row block of them (the blocks wave, wave + nw, ...), a lane 16 rows of one channel, so the rotation stays inside the
// wave (four stages in the lane, three across lanes), the column maximum crosses the waves through LDS, and W is read once.
//   wbits 8: scale[n]    = max over the column * norm / 127   (qmax = 31 in the same layout: 6-bit codes)
//   wbits 4: scale[b, n] = max over the block * norm / 7
// norm undoes the unnormalised butterflies: 1/sqrt(128) after one rotation, 1/128 after two.
//   code = rint(w * qmax / amax)   (ties to even; amax == 0 -> 0)
// ROTATE: W is rotated here (rows through perm, divided by diag, both optional); otherwise it holds rotated values.
// HOLD (8 bits): blocks that a wave keeps in registers between the maximum and the codes: 1 up to 16 blocks, 3 up to 48.
// A lane's 16 codes are one 16-byte piece of both layouts; eight channels and eight pieces make 128-byte runs in each.
// A line of W is shared by four workgroups, which therefore run on the same die.
// What bounds it is the chain of one block through a wave (of three at K = 4608), then the 128-byte lines that four workgroups
// share.  The form before (workgroups of 64 channels x 128 rows, one kernel for the maxima and one that read and rotated W
// again for the codes) took 8.2 + 9.7 us for a 1152 x 1152 int8 set, 7.8 + 9.3 for 1152 x 3456, 9.4 + 11.4 for 1152 x 4608 and
// 8.2 + 9.7 for 4608 x 1152; this one 6.5, 8.3, 12.9 and 16.7 (int4, one kernel and one for the sums, without widened codes: 6.8 + 6.8,
// 10.2 + 5.8, 11.3 + 6.5 and 11.8 + 11.6; now, with them, 6.8, 11.3, 17.0 and 18.2).
constexpr int kPcCols = 8;
constexpr int kPcMostWaves = 16;

__device__ __forceinline__ void exchange_stage(float &a, float &b, bool wide)
{
    // two values' butterflies with the lane 16 (32) away: after the first exchange one register holds both values' lower
    // halves and the other their upper ones; the second one puts sums and differences where they belong
    auto swap = [&](float &x, float &y) {
        const auto r = wide ? __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false)
                            : __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        x = __uint_as_float(r[0]);
        y = __uint_as_float(r[1]);
    };
    swap(a, b);
    const float sum = a + b, diff = a - b;
    a = sum;
    b = diff;
    swap(a, b);
}

// Unnormalised H_128 over the 16 rows of a lane and the eight lanes of a channel (row bits 4, 5, 6 = lane bits 3, 4, 5)
__device__ __forceinline__ void rotate_column_block(float (&v)[16], int lane)
{
#pragma unroll
    for (int h = 1; h < 16; h <<= 1)
#pragma unroll
        for (int i0 = 0; i0 < 16; i0 += 2 * h)
#pragma unroll
            for (int i = i0; i < i0 + h; ++i) {
                const float a = v[i], b = v[i + h];
                v[i] = a + b;
                v[i + h] = a - b;
            }
    const uint32_t s8 = (uint32_t)(lane & 8) << 28;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = butterfly_xlane<8>(v[i], s8);
#pragma unroll
    for (int i = 0; i < 8; ++i) exchange_stage(v[i], v[i + 8], false);
#pragma unroll
    for (int i = 0; i < 8; ++i) exchange_stage(v[i], v[i + 8], true);
}

template <int WBITS, bool ROTATE, int HOLD>
__global__ __launch_bounds__(64 * kPcMostWaves) void prepare_columns_kernel(
    const float *__restrict__ W, int K, int N, const float *__restrict__ diag, const int32_t *__restrict__ perm,
    float norm, float qmax, void *__restrict__ codes, void *__restrict__ tiled, void *__restrict__ wide, float *__restrict__ scales,
    int32_t *__restrict__ colsum, float *__restrict__ colsumw, float *__restrict__ diag_copy)
{
    __shared__ float part[kPcMostWaves][kPcCols];
    __shared__ int sums[kPcMostWaves][kPcCols];
    __shared__ __align__(16) float2 recip[kPcMostWaves][kBlock];     // per wave: d and 1 / d of the block's rows
    const int nb = K / kBlock, nw = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 7, rg = lane >> 3;
    // four consecutive tiles of eight channels, the 128 bytes of a line of W, to the same die
    int tile = blockIdx.x;
    if (tile < ((int)gridDim.x & ~31)) {
        const int i = tile >> 3;
        tile = ((i >> 2) * 8 + (tile & 7)) * 4 + (i & 3);
    }
    const int n = tile * kPcCols + c;

    auto load = [&](int b, float (&v)[16]) {
        const int k0 = b * kBlock + 16 * rg;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            int row = k0 + i;
            if (ROTATE && perm) {
                row = perm[row];
                row = row < 0 ? 0 : (row >= K ? K - 1 : row);
            }
            v[i] = W[(size_t)row * N + n];
        }
    };
    auto rotate = [&](int b, float (&v)[16]) {
        if (!ROTATE) return;
        if (diag) {
            // v / d from r = 1 / d, which the wave forms once per row: q = v r, then q + (v - q d) r (Markstein's correction;
            // the division's ten instructions a value were two fifths of the kernel).  It rounds like the division while the
            // quotient and the remainder v - q d stay normal numbers: |d| between 2^-64 and 2^64, v zero or between 2^-60 and 2^60.
            // (An infinite quotient would become NaN, which the maximum below passes over.)  Other blocks are divided.
            const float d0 = diag[b * kBlock + lane], d1 = diag[b * kBlock + 64 + lane];
            auto plain = [](float d) { return fabsf(d) > 0x1p-64f && fabsf(d) < 0x1p64f; };
            float most = 0.0f;
            uint32_t least = ~0u;                        // twice the bits (no sign) less one: a zero counts as the largest
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                most = fmaxf(most, fabsf(v[i]));
                least = min(least, (__float_as_uint(v[i]) << 1) - 1);
            }
            if (__all(plain(d0) && plain(d1) && most < 0x1p60f && least >= (__float_as_uint(0x1p-60f) << 1) - 1)) {
                float2 *const dr = recip[wave];
                __builtin_amdgcn_wave_barrier();     // LDS serves a wave's requests in order
                dr[lane] = make_float2(d0, 1.0f / d0);
                dr[64 + lane] = make_float2(d1, 1.0f / d1);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float4 p = *reinterpret_cast<const float4 *>(dr + 16 * rg + i);
                    const float q0 = v[i] * p.y, q1 = v[i + 1] * p.w;
                    v[i] = __builtin_fmaf(__builtin_fmaf(-q0, p.x, v[i]), p.y, q0);
                    v[i + 1] = __builtin_fmaf(__builtin_fmaf(-q1, p.z, v[i + 1]), p.w, q1);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = v[i] / diag[b * kBlock + 16 * rg + i];
            }
        }
        rotate_column_block(v, lane);
    };
    auto lane_max = [&](const float (&v)[16], float m) {
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(v[i]));
        return m;
    };
    auto over_rows = [&](float m) {                      // maximum over the eight lanes of a channel
        m = fmaxf(m, row_xor<8>(m));
        m = fmaxf(m, __shfl_xor(m, 16));
        return fmaxf(m, __shfl_xor(m, 32));
    };
    auto sum_rows = [&](int t) {
        t += __shfl_xor(t, 8);
        t += __shfl_xor(t, 16);
        return t + __shfl_xor(t, 32);
    };
    if (diag_copy && blockIdx.x == 0)
        for (int k = threadIdx.x; k < K; k += blockDim.x) diag_copy[k] = diag[k];

    if constexpr (WBITS == 8) {
        auto store = [&](int b, const float (&v)[16], float inv) {
            uint32_t u[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) u[i] = quant_bits(v[i], inv);
            uint32_t w[4];
            int t = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = pack4_low_bytes(u[4 * j], u[4 * j + 1], u[4 * j + 2], u[4 * j + 3]);
                t = __builtin_amdgcn_sdot4((int)w[j], 0x01010101, t, false);
            }
            const uint4 piece = make_uint4(w[0], w[1], w[2], w[3]);
            const int k0 = b * kBlock + 16 * rg;
            *reinterpret_cast<uint4 *>(static_cast<int8_t *>(codes) + (size_t)n * K + k0) = piece;
            *reinterpret_cast<uint4 *>(static_cast<int8_t *>(tiled) + ((size_t)(n >> 4) * (K >> 6) + (k0 >> 6)) * 1024 +
                                       (rg & 3) * 256 + (n & 15) * 16) = piece;
            return t;
        };
        float v[HOLD][16];
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < HOLD; ++i)
            if (wave + nw * i < nb) load(wave + nw * i, v[i]);
#pragma unroll
        for (int i = 0; i < HOLD; ++i)
            if (wave + nw * i < nb) {
                rotate(wave + nw * i, v[i]);
                a = lane_max(v[i], a);
            }
        a = over_rows(a);
        if (rg == 0) part[wave][c] = a;
        __syncthreads();
        for (int w = 0; w < nw; ++w) a = fmaxf(a, part[w][c]);
        if (wave == 0 && rg == 0) scales[n] = a * (norm / qmax);
        const float inv = a > 0.0f ? qmax / a : 0.0f;
        int t = 0;
#pragma unroll
        for (int i = 0; i < HOLD; ++i)
            if (wave + nw * i < nb) t += store(wave + nw * i, v[i], inv);
        t = sum_rows(t);
        if (rg == 0) sums[wave][c] = t;
        __syncthreads();
        if (wave == 0 && rg == 0) {
            for (int w = 1; w < nw; ++w) t += sums[w][c];
            colsum[n] = t;
        }
    } else {
        // colsumw[n] = 16 * sum_g s_w[g][n] * (sum over the 128 codes of group g), added in the groups' order
        float total = 0.0f;
        float v[16], nxt[16];
        if (wave < nb) load(wave, nxt);
        for (int base = 0; base < nb; base += nw) {
            const int b = base + wave;
            if (b < nb) {
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = nxt[i];
                if (b + nw < nb) load(b + nw, nxt);
                rotate(b, v);
                const float a = over_rows(lane_max(v, 0.0f));
                const float scale = a * (norm / qmax);
                const float inv = a > 0.0f ? qmax / a : 0.0f;
                uint32_t u[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] = quant_bits(v[i], inv);
                int t = 0;
                // 8 consecutive k -> 4 bytes: byte j = code(k0+j) & 0xF | (code(k0+4+j) & 0xF) << 4
                uint32_t w[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t lo = pack4_low_bytes(u[8 * j], u[8 * j + 1], u[8 * j + 2], u[8 * j + 3]);
                    const uint32_t hi = pack4_low_bytes(u[8 * j + 4], u[8 * j + 5], u[8 * j + 6], u[8 * j + 7]);
                    w[j] = (lo & 0x0F0F0F0Fu) | ((hi << 4) & 0xF0F0F0F0u);
                    t = __builtin_amdgcn_sdot4((int)lo, 0x01010101, __builtin_amdgcn_sdot4((int)hi, 0x01010101, t, false), false);
                }
                t = sum_rows(t);
                if (rg == 0) {
                    scales[(size_t)b * N + n] = scale;
                    part[wave][c] = scale;
                    sums[wave][c] = t;
                }
                const int k0 = b * kBlock + 16 * rg;
                *reinterpret_cast<uint2 *>(static_cast<uint8_t *>(codes) + (size_t)n * (K / 2) + k0 / 2) = make_uint2(w[0], w[1]);
                // units of 16 input channels (8 bytes), see qgemm_tiled.hip
                *reinterpret_cast<uint2 *>(static_cast<uint8_t *>(tiled) + ((size_t)(n >> 4) * (K >> 6) + (k0 >> 6)) * 512 +
                                           (rg & 3) * 128 + (n & 15) * 8) = make_uint2(w[0], w[1]);
                // 16 * code, one byte each, in the blocks of the int8 form; a word's low nibbles are its first four codes
                if (wide)
                    *reinterpret_cast<uint4 *>(static_cast<int8_t *>(wide) + ((size_t)(n >> 4) * (K >> 6) + (k0 >> 6)) * 1024 +
                                               (rg & 3) * 256 + (n & 15) * 16) =
                        make_uint4((w[0] << 4) & 0xF0F0F0F0u, w[0] & 0xF0F0F0F0u, (w[1] << 4) & 0xF0F0F0F0u, w[1] & 0xF0F0F0F0u);
            }
            __syncthreads();
            if (wave == 0 && rg == 0)
                for (int w = 0; w < nw && base + w < nb; ++w) total += part[w][c] * (float)sums[w][c];
            __syncthreads();
        }
        if (wave == 0 && rg == 0) colsumw[n] = 16.0f * total;
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

hipError_t launch_prepare_rotate_dense(const float *W, int K, int N, const float *diag, const int32_t *perm,
                                       const float *R, float *Wrot, hipStream_t st)
{
    dim3 grid((N + kCols - 1) / kCols, K / kBlock);
    hipLaunchKernelGGL(prepare_rotate_dense_kernel, grid, dim3(kPrepThreads), 0, st, W, K, N, diag, perm, R, Wrot);
    return hipGetLastError();
}

// Where the pair is the faster form: rows so long that a wave of the one kernel would read and rotate its blocks twice or that
// come through a table, and int4 sets so large that its 32-byte pieces of W's lines bound it.  us of a set's replacement, pair / one
// kernel: 8 bits 6272 x 128 30 / 34, 9216 x 4608 134 / 143, 18432 x 128 39 / 84, but 6144 x 1152 44 / 35; int4 4608 x 16384 157 / 214,
// 9216 x 4608 102 / 116, 6272 x 4608 75 / 82, 2176 x 16384 77 / 79, but 4608 x 4608 64 / 63, 2048 x 16384 73 / 71; through a table, a set
// made anew, 4608 x 16 36 / 44, 4608 x 4608 417 / 451 (int4 664 / 691), but 1152 x 4608 100 / 97.
bool prepare_takes_pair(int K, int N, int wbits, bool gathered)
{
    const int nb = K / kBlock;
    if (gathered && nb > kPcMostWaves) return true;
    return wbits == 4 ? (int64_t)K * N > (int64_t)(K > 4096 ? 24 : 32) << 20 : nb > 3 * kPcMostWaves;
}

hipError_t launch_prepare_quant(const float *W, const float *diag, const int32_t *perm, bool rotate, float norm,
                                const Weights &w, float *amax, float *diag_copy, hipStream_t st)
{
    const int K = w.K, N = w.N, nb = K / kBlock;
    if (!diag) diag_copy = nullptr;
    const float qmax = w.wbits == 4 ? 7.0f : w.qbits == 6 ? 31.0f : 127.0f;
    if (prepare_takes_pair(K, N, w.wbits, perm != nullptr)) {
        const dim3 grid((N + kCols - 1) / kCols, nb), threads(kPrepThreads);
        if (w.wbits == 4) {
            hipLaunchKernelGGL((rotate ? prepare_quant_kernel<4, true> : prepare_quant_kernel<4, false>), grid, threads, 0, st, W, K, N, diag, perm,
                               nullptr, norm, qmax, w.codes, w.codes_tiled, w.codes_wide, w.scales, nullptr, diag_copy);
            if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
            hipLaunchKernelGGL(weight_colsumw4_kernel, dim3(N), dim3(64), 0, st, static_cast<const uint8_t *>(w.codes), w.scales, K, N,
                               w.colsumw);
            return hipGetLastError();
        }
        if (!amax || !rotate) return hipErrorInvalidValue;           // (dense blocks end at 36 of them)
        hipLaunchKernelGGL(prepare_absmax_kernel, grid, threads, 0, st, W, K, N, diag, perm, amax, w.colsum, diag_copy);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        hipLaunchKernelGGL((prepare_quant_kernel<8, true>), grid, threads, 0, st, W, K, N, diag, perm, amax, norm, qmax, w.codes,
                           w.codes_tiled, nullptr, w.scales, w.colsum, nullptr);
        return hipGetLastError();
    }
    const int rounds = (nb + kPcMostWaves - 1) / kPcMostWaves;      // blocks of the busiest wave
    auto go = [&](auto kern, int nw) {
        hipLaunchKernelGGL(kern, dim3(N / kPcCols), dim3(64 * nw), 0, st, W, K, N, diag, perm, norm, qmax, w.codes, w.codes_tiled, w.codes_wide,
                           w.scales, w.colsum, w.colsumw, diag_copy);
        return hipGetLastError();
    };
    if (w.wbits == 4) {
        const int nw = (nb + rounds - 1) / rounds;
        return rotate ? go(prepare_columns_kernel<4, true, 0>, nw) : go(prepare_columns_kernel<4, false, 0>, nw);
    }
    if (rounds == 1) return rotate ? go(prepare_columns_kernel<8, true, 1>, nb) : go(prepare_columns_kernel<8, false, 1>, nb);
    const int nw = (nb + 2) / 3;
    return rotate ? go(prepare_columns_kernel<8, true, 3>, nw) : go(prepare_columns_kernel<8, false, 3>, nw);
}

}  // namespace trdq
