// Integer product for launches that leave the chip idle: up to a few thousand tokens, any width, row-major codes.
//
// Operation: Y = dequant(Xq . Wq^T) of Eq. 10's quantised product (int8 weights), the arithmetic of the other kernels.
//
// With few output tiles the tiled and pipelined kernels are bound by the length of one chain: a workgroup walks all of
// K step by step, a barrier and an LDS round trip each (0.3 us per 64 input channels: 8 us at K = 1152 and 20-27 us at
// K = 4608 whatever the token count), while most compute units have no tile at all.  Here the tiles are small and the
// waves of a workgroup split K between them, in units of 128 input channels; their partial sums meet in LDS once, at the
// end.  Integer sums are exact, so the split changes nothing.  Back-to-back launches, before and after: 1152 -> 1152
// at 16 / 128 / 512 tokens 8.4 / 8.4 / 8.6 -> 2.8 / 3.3 / 5.7 us, 4608 -> 1152 at 16 / 512 tokens 24 / 22.6 -> 3.7 / 11.5 us.
// Rows and channels past the edges are clamped on load and not stored.
#include <type_traits>

#include "gemm_common.h"

namespace trdq {
namespace gemm {

namespace {

// Epilogue of one 16 x 16 tile: the lane holds channels n .. n + 3 of token m.  The operands are loaded by a call of
// their own, so that they can be requested ahead of the sums.
struct Finish8 {
    float4 s, bi;
    float sxm;
    int4 cs;
    int zc;
    __device__ __forceinline__ void load(const GemmArgs &g, int64_t m, int n)
    {
        if (m >= g.M) m = g.M - 1;
        if (n >= g.N) n = g.N - 4;
        s = *reinterpret_cast<const float4 *>(g.sw + n);
        bi = g.bias ? *reinterpret_cast<const float4 *>(g.bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
        sxm = g.sx[m];
        if (g.zc) {
            zc = g.zc[m];
            cs = *reinterpret_cast<const int4 *>(g.colsum + n);
        }
    }
    __device__ __forceinline__ void store(const GemmArgs &g, int64_t m, int n, v4i sum, bool debug) const
    {
        if (m >= g.M || n >= g.N) return;
        if (g.zc) sum += v4i{zc * cs.x, zc * cs.y, zc * cs.z, zc * cs.w};
        if (debug) *reinterpret_cast<int4 *>(g.acc_debug + m * g.N + n) = make_int4(sum[0], sum[1], sum[2], sum[3]);
        uint2 o;
        o.x = pack_bf16x2((float)sum[0] * sxm * s.x + bi.x, (float)sum[1] * sxm * s.y + bi.y);
        o.y = pack_bf16x2((float)sum[2] * sxm * s.z + bi.z, (float)sum[3] * sxm * s.w + bi.w);
        *reinterpret_cast<uint2 *>(g.Y + m * g.ldy + n) = o;
    }
};

// int8 weights.  Tile 16 TM tokens x 16 TN channels, K split over the waves by units of 128 input channels.
// Weights come from the block-tiled copy, where a fragment is 1 KB in lane order, straight into registers.  The
// same load from row-major rows would touch 16 rows per instruction and, four lanes of a quad in four rows, takes four
// times as long at the compute unit's address path; so the activations, which are row-major, go through LDS: a copy
// instruction moves 8 rows x 128 bytes, into an area of the wave's own (no barrier), XOR-swizzled for the fragment reads.
// ONE: every wave has a single unit (as many waves as units), so there is no next one to prefetch.
template <int TM, int TN, bool ONE>
__global__ __launch_bounds__(TM * TN >= 16 ? 512 : 768) void qgemm8_direct_kernel(GemmArgs g, int debug)
{
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int XB = TM * 2048;                    // a unit's activations
    constexpr int PER = 2 * TM + 2 * TN;             // requests of a unit
    v4i *const part = reinterpret_cast<v4i *>(smem); // [waves][TM * TN][64], once the activations are consumed
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = blockDim.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    int tm, tn;
    tile_map(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * (16 * TM);
    const int n0 = tn * (16 * TN);
    const int K = g.K, nu = K >> 7;

    int8_t *const mine = smem + wave * ((ONE ? 1 : 2) * XB);
    const uint32_t mine0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)mine;
    const int8_t *const xbase = g.Xq + m0 * K;
    uint32_t vx[2 * TM];                             // copy i: rows 8 i .. 8 i + 7 of the tile
#pragma unroll
    for (int i = 0; i < 2 * TM; ++i) {
        const int row = 8 * i + (lane >> 3), c = (lane & 7) ^ chunk_swizzle<128>(row);
        const int64_t left = g.M - 1 - m0;           // rows past the last token repeat it
        vx[i] = (uint32_t)((row < left ? row : (int)left) * K + c * 16);
    }
    const int8_t *wp[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) {
        int t = n0 / 16 + a;                         // N is a multiple of 16
        if (t * 16 >= g.N) t = g.N / 16 - 1;
        wp[a] = static_cast<const int8_t *>(g.Wc) + (int64_t)t * (K >> 6) * 1024 + lane * 16;
    }
    v4i w[ONE ? 1 : 2][TN][2];
    auto request = [&](int buf, int u) {
#pragma unroll
        for (int i = 0; i < 2 * TM; ++i) dma_1k(vx[i], xbase + u * 128, mine0 + buf * XB + i * 1024);
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                w[buf][a][h] = *reinterpret_cast<const v4i *>(wp[a] + (2 * u + h) * 1024);
    };
    v4i acc[TN][TM];
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    int fro[2];                                      // the lane's piece of a 16-row fragment, per half of the unit
#pragma unroll
    for (int h = 0; h < 2; ++h) fro[h] = r * 128 + ((4 * h + q) ^ chunk_swizzle<128>(r)) * 16;
    auto multiply = [&](int buf) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            v4i x[TM];
#pragma unroll
            for (int b = 0; b < TM; ++b) x[b] = *reinterpret_cast<const v4i *>(mine + buf * XB + b * 2048 + fro[h]);
#pragma unroll
            for (int a = 0; a < TN; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[buf][a][h], x[b], acc[a][b], 0, 0, 0);
        }
    };
    if constexpr (ONE) {
        request(0, wave);
        wait_vmcnt<0>();
        multiply(0);
    } else {
        // units wave, wave + nw, ...; past the last one it is requested again and not multiplied.  Before a unit's
        // fragments are read, everything but the next unit's requests has landed.
        int u = wave;
        request(0, u);
        while (true) {
            request(1, u + nw < nu ? u + nw : nu - 1);
            wait_vmcnt<PER>();
            multiply(0);
            u += nw;
            if (u >= nu) break;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // the fragments are out of the buffer that is refilled
            request(0, u + nw < nu ? u + nw : nu - 1);
            wait_vmcnt<PER>();
            multiply(1);
            u += nw;
            if (u >= nu) break;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        wait_vmcnt<0>();                             // the repeated request, before its area is used for the sums
    }
    // the sums meet in LDS; wave w finishes tiles w, w + waves, ..., whose first operands are requested here
    auto tile_m = [&](int t) { return m0 + (t % TM) * 16 + r; };
    auto tile_n = [&](int t) { return n0 + (t / TM) * 16 + q * 4; };
    Finish8 f[2];
    if (wave < TM * TN) f[0].load(g, tile_m(wave), tile_n(wave));
    if (wave + nw < TM * TN) f[1].load(g, tile_m(wave + nw), tile_n(wave + nw));
    __syncthreads();                                 // the activations' areas are free
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) part[((wave * TN + a) * TM + b) * 64 + lane] = acc[a][b];
    __syncthreads();
    auto sum_tile = [&](int t) {
        v4i sum = part[t * 64 + lane];
        for (int v = 1; v < nw; ++v) sum += part[(v * TM * TN + t) * 64 + lane];
        return sum;
    };
    if (wave < TM * TN) f[0].store(g, tile_m(wave), tile_n(wave), sum_tile(wave), debug);
    for (int t = wave + nw; t < TM * TN; t += nw) {
        if (t != wave + nw) f[1].load(g, tile_m(t), tile_n(t));
        f[1].store(g, tile_m(t), tile_n(t), sum_tile(t), debug);
    }
}

template <int TM, int TN>
hipError_t launch8(const GemmArgs &a, bool debug, hipStream_t st)
{
    GemmArgs g = a;
    g.tiles_m = (int)((g.M + 16 * TM - 1) / (16 * TM));
    g.tiles_n = (g.N + 16 * TN - 1) / (16 * TN);
    const int nu = g.K / 128;
    constexpr int most = TM * TN >= 16 ? 8 : 12;     // waves: registers, and the partial sums' LDS
    const int per = (nu + most - 1) / most, nw = (nu + per - 1) / per;
    const size_t area = (size_t)nw * (per == 1 ? 1 : 2) * TM * 2048, sums = (size_t)nw * TM * TN * 1024;
    const size_t smem = area > sums ? area : sums;
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n)), threads(64 * nw);
    auto kern = per == 1 ? qgemm8_direct_kernel<TM, TN, true> : qgemm8_direct_kernel<TM, TN, false>;
    if (smem > 64 * 1024)
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, threads, smem, st, g, (int)debug);
    return hipGetLastError();
}

// int4 weights: the same tiles, units (= scale groups) and copies.  A lane's weight fragment is the eight packed bytes of
// its unit in the block-tiled copy, widened in registers.  The float sums over the groups keep the order of the other int4
// kernels (one group after the other, so that the outputs are theirs bit for bit): the waves leave the int32 sums of
// their groups in LDS and the wave that finishes a tile folds them in turn.  Up to 12 groups that is one round of
// waves; with more the waves walk K together, a round of up to nine groups at a time, each round folded before the next one's
// sums are laid down (the requests of a unit go out a round ahead).
template <int TM, int TN, bool ONE>
__global__ __launch_bounds__(768) void qgemm4_direct_kernel(GemmArgs g, int debug)
{
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int XB = TM * 2048;                    // a unit's activations
    constexpr int PER = 2 * TM + 2 * TN;             // requests of a unit
    constexpr int MW = ONE ? 12 : 9;                 // most waves
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = blockDim.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    int tm, tn;
    tile_map(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * (16 * TM);
    const int n0 = tn * (16 * TN);
    const int K = g.K, nu = K >> 7;
    // [waves][TM * TN][64]: with one round in the place of the activations, once these are consumed
    v4i *const part = reinterpret_cast<v4i *>(smem + (ONE ? 0 : nw * 2 * XB));

    int8_t *const mine = smem + wave * ((ONE ? 1 : 2) * XB);
    const uint32_t mine0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)mine;
    const int8_t *const xbase = g.Xq + m0 * K;
    uint32_t vx[2 * TM];                             // copy i: rows 8 i .. 8 i + 7 of the tile
#pragma unroll
    for (int i = 0; i < 2 * TM; ++i) {
        const int row = 8 * i + (lane >> 3), c = (lane & 7) ^ chunk_swizzle<128>(row);
        const int64_t left = g.M - 1 - m0;           // rows past the last token repeat it
        vx[i] = (uint32_t)((row < left ? row : (int)left) * K + c * 16);
    }
    const uint8_t *wp[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) {
        int t = n0 / 16 + a;                         // N is a multiple of 16
        if (t * 16 >= g.N) t = g.N / 16 - 1;
        wp[a] = static_cast<const uint8_t *>(g.Wc) + (int64_t)t * (K >> 6) * 512 + lane * 8;
    }
    uint2 w[ONE ? 1 : 2][TN][2];
    auto request = [&](auto buf_tag, int u) {
        constexpr int buf = decltype(buf_tag)::value;
#pragma unroll
        for (int i = 0; i < 2 * TM; ++i) dma_1k(vx[i], xbase + u * 128, mine0 + buf * XB + i * 1024);
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                w[buf][a][h] = *reinterpret_cast<const uint2 *>(wp[a] + (2 * u + h) * 512);
    };
    int fro[2];                                      // the lane's piece of a 16-row fragment, per half of the unit
#pragma unroll
    for (int h = 0; h < 2; ++h) fro[h] = r * 128 + ((4 * h + q) ^ chunk_swizzle<128>(r)) * 16;

    // the tiles this wave finishes are wave, wave + waves, ...; with several rounds there are at most two
    auto tile_m = [&](int t) { return m0 + (t % TM) * 16 + r; };
    auto tile_n = [&](int t) {
        const int n = n0 + (t / TM) * 16 + q * 4;
        return n < g.N ? n : g.N - 4;                // loads only: such a tile is not stored
    };
    auto load_scales = [&](int t, int u0, float4 (&sc)[MW]) {
        const float *const p = g.sw + tile_n(t);
#pragma unroll
        for (int v = 0; v < MW; ++v) sc[v] = *reinterpret_cast<const float4 *>(p + (int64_t)(u0 + v < nu ? u0 + v : nu - 1) * g.N);
    };
    auto fold = [&](int t, int u0, const float4 (&sc)[MW], v4f &f) {
#pragma unroll
        for (int v = 0; v < MW; ++v) {
            if (v < nw && u0 + v < nu) {
                const v4i p = part[(v * TM * TN + t) * 64 + lane];
                if (debug && tile_m(t) < g.M && n0 + (t / TM) * 16 + q * 4 < g.N)
                    *reinterpret_cast<int4 *>(g.acc_debug + ((int64_t)(u0 + v) * g.M + tile_m(t)) * g.N + tile_n(t)) =
                        make_int4(p[0] >> 4, p[1] >> 4, p[2] >> 4, p[3] >> 4);
                f[0] += sc[v].x * (float)p[0];
                f[1] += sc[v].y * (float)p[1];
                f[2] += sc[v].z * (float)p[2];
                f[3] += sc[v].w * (float)p[3];
            }
        }
    };
    auto finish = [&](int t, v4f f) {                // y = (s_x / 16) * f + bias, the codes having been 16 * code
        const int64_t m = tile_m(t);
        const int n = n0 + (t / TM) * 16 + q * 4;
        if (m >= g.M || n >= g.N) return;
        if (g.zc) {
            const float zc = (float)g.zc[m];
            const float4 cw = *reinterpret_cast<const float4 *>(g.colsumw + n);
            f += v4f{zc * cw.x, zc * cw.y, zc * cw.z, zc * cw.w};
        }
        const float sxm = g.sx[m] * 0.0625f;
        const float4 bi = g.bias ? *reinterpret_cast<const float4 *>(g.bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
        uint2 o;
        o.x = pack_bf16x2(sxm * f[0] + bi.x, sxm * f[1] + bi.y);
        o.y = pack_bf16x2(sxm * f[2] + bi.z, sxm * f[3] + bi.w);
        *reinterpret_cast<uint2 *>(g.Y + m * g.ldy + n) = o;
    };
    v4f f[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
    // one round: this wave's unit u0 + wave (past the last one the last is requested again and its sums are not used)
    auto round = [&](auto buf_tag, int u0) {
        constexpr int buf = decltype(buf_tag)::value;
        if constexpr (ONE) {
            wait_vmcnt<0>();
        } else {
            const int nxt = u0 + nw + wave;
            request(std::integral_constant<int, 1 - buf>{}, nxt < nu ? nxt : nu - 1);
            wait_vmcnt<PER>();                       // everything but the requests just made
        }
        v4i acc[TN][TM];
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            v4i x[TM];
#pragma unroll
            for (int b = 0; b < TM; ++b) x[b] = *reinterpret_cast<const v4i *>(mine + buf * XB + b * 2048 + fro[h]);
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                const uint2 p = w[buf][a][h];
                const v4i wa = v4i{(int)((p.x << 4) & 0xF0F0F0F0u), (int)(p.x & 0xF0F0F0F0u),
                                   (int)((p.y << 4) & 0xF0F0F0F0u), (int)(p.y & 0xF0F0F0F0u)};
#pragma unroll
                for (int b = 0; b < TM; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa, x[b], acc[a][b], 0, 0, 0);
            }
        }
        float4 sc[MW];
        if (wave < TM * TN) load_scales(wave, u0, sc);
        __syncthreads();                             // ONE: the activations' areas are free; else the last round is folded
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) part[((wave * TN + a) * TM + b) * 64 + lane] = acc[a][b];
        __syncthreads();
        if constexpr (ONE) {
            for (int t = wave; t < TM * TN; t += nw) {
                if (t != wave) load_scales(t, u0, sc);
                f[0] = v4f{0.f, 0.f, 0.f, 0.f};
                fold(t, u0, sc, f[0]);
                finish(t, f[0]);
            }
        } else {
            if (wave < TM * TN) fold(wave, u0, sc, f[0]);
            if (wave + nw < TM * TN) {
                load_scales(wave + nw, u0, sc);
                fold(wave + nw, u0, sc, f[1]);
            }
        }
    };
    request(std::integral_constant<int, 0>{}, wave < nu ? wave : nu - 1);
    if constexpr (ONE) {
        round(std::integral_constant<int, 0>{}, 0);
    } else {
        for (int u0 = 0;; u0 += 2 * nw) {
            round(std::integral_constant<int, 0>{}, u0);
            if (u0 + nw >= nu) break;
            round(std::integral_constant<int, 1>{}, u0 + nw);
            if (u0 + 2 * nw >= nu) break;
        }
        wait_vmcnt<0>();                             // the repeated request
        if (wave < TM * TN) finish(wave, f[0]);
        if (wave + nw < TM * TN) finish(wave + nw, f[1]);
    }
}

template <int TM, int TN>
hipError_t launch4(const GemmArgs &a, bool debug, hipStream_t st)
{
    GemmArgs g = a;
    g.tiles_m = (int)((g.M + 16 * TM - 1) / (16 * TM));
    g.tiles_n = (g.N + 16 * TN - 1) / (16 * TN);
    const int nu = g.K / 128;
    const bool one = nu <= 12;
    const int per = one ? 1 : (nu + 8) / 9, nw = (nu + per - 1) / per;
    if (!one && TM * TN > 2 * nw) return hipErrorInvalidValue;    // two tiles to finish per wave
    const size_t area = (size_t)nw * (one ? 1 : 2) * TM * 2048, sums = (size_t)nw * TM * TN * 1024;
    const size_t smem = one ? (area > sums ? area : sums) : area + sums;
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n)), threads(64 * nw);
    auto kern = one ? qgemm4_direct_kernel<TM, TN, true> : qgemm4_direct_kernel<TM, TN, false>;
    if (smem > 64 * 1024)
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, threads, smem, st, g, (int)debug);
    return hipGetLastError();
}

}  // namespace

// Tiles in the order they are tried: {16-token tiles, 16-channel tiles}.
constexpr int kDirectTiles[5][2] = {{1, 1}, {1, 2}, {2, 2}, {2, 4}, {4, 4}};

// The smallest tile whose grid is about one round of workgroups: 256 of nine waves, more of fewer.  Measured at
// 1152 -> 1152, us: 64 tokens 2.9 (288 workgroups of 16 x 16, 144 of 16 x 32), 128 tokens 3.3 (32 x 32; 16 x 16 4.4),
// 256 tokens 4.0 (32 x 64), 768 tokens 5.8 (432 of 32 x 64; 64 x 64 7.3); at 4608 -> 1152: 64 tokens 6.4 (16 x 32),
// 256 tokens 9.0 (32 x 64), 768 tokens 13.4 (64 x 64; 32 x 64 15.8).  One unit per wave leaves registers for two rounds
// of 32 x 64 tiles, and 64 x 64 never pays there.
// Two (2.5) workgroups per compute unit is the most that pays for few units too, however many would fit: the kernels with
// tiles in LDS have little K to walk there (640 -> 512 at 4096 7.2 / 6.1, at 2048 in 512 workgroups 5.6 both ways, 768 -> 2304
// at 700 8.3 / 6.3).  One or two units are workgroups of one or two waves, which finish their tiles one after the other:
// small tiles in many workgroups.  us, with a wave of 32 x 64 / now / tiles in LDS: 128 -> 512 at 2048 tokens (16 x 16, 16 per
// compute unit) 6.0 / 3.8 / 4.0, 128 -> 2304 at 256 5.9 / 3.3 / 3.8, 128 -> 512 at 4096 (32 per) 5.1 against 4.4; 256 -> 512 at
// 2048 (16 x 32, 8 per) 5.1 / 4.1 / 4.5, 256 -> 768 at 2048 (12 per) 4.9 against 4.7; widths that no other kernel takes in
// whole tiles a quarter more (256 -> 1168 at 1024 4.2, 6.6).
// Beyond that the kernels with tiles in LDS are ahead: 1152 -> 1152 at 1024 tokens 8.0 both ways, at 1536 11.2 against
// 8.7 us; 4608 -> 1152 at 1024 tokens 20.7 against 17.6 us.  Of shapes that those kernels take only in part (ragged token
// counts, odd widths) 64 x 64 tiles take more: 4608 -> 1168 at 1000 tokens 21.6 against 22.3 us, 3072 -> 1168 at 1024 16.1 / 19.8.
// Widths of whole 128-channel tiles they take as they are, until K is long: 1664 -> 1536 at 1024 tokens (384 workgroups) 13.4
// against 9.3 us, 3072 -> 768 at 1536 15.7 / 13.7, 3584 -> 768 at 2048 17.8 / 16.3 but -> 1024 at 1536 17.2 / 20.0, 4096 -> 768 at
// 2048 18.5 / 20.1.  With ragged tokens (2304 -> 3072 at 400 17.7 / 11.9, 2688 -> 3072 at 400 19.6 / 14.8, 3072 -> 1536 at 1000
// 15.8 / 17.8) and with zero points (3072 -> 1536 at 1024 15.7 / 18.4) the other kernels are slower ones, and the line lies lower.
int qgemm8_direct_tile(int64_t M, int K, int N, bool asym)
{
    const int nu = K / 128;
    if (M <= 0 || nu <= 0 || (int64_t)M > (1 << 20)) return -1;
    auto grid = [&](int i) {
        const int tm = 16 * kDirectTiles[i][0], tn = 16 * kDirectTiles[i][1];
        return ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
    };
    const int64_t cus = num_cus();
    if (nu <= 2) {
        const int64_t most = (nu == 1 ? 16 : 8) * cus * (N % 128 != 0 && N % 144 != 0 ? 5 : 4) / 4;
        if (nu == 2 && grid(0) <= 2 * cus) return 0;
        return grid(nu - 1) <= most ? nu - 1 : -1;
    }
    const int per = (nu + 11) / 12, nw = (nu + per - 1) / per;
    const bool whole = M % 128 == 0 && N % 144 == 0;
    const bool whole128 = N % 128 == 0 && K < (asym || M % 128 != 0 ? 2816 : (M % 1024 != 0 ? 3200 : 4096));
    const int64_t most_wide = whole ? 2 * cus : 5 * cus / 2;
    int64_t round = cus * 9 / (per == 1 ? nw : 9);
    if (round > 2 * cus) round = 2 * cus;
    for (int i = 0; i < 5; ++i) {
        int64_t most = round;
        if (i == 3 && per == 1) {
            most = whole ? 2 * round : 5 * round / 2;
            if (most > most_wide) most = most_wide;
        }
        if (i == 4) most = per == 1 ? 0 : (whole || whole128 ? round : 7 * round / 4);
        if (grid(i) <= most) return i;
    }
    return -1;
}

hipError_t launch_qgemm8_direct(const GemmArgs &a, bool debug, int tile, hipStream_t st)
{
    switch (tile) {
        case 0: return launch8<1, 1>(a, debug, st);
        case 1: return launch8<1, 2>(a, debug, st);
        case 2: return launch8<2, 2>(a, debug, st);
        case 3: return launch8<2, 4>(a, debug, st);
        case 4: return launch8<4, 4>(a, debug, st);
    }
    return hipErrorInvalidValue;
}

// int4 tiles, in the order they are tried: 16 x 32, 32 x 32, 32 x 64.  One workgroup per compute unit, with one
// round of groups two of 32 x 32 (us: 1152 -> 1152 at 64 / 250 / 384 tokens 10.9 / 11.3 / 10.6 -> 5.2 / 5.9 / 6.1, in 576
// workgroups at 500 tokens 8.2 against 7.9 of the 64-token tiles in LDS; 4608 -> 1152 at 64 / 192 / 250 tokens
// 30.3 / 30.6 / 31.1 -> 7.5 / 9.4 / 14.0, those take 22.8).  One or two groups, which those do not take: two, four (256 -> 512
// at 1000 tokens 6.1 -> 4.2, at 2048 5.8 -> 5.5, in 1504 workgroups at 3000 7.0 against 6.2); one, whose workgroup is one wave: six,
// of the smallest tile only (128 -> 512 at 1024 tokens 5.0 -> 4.3, -> 768 at 1024 5.0 -> 4.8, -> 512 at 2048 in eight 5.3 against
// 5.1; 32 x 32 there 5.8).
int qgemm4_direct_tile(int64_t M, int K, int N)
{
    const int nu = K / 128;
    if (M <= 0 || nu <= 0 || nu > 72 || M > (1 << 20)) return -1;
    const int64_t cus = num_cus();
    const int64_t most[3] = {nu == 1 ? 6 * cus : (nu == 2 ? 4 * cus : cus), nu == 1 ? 0 : (nu == 2 ? 4 * cus : (nu <= 12 ? 2 * cus : cus)),
                             nu == 1 ? 0 : cus};
    constexpr int tiles[3][2] = {{1, 2}, {2, 2}, {2, 4}};
    for (int i = 0; i < 3; ++i) {
        const int tm = 16 * tiles[i][0], tn = 16 * tiles[i][1];
        if (((M + tm - 1) / tm) * ((N + tn - 1) / tn) <= most[i]) return i;
    }
    return -1;
}

hipError_t launch_qgemm4_direct(const GemmArgs &a, bool debug, int tile, hipStream_t st)
{
    switch (tile) {
        case 0: return launch4<1, 2>(a, debug, st);
        case 1: return launch4<2, 2>(a, debug, st);
        case 2: return launch4<2, 4>(a, debug, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace gemm
}  // namespace trdq
