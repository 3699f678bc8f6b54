// linear_fused: rotate -> per-token quantise -> int8 product -> dequantising epilogue in one
// kernel (Eq. 10 end to end); the int8 activations never leave the chip.
//
// A workgroup owns a panel of BM tokens for the WHOLE input width K: the prologue rotates and
// quantises the panel straight into LDS (int8, BM x K), then the workgroup sweeps its share
// of the output channels with the same matrix-core loop as qgemm, streaming weight tiles
// through a double-buffered LDS stage.  The 160 KB of LDS per compute unit bound BM * K; the
// panel height shrinks as K grows (64 tokens up to K = 1536, 32 up to 3072, 16 up to 6144).
#include <type_traits>

#include "rotate_core.h"

namespace trdq {

namespace {

constexpr int kThreads = 256;
constexpr int kPad = 16;
constexpr int kBN = 128;   // output channels per weight tile
constexpr int kBK = 128;   // input channels per weight tile = one rotation block / scale group

struct FusedArgs {
    const uint16_t *X;     // bf16 [M, ldx]
    const float *diag;     // [K] or null
    const void *Wc;
    const float *sw;
    const float *bias;
    const int32_t *colsum; // ASYM kernels: sum over k of the weight codes of every output channel [N]
    uint16_t *Y;
    int64_t M, ldx, ldy;
    int K, N;
    int tiles_n;           // ceil(N / kBN)
    int nsplit;            // workgroups sharing one token panel
};

// BM tokens per panel, S lane-rows per token in the prologue, T blocks per lane-row.
// ASYM: the panel is quantised with the asymmetric form of Eq. 1-3 (per-token zero point z, codes
// stored as q - 128); the epilogue adds (128 - z_m) * colsum[n] to the integer sums, which makes
// them the exact sums of (q - z) * w.  Int8 weights only.
template <int BM, int T, int S, bool W4, bool ASYM = false>
__global__ __launch_bounds__(kThreads) void linear_fused_kernel(FusedArgs g)
{
    static_assert(!(W4 && ASYM), "zero points are carried for int8 weights only");
    constexpr int WM = BM >= 64 ? 32 : BM;           // wave tile (tokens)
    constexpr int WGM = BM / WM, WGN = 4 / WGM;
    constexpr int WN = kBN / WGN;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int LDW = kBK + kPad;
    constexpr int CW = W4 ? kBN * (kBK / 32) / kThreads : kBN * (kBK / 16) / kThreads;

    extern __shared__ __align__(16) int8_t smem[];
    const int K = g.K;
    const int nb = K / kBlock;
    const int LDX = K + kPad;
    int8_t *const Xp = smem;                              // [BM][K + 16]   int8 panel
    int8_t *const Ws = smem + BM * LDX;                   // [2][kBN][LDW]  weight stages
    float *const sxs = reinterpret_cast<float *>(Ws + 2 * kBN * LDW);   // [BM]
    int *const zcs = reinterpret_cast<int *>(sxs + BM);                 // [BM] 128 - z (ASYM)

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lg = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.x * BM;

    // ---- prologue: rotate + quantise the panel into LDS -----------------------------------
    {
        const LaneSigns sg(l16);
        const int s = lg % S;
        constexpr int kTokPerPass = (kThreads / 64) * (4 / S);
        for (int r0 = 0; r0 < BM; r0 += kTokPerPass) {
            const int r = r0 + wave * (4 / S) + lg / S;
            const int64_t token = m0 + r;
            const bool ok = r < BM && token < g.M;
            float v[T][8];
            float amax, amin;
            rotate_token<T, S, ASYM>(g.X + token * g.ldx, ok, nb, s, l16, g.diag, sg, v, amax, amin);
            if constexpr (ASYM) {
                const TokenRangeQuant q(amin, amax);
                if (r < BM) {
                    if (s == 0 && l16 == 0) {
                        sxs[r] = ok ? q.scale : 0.0f;
                        zcs[r] = ok ? q.zc : 0;
                    }
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const int b = t * S + s;
                        if (b < nb)
                            *reinterpret_cast<uint2 *>(Xp + r * LDX + b * kBlock + l16 * 8) = q.pack8(v[t]);
                    }
                }
            } else {
                const float inv = token_inv_scale(amax);
                if (r < BM) {
                    if (s == 0 && l16 == 0) sxs[r] = ok ? token_scale(amax) : 0.0f;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const int b = t * S + s;
                        if (b < nb)
                            *reinterpret_cast<uint2 *>(Xp + r * LDX + b * kBlock + l16 * 8) = quant_pack8(v[t], inv);
                    }
                }
            }
        }
    }

    // ---- weight staging -----------------------------------------------------------------------
    const int wm = wave % WGM, wn = wave / WGM;
    const int tiles_per = (g.tiles_n + g.nsplit - 1) / g.nsplit;
    const int tn_begin = blockIdx.y * tiles_per;
    const int tn_end = min(tn_begin + tiles_per, g.tiles_n);
    const int KT = K / kBK;
    const int iters = (tn_end - tn_begin) * KT;

    uint4 wr[CW];
    int wrow[CW], wcol[CW], wdst[CW];
#pragma unroll
    for (int i = 0; i < CW; ++i) {
        const int ch = tid + i * kThreads;
        if constexpr (W4) {
            wrow[i] = ch / (kBK / 32); wcol[i] = (ch % (kBK / 32)) * 16;
            wdst[i] = wrow[i] * LDW + (ch % (kBK / 32)) * 32;
        } else {
            wrow[i] = ch / (kBK / 16); wcol[i] = (ch % (kBK / 16)) * 16;
            wdst[i] = wrow[i] * LDW + wcol[i];
        }
    }
    auto load_tile = [&](int it) {
        const int tn = tn_begin + it / KT, kt = it % KT;
#pragma unroll
        for (int i = 0; i < CW; ++i) {
            int n = tn * kBN + wrow[i];
            if (n >= g.N) n = g.N - 1;
            const uint8_t *src = static_cast<const uint8_t *>(g.Wc) +
                                 (W4 ? (size_t)n * (K / 2) + kt * (kBK / 2) : (size_t)n * K + kt * kBK) + wcol[i];
            wr[i] = *reinterpret_cast<const uint4 *>(src);
        }
    };
    auto store_tile = [&](int buf) {
        int8_t *ws = Ws + buf * kBN * LDW;
#pragma unroll
        for (int i = 0; i < CW; ++i) {
            if constexpr (W4) {
                const uint4 p = wr[i];
                uint4 a, b;
                a.x = (p.x << 4) & 0xF0F0F0F0u; a.y = p.x & 0xF0F0F0F0u;
                a.z = (p.y << 4) & 0xF0F0F0F0u; a.w = p.y & 0xF0F0F0F0u;
                b.x = (p.z << 4) & 0xF0F0F0F0u; b.y = p.z & 0xF0F0F0F0u;
                b.z = (p.w << 4) & 0xF0F0F0F0u; b.w = p.w & 0xF0F0F0F0u;
                *reinterpret_cast<uint4 *>(ws + wdst[i]) = a;
                *reinterpret_cast<uint4 *>(ws + wdst[i] + 16) = b;
            } else {
                *reinterpret_cast<uint4 *>(ws + wdst[i]) = wr[i];
            }
        }
    };

    v4i acc[TN][TM];
    v4f facc[W4 ? TN : 1][W4 ? TM : 1];
    auto reset = [&]() {
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                acc[a][b] = v4i{0, 0, 0, 0};
                if constexpr (W4) facc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
            }
    };
    reset();

    if (iters > 0) { load_tile(0); store_tile(0); }
    __syncthreads();     // also publishes the panel and the token scales

    const int8_t *xrow = Xp + (wm * WM + l16) * LDX + lg * 16;
    for (int it = 0; it < iters; ++it) {
        const int buf = it & 1;
        const int tn = tn_begin + it / KT, kt = it % KT;
        if (it + 1 < iters) load_tile(it + 1);

        const int8_t *ws = Ws + buf * kBN * LDW + (wn * WN + l16) * LDW + lg * 16;
#pragma unroll
        for (int kk = 0; kk < kBK; kk += 64) {
            v4i af[TN], bf[TM];
#pragma unroll
            for (int a = 0; a < TN; ++a) af[a] = *reinterpret_cast<const v4i *>(ws + a * 16 * LDW + kk);
#pragma unroll
            for (int b = 0; b < TM; ++b)
                bf[b] = *reinterpret_cast<const v4i *>(xrow + b * 16 * LDX + kt * kBK + kk);
#pragma unroll
            for (int a = 0; a < TN; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[b], acc[a][b], 0, 0, 0);
        }

        const int n_base = tn * kBN + wn * WN + lg * 4;
        if constexpr (W4) {
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                const int n = n_base + a * 16;
                float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
                if (n < g.N) s = *reinterpret_cast<const float4 *>(g.sw + (size_t)kt * g.N + n);
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    facc[a][b][0] += s.x * (float)acc[a][b][0];
                    facc[a][b][1] += s.y * (float)acc[a][b][1];
                    facc[a][b][2] += s.z * (float)acc[a][b][2];
                    facc[a][b][3] += s.w * (float)acc[a][b][3];
                    acc[a][b] = v4i{0, 0, 0, 0};
                }
            }
        }

        if (kt == KT - 1) {
            // epilogue of channel tile tn
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                const int n = n_base + a * 16;
                if (n >= g.N) continue;
                float4 s = make_float4(1.f, 1.f, 1.f, 1.f), bi = make_float4(0.f, 0.f, 0.f, 0.f);
                if constexpr (!W4) s = *reinterpret_cast<const float4 *>(g.sw + n);
                if (g.bias) bi = *reinterpret_cast<const float4 *>(g.bias + n);
                int4 cs = make_int4(0, 0, 0, 0);
                if constexpr (ASYM) cs = *reinterpret_cast<const int4 *>(g.colsum + n);
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    const int r = wm * WM + b * 16 + l16;
                    const int64_t m = m0 + r;
                    if (m >= g.M) continue;
                    const float sxm = W4 ? sxs[r] * 0.0625f : sxs[r];
                    if constexpr (ASYM) {
                        const int zc = zcs[r];
                        acc[a][b] += v4i{zc * cs.x, zc * cs.y, zc * cs.z, zc * cs.w};
                    }
                    float y0, y1, y2, y3;
                    if constexpr (W4) {
                        y0 = sxm * facc[a][b][0] + bi.x;
                        y1 = sxm * facc[a][b][1] + bi.y;
                        y2 = sxm * facc[a][b][2] + bi.z;
                        y3 = sxm * facc[a][b][3] + bi.w;
                    } else {
                        y0 = (float)acc[a][b][0] * sxm * s.x + bi.x;
                        y1 = (float)acc[a][b][1] * sxm * s.y + bi.y;
                        y2 = (float)acc[a][b][2] * sxm * s.z + bi.z;
                        y3 = (float)acc[a][b][3] * sxm * s.w + bi.w;
                    }
                    uint2 o;
                    o.x = pack_bf16x2(y0, y1);
                    o.y = pack_bf16x2(y2, y3);
                    *reinterpret_cast<uint2 *>(g.Y + m * g.ldy + n) = o;
                }
            }
            reset();
        }

        if (it + 1 < iters) store_tile(buf ^ 1);
        __syncthreads();
    }
}

// ---- few tokens: one 16-token panel per workgroup, a wave per rotation block -----------------------
// With up to a few hundred tokens the unfused pair is bound by two launches and two chains of memory
// latency, not by arithmetic, and so is this kernel: what counts is the length of the one chain that is
// left.  A workgroup owns 16 tokens and 16 * TN output channels for the whole K; a wave owns BPW rotation
// blocks (128 input channels each; one up to K = 1536, three at K = 4608), and does everything for them:
//
//   loads       X, the diagonal, and the weight fragments straight into registers (every weight byte meets
//               exactly one matrix instruction: LDS would buy nothing), all requested up front;
//   rotation    lane (token r, q) starts with the 8-channel chunks 32 c + 8 q, c = 0..3: index bits 6, 5
//               and 2..0 are butterflies inside the lane, bits 4 and 3 sit in the lane number; a swap of two
//               registers between lane halves (rows) turns such a bit into a register bit and a register bit
//               into the lane bit, so that afterwards the lane holds the 32 consecutive channels 32 q ..;
//   codes       after the token maxima have met in LDS, the lane's 32 codes are its operands of the two
//               matrix instructions of the block as they are: the instruction does not care which input
//               channels a lane supplies as long as both operands agree, so the weights are loaded for the
//               same 32 channels and no code crosses a lane;
//   product     2 TN matrix instructions per block; the waves' partial sums (int8 weights: one per wave, int4:
//               one per block, i.e. per scale group) meet in LDS, wave w finishes channel tiles w, w + waves, ...
//
// The launcher takes the narrowest tile whose grid is one round of workgroups (see small_tiles): repeating the rotation
// on idle compute units is free, and fewer weight bytes per compute unit arrive sooner.  The arguments that the
// first loads need are the ones delivered in registers at wave launch.
//
// Measured, launches replayed back to back (an empty kernel: 2.2 us): 1152 -> 1152 int8 at 16 / 128 / 256 / 512 tokens
// 5.0 / 5.6 / 6.0 / 6.9 us, against 10.0 / 10.1 / 10.2 / 10.5 for a form that split K over eight waves, rotated
// with lane exchanges (630 vector instructions per wave instead of 290), read row-major weights and passed the codes
// through LDS; int4 5.4 / 6.1 / 6.6 / 7.6; 4608 -> 1152 at 16 tokens 12.2 (int8), 12.9 (int4).
constexpr int64_t kSmallMaxWorkgroups = 512;    // of the widest tile: at most two rounds
constexpr int kSmallMaxBlocks = 36;

// butterfly over an index bit that sits in lane bit 5 (HALF = 32) or 4 (16) of registers x (register bit 0)
// and y (register bit 1): the two bits trade places, x becomes the sum and y the difference
template <int HALF>
__device__ __forceinline__ void butterfly_swap(float &x, float &y)
{
    uint32_t a = __float_as_uint(x), b = __float_as_uint(y);
    if constexpr (HALF == 32) {
        const auto t = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = t[0]; b = t[1];
    } else {
        const auto t = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = t[0]; b = t[1];
    }
    x = __uint_as_float(a) + __uint_as_float(b);
    y = __uint_as_float(a) - __uint_as_float(b);
}

// v[8 c + j] = element 32 c + 8 q + j of the block in lane q (= lane / 16) -> the unnormalised H_128 of the
// block, element 32 q + 8 c + j in v[8 c + j]
__device__ __forceinline__ void fwht128_quarters(float (&v)[32])
{
    auto bf = [](float &a, float &b) { const float s = a + b; b = a - b; a = s; };
#pragma unroll
    for (int h = 1; h < 8; h <<= 1)
#pragma unroll
        for (int i = 0; i < 32; ++i)
            if (!(i & h)) bf(v[i], v[i + h]);
#pragma unroll
    for (int h = 8; h < 32; h <<= 1)
#pragma unroll
        for (int i = 0; i < 32; ++i)
            if (!(i & h)) bf(v[i], v[i + h]);
#pragma unroll
    for (int i = 0; i < 16; ++i) butterfly_swap<32>(v[i], v[i + 16]);
#pragma unroll
    for (int i = 0; i < 32; ++i)
        if (!(i & 8)) butterfly_swap<16>(v[i], v[i + 8]);
}

template <int TN, int BPW, bool W4, bool ASYM>
__global__ __launch_bounds__(768) void linear_fused_small_kernel(
    const uint16_t *__restrict__ X, const float *__restrict__ diag, const uint8_t *__restrict__ Wc, int64_t ldx, int M,
    int K, int N, const float *__restrict__ sw, const float *__restrict__ bias, const int32_t *__restrict__ colsum,
    uint16_t *__restrict__ Y, int64_t ldy)
{
    static_assert(!(W4 && ASYM), "zero points are carried for int8 weights only");
    extern __shared__ __align__(16) int8_t smem[];
    float *const ext_s = reinterpret_cast<float *>(smem);                 // [waves][32]: token maxima (and minima)
    v4i *const part = reinterpret_cast<v4i *>(smem + 12 * 32 * 4);        // [waves or blocks][TN][64] partial sums

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = blockDim.x >> 6;
    const int nb = K / kBlock;
    const int r = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.x * (TN * 16);
    const int m = blockIdx.y * 16 + r;
    const bool tok_ok = m < M;
    const int b0 = wave * BPW;                                           // the wave's first block

    // Loads return in order, so the order of issue is the order of need.  Tokens past the end and a last
    // wave's blocks past the row are clamped: loaded and rotated like the others, their sums are not used.
    uint4 raw[BPW][4];
    float4 dv[8];
    auto load_d = [&](int i) {
        const int b = b0 + i < nb ? b0 + i : nb - 1;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                dv[2 * c + h] = diag ? *reinterpret_cast<const float4 *>(diag + b * kBlock + c * 32 + q * 8 + h * 4)
                                     : make_float4(1.f, 1.f, 1.f, 1.f);
    };
    {
        const uint16_t *const xt = X + (int64_t)(tok_ok ? m : M - 1) * ldx + q * 8;
#pragma unroll
        for (int i = 0; i < BPW; ++i) {
            const int b = b0 + i < nb ? b0 + i : nb - 1;
#pragma unroll
            for (int c = 0; c < 4; ++c) raw[i][c] = *reinterpret_cast<const uint4 *>(xt + b * kBlock + c * 32);
            if (i == 0) load_d(0);
        }
    }
    // weights of channel n0 + 16 a + r, the lane's 32 input channels of each of the wave's blocks, from the
    // block-tiled copy: a load's lanes cover runs of 256 (128) bytes.  (Row-major rows would put the four lanes of
    // a quad in four rows, which the compute unit's address path takes four times as long for.)
    constexpr int WR = W4 ? 1 : 2;                   // 16-byte pieces of them
    // (six blocks' worth of int8 fragments do not fit beside the activations: they follow the rotation)
    constexpr bool kLateW = !W4 && BPW == 3 && TN > 1;
    uint4 wf[BPW][TN][WR];
    const uint32_t wofs = (uint32_t)((q >> 1) * (W4 ? 512 : 1024) + (q & 1) * (W4 ? 256 : 512) + r * (W4 ? 8 : 16));
    auto load_w = [&]() {
#pragma unroll
        for (int i = 0; i < BPW; ++i) {
            const int b = b0 + i < nb ? b0 + i : nb - 1;
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                const int t = n0 + a * 16 < N ? n0 / 16 + a : N / 16 - 1;      // N is a multiple of 16
                // the lane's first 16 input channels: k block 2 b + q / 2, piece 2 (q % 2) of it
                const uint8_t *src = Wc + ((size_t)t * (K >> 6) + 2 * b) * (W4 ? 512 : 1024) + wofs;
                if constexpr (W4) {
                    const uint2 lo = *reinterpret_cast<const uint2 *>(src), hi = *reinterpret_cast<const uint2 *>(src + 128);
                    wf[i][a][0] = make_uint4(lo.x, lo.y, hi.x, hi.y);
                } else {
                    wf[i][a][0] = *reinterpret_cast<const uint4 *>(src);
                    wf[i][a][1] = *reinterpret_cast<const uint4 *>(src + 256);
                }
            }
        }
    };
    if constexpr (!kLateW) load_w();

    float v[BPW][32];
    float amax = 0.0f, amin = 0.0f;
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint4 x = raw[i][c];
            const float4 d0 = dv[2 * c], d1 = dv[2 * c + 1];
            v[i][8 * c + 0] = bf16_lo(x.x) * d0.x; v[i][8 * c + 1] = bf16_hi(x.x) * d0.y;
            v[i][8 * c + 2] = bf16_lo(x.y) * d0.z; v[i][8 * c + 3] = bf16_hi(x.y) * d0.w;
            v[i][8 * c + 4] = bf16_lo(x.z) * d1.x; v[i][8 * c + 5] = bf16_hi(x.z) * d1.y;
            v[i][8 * c + 6] = bf16_lo(x.w) * d1.z; v[i][8 * c + 7] = bf16_hi(x.w) * d1.w;
        }
        if (i + 1 < BPW) load_d(i + 1);
        fwht128_quarters(v[i]);
#pragma unroll
        for (int j = 0; j < 32; j += 2) {
            if constexpr (ASYM) {
                amax = fmaxf(fmaxf(amax, v[i][j]), v[i][j + 1]);
                amin = fminf(fminf(amin, v[i][j]), v[i][j + 1]);
            } else {
                amax = fmaxf(fmaxf(amax, fabsf(v[i][j])), fabsf(v[i][j + 1]));
            }
        }
    }
    if constexpr (kLateW) {
        __builtin_amdgcn_sched_barrier(0);
        load_w();
        __builtin_amdgcn_sched_barrier(0);
    }
    // token extremes: over the lane's four quarters, then over the waves (a clamped block repeats the row's
    // last one and changes nothing)
    amax = fmaxf(amax, __shfl_xor(amax, 16));
    amax = fmaxf(amax, __shfl_xor(amax, 32));
    if constexpr (ASYM) {
        amin = fminf(amin, __shfl_xor(amin, 16));
        amin = fminf(amin, __shfl_xor(amin, 32));
    }
    if (q == 0) {
        ext_s[wave * 32 + r] = amax;
        if constexpr (ASYM) ext_s[wave * 32 + 16 + r] = amin;
    }
    // operands of the epilogue for the wave's first channel tile: requested here, used after the last barrier
    const int a_own = wave < TN ? wave : 0;
    const int n_own = n0 + a_own * 16 + q * 4 < N ? n0 + a_own * 16 + q * 4 : N - 4;
    float4 sw_own = make_float4(1.f, 1.f, 1.f, 1.f), bi_own = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (!W4) sw_own = *reinterpret_cast<const float4 *>(sw + n_own);
    if (bias) bi_own = *reinterpret_cast<const float4 *>(bias + n_own);
    __syncthreads();
    for (int w = 0; w < nw; ++w) {
        amax = fmaxf(amax, ext_s[w * 32 + r]);
        if constexpr (ASYM) amin = fminf(amin, ext_s[w * 32 + 16 + r]);
    }
    const TokenRangeQuant rq(amin, amax);            // ASYM
    const float inv = token_inv_scale(amax);
    auto code_bits = [&](float x) -> uint32_t {
        if constexpr (ASYM) return rq.bits(x);
        else return quant_bits(x, inv);
    };

    v4i acc[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) acc[a] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
        if (b0 + i < nb) {                           // wave-uniform
            v4i xf[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float *p = v[i] + 16 * h + 4 * w;
                    xf[h][w] = (int)pack4_low_bytes(code_bits(p[0]), code_bits(p[1]), code_bits(p[2]), code_bits(p[3]));
                }
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                v4i wl, wh;
                if constexpr (W4) {
                    const uint4 p = wf[i][a][0];     // 16 * code, see Weights
                    wl = v4i{(int)((p.x << 4) & 0xF0F0F0F0u), (int)(p.x & 0xF0F0F0F0u),
                             (int)((p.y << 4) & 0xF0F0F0F0u), (int)(p.y & 0xF0F0F0F0u)};
                    wh = v4i{(int)((p.z << 4) & 0xF0F0F0F0u), (int)(p.z & 0xF0F0F0F0u),
                             (int)((p.w << 4) & 0xF0F0F0F0u), (int)(p.w & 0xF0F0F0F0u)};
                } else {
                    wl = __builtin_bit_cast(v4i, wf[i][a][0]);
                    wh = __builtin_bit_cast(v4i, wf[i][a][1]);
                }
                acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl, xf[0], W4 ? v4i{0, 0, 0, 0} : acc[a], 0, 0, 0);
                acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh, xf[1], acc[a], 0, 0, 0);
                if constexpr (W4) part[((b0 + i) * TN + a) * 64 + lane] = acc[a];
            }
        }
    }
    if constexpr (!W4) {
#pragma unroll
        for (int a = 0; a < TN; ++a) part[(wave * TN + a) * 64 + lane] = acc[a];
    }
    __syncthreads();

    // wave w finishes channel tiles w, w + waves, ...: lane holds channels n .. n + 3 of token r
    for (int a = wave; a < TN; a += nw) {
        const int n = n0 + a * 16 + q * 4;
        if (n >= N || !tok_ok) continue;
        float4 s = sw_own, bi = bi_own;
        if (a != wave) {
            if constexpr (!W4) s = *reinterpret_cast<const float4 *>(sw + n);
            if (bias) bi = *reinterpret_cast<const float4 *>(bias + n);
        }
        v4f f;
        if constexpr (W4) {
            // the groups' sums in ascending order, each with its scale, as the other int4 products add them
            f = v4f{0.f, 0.f, 0.f, 0.f};
            for (int g = 0; g < nb; ++g) {
                const float4 sg = *reinterpret_cast<const float4 *>(sw + (size_t)g * N + n);
                const v4i t = part[(g * TN + a) * 64 + lane];
                f[0] += sg.x * (float)t[0]; f[1] += sg.y * (float)t[1];
                f[2] += sg.z * (float)t[2]; f[3] += sg.w * (float)t[3];
            }
            const float sxm = token_scale(amax) * 0.0625f;
            f = v4f{sxm * f[0] + bi.x, sxm * f[1] + bi.y, sxm * f[2] + bi.z, sxm * f[3] + bi.w};
        } else {
            v4i sum = part[a * 64 + lane];
            for (int w = 1; w < nw; ++w) sum += part[(w * TN + a) * 64 + lane];
            float sxm;
            if constexpr (ASYM) {
                const int4 cs = *reinterpret_cast<const int4 *>(colsum + n);
                sum += v4i{rq.zc * cs.x, rq.zc * cs.y, rq.zc * cs.z, rq.zc * cs.w};
                sxm = rq.scale;
            } else {
                sxm = token_scale(amax);
            }
            f = v4f{(float)sum[0] * sxm * s.x + bi.x, (float)sum[1] * sxm * s.y + bi.y,
                    (float)sum[2] * sxm * s.z + bi.z, (float)sum[3] * sxm * s.w + bi.w};
        }
        uint2 o;
        o.x = pack_bf16x2(f[0], f[1]);
        o.y = pack_bf16x2(f[2], f[3]);
        *reinterpret_cast<uint2 *>(Y + (int64_t)m * ldy + n) = o;
    }
}

int small_blocks_per_wave(int K) { return (K / kBlock + 11) / 12; }

// Channel tiles (of 16) per workgroup: the narrowest of the built ones whose grid is one round of workgroups,
// else the widest.  Several blocks per wave leave registers for one or two tiles only.
// A round is one workgroup per compute unit, but a workgroup of one or two blocks is one or two waves: it finishes its
// tiles one after the other, and a compute unit has room for more of them: four.  With two blocks that is for where three
// tiles do not make one round, and from two tiles on (with one a wave rotates more than it multiplies).  us, one workgroup
// per compute unit against this (int8; with zero points): 128 -> 512 at 700 / 1024 tokens 5.8 / 5.9, 4.0 / 4.3 (6.4 / 6.5,
// 4.2 / 4.5); 256 -> 512 at 700 / 1024 5.4 / 5.4, 4.5 / 4.9 (6.0 / 6.1, 4.8 / 5.3); three blocks gain nothing (384 -> 512 at
// 1024 5.4, in 704 workgroups 5.6).
int small_tiles(int64_t M, int K, int N)
{
    const int64_t panels = (M + 15) / 16, cus = num_cus();
    static constexpr int opts[] = {1, 2, 3, 5, 9};
    const int bpw = small_blocks_per_wave(K), nb = K / kBlock;
    const int n_opts = bpw == 1 ? 5 : 2;
    auto grid = [&](int tn) { return panels * ((N + tn * 16 - 1) / (tn * 16)); };
    const bool several = nb == 1 || (nb == 2 && grid(3) > cus);
    for (int i = 0; i < n_opts; ++i)
        if (grid(opts[i]) <= (several && (nb == 1 || i > 0) ? 4 * cus : cus)) return opts[i];
    return opts[n_opts - 1];
}

// Workgroups of the widest tile: what tells how many rounds a shape needs at least.
int64_t small_workgroups(int64_t M, int K, int N)
{
    const int bn = small_blocks_per_wave(K) == 1 ? 144 : 32;
    return ((M + 15) / 16) * ((N + bn - 1) / bn);
}

template <int TN, int BPW, bool W4, bool ASYM>
hipError_t launch_small(const FusedArgs &a, hipStream_t st)
{
    const int nb = a.K / kBlock, nw = (nb + BPW - 1) / BPW;
    const size_t smem = 12 * 32 * 4 + (size_t)(W4 ? nb : nw) * TN * 1024;
    auto kern = linear_fused_small_kernel<TN, BPW, W4, ASYM>;
    if (smem > 64 * 1024)
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem); e != hipSuccess) return e;
    // consecutive workgroups take the channel tiles of one panel
    const dim3 grid((unsigned)((a.N + TN * 16 - 1) / (TN * 16)), (unsigned)((a.M + 15) / 16));
    hipLaunchKernelGGL(kern, grid, dim3(64 * nw), smem, st, a.X, a.diag, static_cast<const uint8_t *>(a.Wc), a.ldx,
                       (int)a.M, a.K, a.N, a.sw, a.bias, a.colsum, a.Y, a.ldy);
    return hipGetLastError();
}

template <bool W4, bool ASYM>
hipError_t launch_small_any(const FusedArgs &a, hipStream_t st)
{
    const int tn = small_tiles(a.M, a.K, a.N);
    switch (small_blocks_per_wave(a.K)) {
        case 1:
            switch (tn) {
                case 1: return launch_small<1, 1, W4, ASYM>(a, st);
                case 2: return launch_small<2, 1, W4, ASYM>(a, st);
                case 3: return launch_small<3, 1, W4, ASYM>(a, st);
                case 5: return launch_small<5, 1, W4, ASYM>(a, st);
                default: return launch_small<9, 1, W4, ASYM>(a, st);
            }
        case 2: return tn == 1 ? launch_small<1, 2, W4, ASYM>(a, st) : launch_small<2, 2, W4, ASYM>(a, st);
        default: return tn == 1 ? launch_small<1, 3, W4, ASYM>(a, st) : launch_small<2, 3, W4, ASYM>(a, st);
    }
}

template <int BM, int T, int S, bool W4, bool ASYM>
hipError_t launch_one(const FusedArgs &a, hipStream_t st)
{
    FusedArgs g = a;
    const int64_t panels = (g.M + BM - 1) / BM;
    g.tiles_n = (g.N + kBN - 1) / kBN;
    // enough workgroups to fill the compute units twice; every extra split repeats the prologue
    int64_t want = (2 * num_cus() + panels - 1) / panels;
    want = want < 1 ? 1 : (want > g.tiles_n ? g.tiles_n : want);
    const int tiles_per = (int)((g.tiles_n + want - 1) / want);
    g.nsplit = (g.tiles_n + tiles_per - 1) / tiles_per;   // no workgroup without a channel tile
    const size_t smem = (size_t)BM * (g.K + kPad) + 2 * (size_t)kBN * (kBK + kPad) + 2 * BM * sizeof(float);
    auto kern = linear_fused_kernel<BM, T, S, W4, ASYM>;
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)panels, (unsigned)g.nsplit), dim3(kThreads), smem, st, g);
    return hipGetLastError();
}

template <int BM, int S, bool W4, bool ASYM>
hipError_t launch_t(int T, const FusedArgs &a, hipStream_t st)
{
    if (T <= 3) return launch_one<BM, 3, S, W4, ASYM>(a, st);
    if (T <= 6) return launch_one<BM, 6, S, W4, ASYM>(a, st);
    if (T <= 9) return launch_one<BM, 9, S, W4, ASYM>(a, st);
    return launch_one<BM, 12, S, W4, ASYM>(a, st);
}

template <bool W4, bool ASYM = false>
hipError_t launch_w(const FusedArgs &a, hipStream_t st)
{
    const int nb = a.K / kBlock;
    if (nb <= 12) return launch_t<64, 1, W4, ASYM>(nb, a, st);
    if (nb <= 24) return launch_t<32, 2, W4, ASYM>((nb + 1) / 2, a, st);
    return launch_t<16, 4, W4, ASYM>((nb + 3) / 4, a, st);
}

}  // namespace

bool fused_supports(int K) { return K % kBlock == 0 && K / kBlock <= 48; }

// The few-token kernel: few enough workgroups that repeating the rotation per channel tile costs less than a second launch.
bool fused_takes_few_tokens(int64_t M, int K, int N)
{
    return K <= kSmallMaxBlocks * kBlock && small_workgroups(M, K, N) <= kSmallMaxWorkgroups;
}

// The layer's choice: the few-token kernel in a single round of workgroups (two of the small ones that one or two blocks
// make).  In a second round the repeated rotation costs more than the pair's second launch.  us, fused against the pair: 1152 ->
// 4608 at 128 tokens (256 workgroups) 6.9 / 8.7, at 256 12.0 / 11.3; 768 -> 3072 at 256 (352) 10.4 / 8.8; 256 -> 512 at 2048
// (512) 6.2 / 7.0, at 4096 12.6 / 8.2; int4 1152 -> 4608 at 128 7.5 / 11.0, at 256 13.3 / 11.2.  Where a wave has two or three
// blocks the line dates from a slower pair: it still holds at 1664 -> 1152 (64 tokens 7.0 / 7.2; int4 7.5 / 8.4) and for int4 up to
// 3072 channels (2304 -> 1152 at 64 9.1 / 9.3), no longer for int8 from 2304 on (2304 -> 1152 at 16 tokens 7.8 / 7.0, 4608 ->
// 1152 at 16 / 64 11.9 / 8.4, 14.3 / 9.2) and for int4 at 4608 (at 64 13.9 / 12.1).  Those are replays of a graph: launched by the
// host one by one, a second launch costs 3 to 5 us (2176 -> 176 at 64 tokens 7.2 / 10.5; the four linears of a block of width
// 1024 at one token 23 / 29), so the line stays.
bool fused_pays(int64_t M, int K, int N)
{
    return M > 0 && K % kBlock == 0 && K <= kSmallMaxBlocks * kBlock &&
           small_workgroups(M, K, N) <= (int64_t)num_cus() * (K <= 2 * kBlock ? 2 : 1);
}

// Where trdq_layer_forward takes the fused kernel for a caller that gave no workspace: a fixed range of shapes, so that
// which calls need one does not move with the measured choice above.
bool fused_needs_no_workspace(int64_t M, int K, int N, int wbits)
{
    if (wbits != 8 || K > 1536 || K % kBlock != 0 || M <= 0) return false;
    const int bn = N % 144 == 0 ? 144 : 128;
    return ((M + 15) / 16) * ((N + bn - 1) / bn) <= num_cus();
}

hipError_t launch_linear_fused(const Weights &w, const uint16_t *X, int64_t M, int64_t ldx,
                               const float *diag, const float *bias, uint16_t *Y, int64_t ldy,
                               hipStream_t st, bool asym)
{
    if (M == 0) return hipSuccess;
    if (asym && (w.wbits != 8 || !w.colsum)) return hipErrorInvalidValue;
    FusedArgs a;
    a.X = X; a.diag = diag; a.Wc = w.codes; a.sw = w.scales; a.bias = bias; a.colsum = w.colsum; a.Y = Y;
    a.M = M; a.ldx = ldx; a.ldy = ldy; a.K = w.K; a.N = w.N; a.tiles_n = 0; a.nsplit = 1;
    if (fused_takes_few_tokens(a.M, a.K, a.N)) {
        a.Wc = w.codes_tiled;
        if (asym) return launch_small_any<false, true>(a, st);
        return w.wbits == 4 ? launch_small_any<true, false>(a, st) : launch_small_any<false, false>(a, st);
    }
    if (asym) return launch_w<false, true>(a, st);
    return w.wbits == 4 ? launch_w<true>(a, st) : launch_w<false>(a, st);
}

}  // namespace trdq
