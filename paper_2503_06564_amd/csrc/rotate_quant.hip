// rotate_quant: G_t(X) = (X . Delta_t) . R of Eq. 10 followed by the per-token dynamic
// int8 quantiser (Eq. 1-2 symmetric, Eq. 1-3 with zero points).  One streaming pass: 2 bytes in, 1 byte out
// per element, 4 bytes of scale per token.
//
// A workgroup owns 4 QUADS tokens and its waves split the K / 128 blocks; 16 lanes rotate one token's block, 8 channels
// to a lane (rotate_lanes.h), and keep the results until the token maximum, exchanged through LDS, is known.
//
// What bounds it is latency up to a few thousand tokens and the memory beyond.  The form before this one put the H_16 factor of
// the rotation on the bf16 matrix pipe (the diagonal as three exact bf16 pieces): 241 vector instructions per 16 tokens and
// block against 344 here, but its 166 ... 198 registers left two or three waves per SIMD, its 16-token workgroups one per
// compute unit at 4096 tokens, and a workgroup began by staging the pieces of the diagonal in LDS.  Here a wave needs 50
// registers and no table, so six to eight waves per SIMD cover each other's loads, exchange and stores, and the extra vector
// work runs under the memory time.  us, that form and this one, alone and back to back, inputs in the caches / behind the
// memory-side one:
//   rows          256 tokens x 1152  5.0 ->  3.0             4096 x 1152   5.7 ->  4.5 /  6.1 ->  5.4   32768 x 1152 22.5 -> 20.7 / 26.9 -> 23.4
//                 256 x 4608        10.6 ->  3.9             4096 x 4608  14.7 -> 12.4 / 17.0 -> 14.9   32768 x 4608 95.9 -> 81.5 / 97.7 -> 81.6
//   block-tiled   4096 x 1152        5.5 ->  4.5 /  5.9 ->  5.4   32768 x 1152 22.1 -> 20.9 / 26.1 -> 26.5
//                 4096 x 4608       13.6 -> 12.6 / 15.9 -> 14.7   32768 x 4608 92.8 -> 84.7 / 92.3 -> 86.2
// (block-tiled 32768 x 4608 since its input is read non-temporally: 79 / 82)
// (a kernel that only reads two bytes and writes one: 2.8 / 4.0, 9.5 / 12.0 at 4096 tokens, 18.8 / 20.0, 74.3 / 74.5 at 32768).
// Between the products of a transformer block, whose outputs are still being written back, it takes 7.2 and 13.5 us at 4096
// tokens and 28.5 and 101 at 32768 (kernel trace).  Codes that differ from float64's: 2.2e-6 of them against 2.6e-6 at K = 1152.
#include "device_utils.h"
#include "rotate_lanes.h"
#include "trdq_internal.h"

namespace trdq {

namespace {

// From here on (in values; zero points: their own line) the input is read as what nobody will read again, so that more of the codes stay
// for the product in the memory-side cache of 256 MB.  us on one input, ordinary / non-temporal: 113 M values 24576 x 4608 as rows 59.2 / 57.0,
// block-tiled 61.7 / 57.8, with zero points 59.5 / 57.6, 49152 x 2304 62.2 / 62.2, 67.1 / 65.3, 67.7 / 69.0; 151 M 32768 x 4608 79.7 / 73.9,
// 84.0 / 75.6, 79.7 / 75.4, 65536 x 2304 83.5 / 81.7, 90.1 / 85.4, 89.6 / 89.5; the pass and its product, 4608 -> 1152, at 24576 tokens
// 168 / 161, at 32768 230 / 210.  With fewer values an input that the cache still holds would come from memory: 90 M 38912 x 2304
// 44.1 / 48.9, 45.8 / 52.6, 49.9 / 52.9, 22400 x 4096 45.4 / 47.8, 45.8 / 48.5, 19420 x 4608 45.0 / 46.5, 44.1 / 47.2.  (Layers in which
// each pass reads what the product before it wrote gain below, too: 1152 -> 4608 -> 1152 at 24576 352 / 300.)
constexpr int64_t kOnceValues = (int64_t)108 << 20, kOnceValuesAsym = (int64_t)144 << 20;

// 16 bytes of the input; ONCE: non-temporal.  (A template: of a branch between the two loads the compiler makes one ordinary load.)
template <bool ONCE>
__device__ __forceinline__ uint4 load_in16(const uint16_t *p)
{
    if constexpr (ONCE) {
        typedef unsigned int v4u __attribute__((ext_vector_type(4)));
        const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    return *reinterpret_cast<const uint4 *>(p);
}

// QUADS: groups of four tokens per workgroup; SPW: most blocks per wave.
// ASYM: the asymmetric quantiser (per-token minimum and maximum, zero point): codes q in 0..255 are stored as q - 128 so
// that they stay int8 for the matrix instruction, and zc[i] = 128 - z_i is what the product's epilogue needs with the
// weights' column sums.
// tiled: Xq in 1 KB blocks of 16 tokens x 64 k, the 16-byte piece p of row r at p * 256 + r * 16.
template <int QUADS, int SPW, bool ASYM, bool ONCE>
__global__ __launch_bounds__(SPW <= 3 ? 768 : 576, SPW <= 3 ? 6 : 3) void rotate_quant_kernel(
    const uint16_t *__restrict__ X, int64_t M, int nb, int64_t ldx,
    const float *__restrict__ diag, int8_t *__restrict__ Xq, float *__restrict__ sx,
    int32_t *__restrict__ zc, const uint4 *__restrict__ warm, int64_t warm_chunks, float qmax, float sx_mul, int tiled)
{
    constexpr int TOK = 4 * QUADS;
    extern __shared__ __align__(16) float ext_s[];   // [2][nw][TOK] (maxima, minima); after it a 1 KB dump area for the weight copies
    const int K = nb * kBlock;
    const int nw = blockDim.x >> 6;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t4 = lane >> 4;                        // token of the quad
    const Lane16 ln(lane & 15);
    const int c_in = (15 - ln.chunk) * 8;
    const int64_t m0 = (int64_t)blockIdx.x * TOK;

    uint4 raw[SPW][QUADS];
    float4 dg[SPW][2];
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i < nb ? wave + nw * i : nb - 1;    // wave-uniform
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            int64_t token = m0 + q * 4 + t4;
            if (token >= M) token = M - 1;           // clamped: rotated like the others, never stored
            raw[i][q] = load_in16<ONCE>(X + token * ldx + b * kBlock + c_in);
        }
        dg[i][0] = dg[i][1] = make_float4(1.f, 1.f, 1.f, 1.f);
        if (diag) {
            dg[i][0] = *reinterpret_cast<const float4 *>(diag + b * kBlock + c_in);
            dg[i][1] = *reinterpret_cast<const float4 *>(diag + b * kBlock + c_in + 4);
        }
    }
    float out[SPW][QUADS][8];
    float amax[QUADS], amin[QUADS];                  // ASYM: maximum (>= 0) and minimum (<= 0); else the absolute maximum
#pragma unroll
    for (int q = 0; q < QUADS; ++q) amax[q] = amin[q] = 0.0f;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i;
        if (b < nb) {
            const float4 d0 = dg[i][0], d1 = dg[i][1];
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                const uint4 x = raw[i][q];
                float (&v)[8] = out[i][q];
                scaled_h8(x, d0, d1, v);
                cross16(v, ln);
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    if constexpr (ASYM) {
                        amax[q] = fmaxf(fmaxf(amax[q], v[j]), v[j + 1]);
                        amin[q] = fminf(fminf(amin[q], v[j]), v[j + 1]);
                    } else {
                        amax[q] = fmaxf(fmaxf(amax[q], fabsf(v[j])), fabsf(v[j + 1]));
                    }
                }
            }
        }
    }
    // Optional: read the next kernel's weights once (at most four 16-byte pieces per lane, spread over the whole grid; more
    // than that is left cold).  They only have to pass through the memory-side cache so that the product does not start on
    // cold DRAM: the copies go straight to a 1 KB dump area in LDS that nobody reads, and nothing waits for them before the
    // end of the kernel.  (The compiler does not count them among its outstanding loads: its waits can only become
    // stricter by that, because the counter retires in order.)
    if (warm_chunks > 0) {
        const uint32_t dump = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)ext_s +
                              (uint32_t)(sizeof(float) * (size_t)nw * 2 * TOK);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t c0 = ((int64_t)t * gridDim.x + blockIdx.x) * blockDim.x + (wave << 6);   // wave-uniform
            if (c0 < warm_chunks) {
                int64_t c = c0 + lane;
                if (c >= warm_chunks) c = warm_chunks - 1;
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                             :: "v"((uint32_t)(c << 4)), "s"(warm), "s"(dump) : "memory", "m0");
            }
        }
    }
    // token extremes: over the 16 lanes, then over the waves through LDS
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        amax[q] = row16_max(amax[q]);
        if constexpr (ASYM) amin[q] = -row16_max(-amin[q]);
        if ((lane & 15) == 0) {
            ext_s[wave * TOK + q * 4 + t4] = amax[q];
            if constexpr (ASYM) ext_s[(nw + wave) * TOK + q * 4 + t4] = amin[q];
        }
    }
    __syncthreads();
    // out holds sqrt(128) * V.  Symmetric: s_x = max|V| / qmax, codes = rint(V / s_x) = rint(out * qmax / max|out|), qmax =
    // 2^(bits - 1) - 1 and sx_mul = (1 / sqrt(128)) / qmax from the host.  Asymmetric (range [lo, hi] with lo <= 0 <= hi):
    // s_x = (hi - lo) / 255, z = -rint(lo / s_x), stored code = clamp(rint(V / s_x) + z, 0, 255) - 128; the integer offset
    // rides in the rounding constant of the same FMA.
    uint2 code[SPW][QUADS];
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        for (int wv = 0; wv < nw; ++wv) {
            amax[q] = fmaxf(amax[q], ext_s[wv * TOK + q * 4 + t4]);
            if constexpr (ASYM) amin[q] = fminf(amin[q], ext_s[(nw + wv) * TOK + q * 4 + t4]);
        }
        const int64_t token = m0 + q * 4 + t4;
        const bool token_ok = token < M;
        float inv, magic = kRoundMagic;
        if constexpr (ASYM) {
            const float range = amax[q] - amin[q];
            inv = range > 0.0f ? 255.0f / range : 0.0f;
            const float z = -rintf(amin[q] * inv);
            magic = kRoundMagic + (z - 128.0f);
            if (wave == 0 && (lane & 15) == 0 && token_ok) {
                sx[token] = range * (0.08838834764831845f / 255.0f);
                zc[token] = 128 - (int)z;
            }
        } else {
            inv = amax[q] > 0.0f ? qmax / amax[q] : 0.0f;
            if (wave == 0 && (lane & 15) == 0 && token_ok) sx[token] = amax[q] * sx_mul;
        }
        // symmetric codes cannot leave the int8 range; the clamp only acts on the asymmetric range ends
        auto code_bits = [&](float v) -> uint32_t {
            const float t = __builtin_fmaf(v, inv, magic);
            return __float_as_uint(ASYM ? __builtin_amdgcn_fmed3f(t, kRoundMagic - 128.0f, kRoundMagic + 127.0f) : t);
        };
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
            const float (&v)[8] = out[i][q];
            code[i][q].x = pack4_low_bytes(code_bits(v[0]), code_bits(v[1]), code_bits(v[2]), code_bits(v[3]));
            code[i][q].y = pack4_low_bytes(code_bits(v[4]), code_bits(v[5]), code_bits(v[6]), code_bits(v[7]));
        }
    }
    const int half = ln.chunk & 1, pair = ln.chunk >> 1;        // the lane's half of which 16-byte piece
    auto piece = [&](int64_t token, int b) {
        return tiled ? Xq + ((token >> 4) * (K >> 6) + 2 * b + (pair >> 2)) * (int64_t)1024 + (pair & 3) * 256 + (token & 15) * 16
                     : Xq + token * (int64_t)K + b * kBlock + pair * 16;
    };
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i;
        if constexpr (QUADS == 2) {
            // the lanes of a piece trade: each stores the 16 bytes of one quad's token
            const uint2 give = half ? code[i][0] : code[i][1], keep = half ? code[i][1] : code[i][0];
            uint2 got;
            got.x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give.x, kDppXor1, 0xF, 0xF, true);
            got.y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give.y, kDppXor1, 0xF, 0xF, true);
            const int64_t token = m0 + half * 4 + t4;
            if (b < nb && token < M)
                *reinterpret_cast<uint4 *>(piece(token, b)) =
                    half ? make_uint4(got.x, got.y, keep.x, keep.y) : make_uint4(keep.x, keep.y, got.x, got.y);
        } else {
            static_assert(QUADS == 1, "one or two quads");
            const int64_t token = m0 + t4;
            if (b < nb && token < M) *reinterpret_cast<uint2 *>(piece(token, b) + half * 8) = code[i][0];
        }
    }
    // the copies to the dump area must have landed before the workgroup's LDS is given away
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace

bool rotate_quant_reads_once(int64_t M, int K, bool asym) { return M * K >= (asym ? kOnceValuesAsym : kOnceValues); }

namespace {

template <int QUADS, int SPW>
hipError_t launch_spw(const uint16_t *X, int64_t M, int nb, int64_t ldx, const float *diag,
                      int8_t *Xq, float *sx, int32_t *zc, const void *warm, int64_t warm_bytes, hipStream_t st,
                      int abits, bool tiled)
{
    constexpr int TOK = 4 * QUADS;
    const int nw = (nb + SPW - 1) / SPW;
    const float qmax = (float)((1 << (abits - 1)) - 1);
    const float sx_mul = 0.08838834764831845f / qmax;
    const size_t smem = sizeof(float) * (size_t)nw * 2 * TOK + 1024;                 // extremes, dump area
    const int64_t warm_chunks = (warm && warm_bytes < ((int64_t)1 << 32)) ? warm_bytes / 16 : 0;   // 32-bit byte offsets in the copy
    const bool once = rotate_quant_reads_once(M, nb * kBlock, zc != nullptr);
    auto kern = zc ? (once ? rotate_quant_kernel<QUADS, SPW, true, true> : rotate_quant_kernel<QUADS, SPW, true, false>)
                   : (once ? rotate_quant_kernel<QUADS, SPW, false, true> : rotate_quant_kernel<QUADS, SPW, false, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)((M + TOK - 1) / TOK)), dim3(64 * nw), smem, st,
                       X, M, nb, ldx, diag, Xq, sx, zc, static_cast<const uint4 *>(warm), warm_chunks, qmax, sx_mul, (int)tiled);
    return hipGetLastError();
}

}  // namespace

// Largest K of the zero points, other widths than 8 bits and tiled codes, and of the symmetric 8-bit pass (in blocks).
constexpr int kRQMaxBlocks = 36, kRQMostBlocks = 64;
constexpr int64_t kRQMostTokens = (int64_t)1 << 24;  // per launch: a grid holds fewer than 2^32 threads

hipError_t launch_rotate_quant(const uint16_t *X, int64_t M, int K, int64_t ldx, const float *diag,
                               int8_t *Xq, float *sx, int32_t *zc, const void *warm, int64_t warm_bytes, hipStream_t st,
                               int abits, bool tiled)
{
    if (M == 0) return hipSuccess;
    if (abits < 2 || abits > 8) return hipErrorInvalidValue;
    const int nb = K / kBlock;
    if (nb > kRQMostBlocks || (nb > kRQMaxBlocks && (zc || abits != 8 || tiled))) return hipErrorInvalidValue;
    if (M > kRQMostTokens) {
        hipError_t e = launch_rotate_quant(X, kRQMostTokens, K, ldx, diag, Xq, sx, zc, warm, warm_bytes, st, abits, tiled);
        if (e != hipSuccess) return e;
        return launch_rotate_quant(X + kRQMostTokens * ldx, M - kRQMostTokens, K, ldx, diag, Xq + kRQMostTokens * K,
                                   sx + kRQMostTokens, zc ? zc + kRQMostTokens : nullptr, nullptr, 0, st, abits, tiled);
    }
    auto go = [&](auto kern) { return kern(X, M, nb, ldx, diag, Xq, sx, zc, warm, warm_bytes, st, abits, tiled); };
    // Three blocks per wave (us at 4096 / 32768 tokens x 1152 with two 4.6 / 21.8, three 4.6 / 20.7, six 5.0 / 20.1); one block and
    // a wave per workgroup would leave a quad too little (128 channels at 32768 tokens: four tokens 5.0, eight 4.5); nine where
    // twelve waves leave two workgroups per compute unit and there are tokens for several rounds (4608 at 16384 / 32768
    // tokens: three 38.6 / 88.2, nine 36.4 / 79.8, at 4096 12.5 / 12.6), and beyond twelve waves of three.
    if (nb == 1) return go(launch_spw<2, 1>);
    // Four and six blocks with tokens for many rounds: a wave per quad, nobody to wait for (three per wave, a wave per quad: 512 at
    // 24576 / 32768 tokens 9.2 / 11.2, 8.5 / 10.1; 768 12.0 / 15.1, 11.1 / 13.9; 16384 tokens 8.5, 8.6; five blocks level).
    if (M >= 24576 && nb == 4) return go(launch_spw<1, 4>);
    if (M >= 24576 && nb == 6) return go(launch_spw<1, 6>);
    // Block-tiled codes of wide rows: eight tokens, so that a piece's stores are 128 consecutive bytes (4608 at 32768 tokens: four
    // 92, eight 84; 3072 61 / 53; up to 2304 channels no difference), and as many blocks per wave as leave four or eight
    // waves (three per wave make nine to eleven, of which a compute unit holds one workgroup and the last wave little
    // work).  us, three per wave against this, inputs in the memory-side cache / behind it:
    //   five:  2560 at 8192 tokens 14.2 / 16.8, 13.3 / 16.1, at 20480 29.7 / 34.3, 28.4 / 31.5
    //   seven: 3328 at 8192 19.6 / 22.1, 16.6 / 20.3, 3584 at 6144 15.7 / 19.4, 14.3 / 16.6, at 16384 35.0 / 40.0, 30.8 / 36.1
    //   four:  3840 at 8192 22.2 / 25.0, 19.1 / 22.4, 4096 at 16384 37.5 / 40.6, 34.8 / 39.1
    // With fewer tokens four per wave and four tokens (three, four: 3584 at 4096 11.0 / 14.3, 9.9 / 11.9; 4096 at 6144 17.1 /
    // 20.5, 14.5 / 18.4; at 2048 level).  Three per wave stay ahead at 22 ... 24 blocks (3072 at 8192: three 14.7 / 17.8, six
    // 15.2 / 17.6) and from 33 on, where twelve waves are even (eight tokens from 4096: 4480 there 12.4 / 16.1, 12.2 / 14.5).
    if (tiled && nb > 18) {
        if (nb <= 20 && M >= 8192) return go(launch_spw<2, 5>);
        if ((nb == 21 && M >= 8192) || (nb >= 25 && nb <= 28 && M >= 6144)) return go(launch_spw<2, 7>);
        if (nb >= 28 && nb <= 32 && M >= 3072) return M >= 8192 ? go(launch_spw<2, 4>) : go(launch_spw<1, 4>);
        if ((nb <= 24 && M >= 8192) || (nb > 32 && M >= 4096)) return go(launch_spw<2, 3>);
        return go(launch_spw<1, 3>);
    }
    if (nb > kRQMaxBlocks || (nb > 24 && M >= 8192)) return go(launch_spw<1, 9>);
    return go(launch_spw<1, 3>);
}

}  // namespace trdq
