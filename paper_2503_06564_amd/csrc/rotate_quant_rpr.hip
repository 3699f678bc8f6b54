// rotate_quant_rpr: the full activation transform of Eq. 9,
//   G_t(X) = (X . Delta_t) . R^(1) . P . R^(2),
// first block rotation, zigzag permutation P (Sec. 3.2), second block rotation, followed by the
// per-token dynamic int8 quantiser (Eq. 1-2 symmetric, Eq. 1-3 with zero points).  Both rotations use the same
// block-diagonal Hadamard blocks as rotate_quant; (U P)[k'] = U[perm[k']].
//
// The permutation moves channels between blocks, so a token's whole rotated row has to exist before the second rotation
// starts: a workgroup owns 4 QUADS tokens and keeps their first-rotation output in LDS as fp32.
//   stage 1: a wave rotates its blocks, four tokens at a time (16 lanes to a token's block, 8 channels to a lane), and
//            writes them to LDS by channel;
//   stage 2: it gathers the channels perm[k'] of its output blocks from LDS, rotates them the same way, keeps them in
//            registers until the token maxima are known (exchanged through LDS), then quantises and stores.
// What bounds it is vector issue: 128 channels of 16 tokens cost about 650 vector instructions.  The rotation is butterflies
// on the vector ALU: three stages in the lane and four across the 16 lanes, each of the latter one multiply-add whose
// operand comes from the other lane (the form that multiplied by H_16 on the fp32 matrix instruction held the vector
// ALU for 1024 cycles per 16-token block and rotation, twice the cost, and its 16 columns asked for workgroups of 16 or
// 8 tokens: at K = 4608 one per compute unit, each phase of which waited for the one before).
// us at 4096 / 32768 tokens, that form and this one: 1152 channels 10.0 / 65.6 -> 6.7 / 34.6 (3.3 TB/s), 4608 channels
// 31.7 / 231 -> 17.8 / 122 (3.7 TB/s).  Relative error against float64 1.3e-7 -> 1.0e-7 (sums by pairs, and the diagonal
// inside the first stage's multiply-add).
// Both rotations are unnormalised; the factor 1/128 goes into the scale.  Entries of perm are clamped to [0, K) on the
// way in, so a bad table gives wrong numbers, never an access outside the row.
#include "device_utils.h"
#include "rotate_lanes.h"
#include "trdq_internal.h"

namespace trdq {

namespace {

constexpr int kRowPad = 4;     // floats of padding per LDS row

// QUADS: groups of four tokens per workgroup; SPW: most blocks per wave; ASYM: zero points (codes stored as q - 128,
// zc[i] = 128 - z_i), as in rotate_quant.
template <int QUADS, int SPW, bool ASYM>
__global__ __launch_bounds__(768, 6) void rotate_quant_rpr_kernel(
    const uint16_t *__restrict__ X, int64_t M, int nb, int64_t ldx,
    const float *__restrict__ diag, const int32_t *__restrict__ perm,
    int8_t *__restrict__ Xq, float *__restrict__ sx, int32_t *__restrict__ zc,
    const uint4 *__restrict__ warm, int64_t warm_chunks)
{
    constexpr int TOK = 4 * QUADS;
    extern __shared__ __align__(16) float lds[];
    const int K = nb * kBlock;
    const int nw = blockDim.x >> 6;
    const int rowf = K + kRowPad;                    // floats per LDS row
    float *const T = lds;                            // [TOK][rowf]: first-rotation output
    float *const ext_s = lds + (size_t)TOK * rowf;   // [2][nw][TOK] (maxima, minima); after it a 1 KB dump area for the weight copies

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t4 = lane >> 4;                        // token of the quad
    const Lane16 ln(lane & 15);
    const int c_in = (15 - ln.chunk) * 8, c_out = ln.chunk * 8;
    const int64_t m0 = (int64_t)blockIdx.x * TOK;

    // ---- stage 1: T[token][.] = (x * d) H_128 per block ------------------------------------------
    // everything is requested first; a block past the row is clamped (a redundant, cached read)
    uint4 raw[SPW][QUADS];
    float4 dg[SPW][2];
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i < nb ? wave + nw * i : nb - 1;    // wave-uniform
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            int64_t token = m0 + q * 4 + t4;
            if (token >= M) token = M - 1;           // clamped: rotated like the others, never stored
            raw[i][q] = *reinterpret_cast<const uint4 *>(X + token * ldx + b * kBlock + c_in);
        }
        dg[i][0] = dg[i][1] = make_float4(1.f, 1.f, 1.f, 1.f);
        if (diag) {
            dg[i][0] = *reinterpret_cast<const float4 *>(diag + b * kBlock + c_in);
            dg[i][1] = *reinterpret_cast<const float4 *>(diag + b * kBlock + c_in + 4);
        }
    }
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i;
        if (b < nb) {
            const float4 d0 = dg[i][0], d1 = dg[i][1];
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                const uint4 x = raw[i][q];
                float v[8];
                scaled_h8(x, d0, d1, v);
                cross16(v, ln);
                float *dst = T + (size_t)(q * 4 + t4) * rowf + b * kBlock + c_out;
                *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4 *>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
            }
        }
    }
    // Optional: pull the following product's weight codes through the memory-side cache (see
    // rotate_quant): up to four direct-to-LDS copies per wave into a dump area nobody reads.
    if (warm_chunks > 0) {
        const uint32_t dump = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)lds +
                              (uint32_t)(sizeof(float) * ((size_t)TOK * rowf + (size_t)nw * 2 * TOK));
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
    // the channels this lane gathers, requested before the barrier
    int4 idx[SPW][2];
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i < nb ? wave + nw * i : nb - 1;
        idx[i][0] = *reinterpret_cast<const int4 *>(perm + b * kBlock + c_in);
        idx[i][1] = *reinterpret_cast<const int4 *>(perm + b * kBlock + c_in + 4);
    }
    __syncthreads();

    // ---- stage 2: gather by perm, rotate again, keep in registers ---------------------------------
    float out[SPW][QUADS][8];
    float amax[QUADS], amin[QUADS];                  // ASYM: maximum (>= 0) and minimum (<= 0); else the absolute maximum
#pragma unroll
    for (int q = 0; q < QUADS; ++q) amax[q] = amin[q] = 0.0f;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int b = wave + nw * i;
        if (b < nb) {
            int k[8] = {idx[i][0].x, idx[i][0].y, idx[i][0].z, idx[i][0].w, idx[i][1].x, idx[i][1].y, idx[i][1].z, idx[i][1].w};
#pragma unroll
            for (int j = 0; j < 8; ++j) k[j] = max(0, min(k[j], K - 1)) + t4 * rowf;
#pragma unroll
            for (int q = 0; q < QUADS; ++q) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = T[k[j] + q * 4 * rowf];
                cross16(v, ln);
                fwht8_inlane(v);
#pragma unroll
                for (int j = 0; j < 8; ++j) out[i][q][j] = v[j];
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

    // out holds 128 * V.  Symmetric: s_x = max|V| / 127; codes = rint(V / s_x) = rint(out * 127 / max|out|).
    // Asymmetric (range [lo, hi] with lo <= 0 <= hi): s_x = (hi - lo) / 255, z = -rint(lo / s_x), stored code =
    // clamp(rint(V / s_x) + z, 0, 255) - 128; the integer offset rides in the rounding constant of the same FMA.
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
                sx[token] = range * (0.0078125f / 255.0f);
                zc[token] = 128 - (int)z;
            }
        } else {
            inv = amax[q] > 0.0f ? 127.0f / amax[q] : 0.0f;
            if (wave == 0 && (lane & 15) == 0 && token_ok) sx[token] = amax[q] * (0.0078125f / 127.0f);
        }
        auto code_bits = [&](float v) -> uint32_t {
            const float t = __builtin_fmaf(v, inv, magic);
            // symmetric codes cannot leave +-127; the clamp only acts on the asymmetric range ends
            return __float_as_uint(ASYM ? __builtin_amdgcn_fmed3f(t, kRoundMagic - 128.0f, kRoundMagic + 127.0f) : t);
        };
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
            const int b = wave + nw * i;
            if (b < nb && token_ok) {
                const float (&v)[8] = out[i][q];
                uint2 c;
                c.x = pack4_low_bytes(code_bits(v[0]), code_bits(v[1]), code_bits(v[2]), code_bits(v[3]));
                c.y = pack4_low_bytes(code_bits(v[4]), code_bits(v[5]), code_bits(v[6]), code_bits(v[7]));
                *reinterpret_cast<uint2 *>(Xq + token * (int64_t)K + b * kBlock + c_out) = c;
            }
        }
    }
    // the copies to the dump area must have landed before the workgroup's LDS is given away
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int QUADS, int SPW>
hipError_t launch_rpr(const uint16_t *X, int64_t M, int nb, int64_t ldx, const float *diag,
                      const int32_t *perm, int8_t *Xq, float *sx, int32_t *zc, const void *warm, int64_t warm_bytes,
                      hipStream_t st)
{
    constexpr int TOK = 4 * QUADS;
    const int K = nb * kBlock, nw = (nb + SPW - 1) / SPW;
    const size_t smem = sizeof(float) * ((size_t)TOK * (K + kRowPad) + (size_t)nw * 2 * TOK) + 1024;
    auto kern = zc ? rotate_quant_rpr_kernel<QUADS, SPW, true> : rotate_quant_rpr_kernel<QUADS, SPW, false>;
    if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), 160 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)((M + TOK - 1) / TOK)), dim3(64 * nw), smem, st,
                       X, M, nb, ldx, diag, perm, Xq, sx, zc, static_cast<const uint4 *>(warm),
                       (warm && warm_bytes < ((int64_t)1 << 32)) ? warm_bytes / 16 : 0);
    return hipGetLastError();
}

}  // namespace

// K up to 4608 (36 blocks): 12 waves x 3 blocks.
bool rotate_quant_rpr_supports(int K) { return K > 0 && K % kBlock == 0 && K / kBlock <= 36; }

hipError_t launch_rotate_quant_rpr(const uint16_t *X, int64_t M, int K, int64_t ldx, const float *diag,
                                   const int32_t *perm, int8_t *Xq, float *sx, const void *warm, int64_t warm_bytes,
                                   hipStream_t st, int32_t *zc)
{
    if (M == 0) return hipSuccess;
    if (!rotate_quant_rpr_supports(K)) return hipErrorInvalidValue;
    const int nb = K / kBlock;
    constexpr int64_t most = (int64_t)1 << 24;       // tokens per launch: a grid holds fewer than 2^32 threads
    if (M > most) {
        hipError_t e = launch_rotate_quant_rpr(X, most, K, ldx, diag, perm, Xq, sx, warm, warm_bytes, st, zc);
        if (e != hipSuccess) return e;
        return launch_rotate_quant_rpr(X + most * ldx, M - most, K, ldx, diag, perm, Xq + most * K, sx + most, nullptr, 0, st,
                                       zc ? zc + most : nullptr);
    }
    // Eight tokens per workgroup while a wave has one block: the indices and the diagonal serve two quads (us at 4096 /
    // 32768 tokens, eight against four: 1152 channels 6.7 / 34.6, 6.8 / 39.2; 1536 7.7 / 45.5, 8.4 / 49.6).  Four beyond, where
    // eight leave room for one or two workgroups per compute unit (2304 10.9 / 61.1, 10.2 / 58.8; 4608 20.8 / 141, 17.8 / 122).
    if (nb <= 12) return launch_rpr<2, 1>(X, M, nb, ldx, diag, perm, Xq, sx, zc, warm, warm_bytes, st);
    if (nb <= 24) return launch_rpr<1, 2>(X, M, nb, ldx, diag, perm, Xq, sx, zc, warm, warm_bytes, st);
    return launch_rpr<1, 3>(X, M, nb, ldx, diag, perm, Xq, sx, zc, warm, warm_bytes, st);
}

}  // namespace trdq
