// W8A8 integer product on block-tiled operands: 256 x 144 (and 128 x 144) output tiles, two
// workgroups per compute unit.
//
// Operation: Y = dequant(Xq . Wq^T) of Eq. 10's quantised product (per-token and per-channel
// scales, optional bias, bf16 output), the arithmetic of the other int8 kernels.
//
// Why another kernel.  With 128 x 144 tiles the k-loop is bound by what the L2 delivers into LDS
// (17 KB of copies per 72 matrix instructions) and by LDS reads (a wave tile of 32 x 144 reads
// 0.6 KB per matrix instruction).  A wave tile of 64 tokens x 144 channels needs 0.36 KB of reads
// and, as a 256 x 144 workgroup tile, 25 KB of copies per 144 matrix instructions.  Two such
// workgroups fit a compute unit only if a k-step is 64 bytes deep (three stages of 25 KB each),
// and a 64-byte-deep copy of row-major operands fetches half cache lines, which doubles the
// traffic between L2 and L1.  Hence both operands are stored in 1 KB blocks of 16 rows x 64 bytes
// of k (block (row / 16, k / 64) at ((row / 16) * K / 64 + k / 64) * 1024; inside a block the
// 16-byte piece p of row r at p * 256 + r * 16, the lane order of the matrix instruction's operand):
// one direct-to-LDS copy moves one block, eight whole cache lines, and one block is one operand
// fragment of v_mfma_i32_16x16x64_i8, read back from LDS as 1 KB in lane order.  trdq_rotate_quant_tiled writes activations in this form;
// the weights get a second copy of their codes in it when they are prepared.
//
// A launch may mix tile heights: workgroups [0, n_big) take 256-token tiles over the first nbn
// channel tiles, the others 128-token tiles over the remaining channel tiles, so that a shape
// whose 256-token tiles would fill the chip one and a half times still runs as one round of two
// workgroups per compute unit (a tall and a short one, whose prologues and epilogues fall at
// different times).
#include <type_traits>
#include <utility>

#include "gemm_common.h"

namespace trdq {
namespace gemm {

namespace {

constexpr int kBN = 144;                     // channels per tile
constexpr int kTN = kBN / 16;                // weight fragments per k-step
constexpr int kNS = 3;                       // stages of the ring
constexpr int kStageBig = (256 / 16 + kTN) * 1024;
constexpr int kParOff = 3 * kStageBig;     // epilogue operands: [144 s_w][pad][144 bias][pad][256 s_x]
constexpr int kParSw = 0, kParBias = 1024, kParSx = 2048;
constexpr int kParCs = 3072, kParZc = 4096;  // asymmetric activations: [144 column sums][pad][256 zero-point terms]
constexpr int par_bytes(bool asym) { return asym ? 5120 : 3072; }
constexpr int tiled_lds(bool asym) { return kParOff + par_bytes(asym); }   // 79872 or 81920 B: two workgroups per compute unit

// Where the activations are: kBlocks: the block-tiled form, whole tiles.  kRows: row-major [M, K], any M and N from one
// tile on.  kRowsAsym: the same with zero points.
enum { kBlocks = 0, kRows = 1, kRowsAsym = 2 };

template <int... Is, class F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, Is...>, F &&f)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for_n(F &&f)
{
    static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

// A block in memory and in LDS: the 16-byte piece p (16 bytes of k) of row r sits at p * 256 + r * 16,
// which is lane (16 p + r)'s operand of the matrix instruction at 16 bytes per lane: a copy and a
// fragment read both move the block's 1 KB in lane order.
__device__ __forceinline__ int blk_off(int r, int p) { return p * 256 + r * 16; }

__device__ __forceinline__ void copy_1k_if(int on, uint32_t voff, const void *sbase, uint32_t lds_addr)
{
    asm volatile("s_cmp_eq_u32 %3, 0\n\ts_cbranch_scc1 .Lskip%=\n\t"
                 "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n"
                 ".Lskip%=:"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr), "s"(__builtin_amdgcn_readfirstlane(on))
                 : "memory", "scc");
}

__device__ __forceinline__ void copy_256_if(int on, uint32_t voff, const void *sbase, uint32_t lds_addr)
{
    asm volatile("s_cmp_eq_u32 %3, 0\n\ts_cbranch_scc1 .Lskip%=\n\t"
                 "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1\n"
                 ".Lskip%=:"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr), "s"(__builtin_amdgcn_readfirstlane(on))
                 : "memory", "scc");
}

// First token and channel of a tile.  M need not be a multiple of the tile's height (with row-major activations neither
// of 128, and N not of the width): the last tile then starts early enough to end at the last token or channel.  What it shares with its neighbour is computed twice
// and stored twice, the same values.
__device__ __forceinline__ int64_t tile_m0(const GemmArgs &g, int tm, int bm)
{
    const int64_t m0 = (int64_t)tm * bm;
    return m0 > g.M - bm ? g.M - bm : m0;
}
template <int FORM>
__device__ __forceinline__ int tile_n0(const GemmArgs &g, int tn, int bn = kBN)
{
    const int n0 = tn * bn;
    return FORM != kBlocks && n0 > g.N - bn ? g.N - bn : n0;
}

// Row-major activations: a copy instruction moves 16 rows x 64 bytes, four lanes to a row (lanes of a quad in four
// rows take four times as long at the compute unit's address path), so the rows lie 64 bytes apart in LDS, their
// 16-byte pieces XOR-swizzled for the fragment reads.
template <int FORM>
__device__ __forceinline__ uint32_t x_copy_off(int lane, int K)
{
    if constexpr (FORM == kBlocks) return (uint32_t)(lane * 16);
    else return (uint32_t)((lane >> 2) * K + ((lane & 3) ^ chunk_swizzle<64>(lane >> 2)) * 16);
}
template <int FORM>
__device__ __forceinline__ int x_frag_off(int r, int p)
{
    if constexpr (FORM == kBlocks) return blk_off(r, p);
    else return r * 64 + (p ^ chunk_swizzle<64>(r)) * 16;
}

// One output tile of BM tokens x 144 channels.  Wave w owns token rows w * BM/4 .. of the tile
// and all 144 channels: TM = BM / 64 activation fragments (its own, which only it reads) and the
// nine weight fragments (shared) per k-step; the lane ends with channels n .. n+3 of one token per
// accumulator tile.  Per k-step: wait until the next step's blocks have landed, barrier (which
// also retires every read of the current step's stage), refill that stage with the step three
// ahead, then 9 x TM matrix instructions on the fragments in registers while the next step's
// fragments are read: a weight fragment's registers are refilled as soon as its TM instructions
// have issued, the activation fragments alternate between two sets.
template <int BM, bool DEBUG, int FORM, int LINES>
__device__ __forceinline__ void run_tile(const GemmArgs &g, int tm, int tn, int8_t *smem)
{
    constexpr int TM = BM / 64;
    constexpr int XB = BM / 16;                       // activation blocks per stage
    constexpr int STAGE = (XB + kTN) * 1024;
    constexpr int PMIN = TM + 2;                      // copies per wave and k-step: TM + 2 (wave 0: + 3)
    static_assert(kNS * STAGE <= kParOff, "ring must not reach the epilogue operands");
    static_assert(2 * PMIN + 4 < 64, "vmcnt is a 6-bit counter");

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)smem;
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c0 = __builtin_readcyclecounter();
    const uint64_t clk_t0 = wall_clock64();
#endif
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int KT = g.K >> 6;                          // k-steps
    const int64_t m0 = tile_m0(g, tm, BM);
    const int n0 = tile_n0<FORM>(g, tn);

    const int64_t gstride = (int64_t)KT * 1024;      // bytes from one 16-row group to the next
    const int8_t *const xsrc = g.Xq + (m0 + wave * TM * 16) * g.K;
    const int8_t *const wsrc = static_cast<const int8_t *>(g.Wc) + (int64_t)(n0 / 16) * gstride;
    const uint32_t voff = (uint32_t)(lane * 16);        // copies keep the block's order
    const uint32_t voffx = x_copy_off<FORM>(lane, g.K);
    constexpr int XSTEP = FORM == kBlocks ? 1024 : 64;  // bytes from one k-step of the activations to the next

    const int8_t *xs[TM], *ws[2];
#pragma unroll
    for (int b = 0; b < TM; ++b) xs[b] = xsrc + b * gstride;
#pragma unroll
    for (int i = 0; i < 2; ++i) ws[i] = wsrc + (wave + 4 * i) * gstride;
    const int8_t *const ws8 = wsrc + 8 * gstride;     // the ninth weight block: wave 0 copies it
    // copy c (0 .. TM + 2) of this wave's share of k-step s into stage st: its TM activation blocks, two
    // weight blocks, and for wave 0 the ninth weight block
    auto issue_one = [&](auto c_tag, int s, int st, auto if_tag, bool on = true) {
        constexpr int c = decltype(c_tag)::value;
        constexpr bool IF = decltype(if_tag)::value;    // requested only if `on`
        const uint32_t sbase = lds0 + st * STAGE;
        const int64_t so = (int64_t)s * 1024;
        auto copy = [&](uint32_t v, const int8_t *src, uint32_t to) {
            if constexpr (IF) copy_1k_if(on, v, src, to);
            else dma_1k(v, src, to);
        };
        if constexpr (c < TM) copy(voffx, xs[c] + (int64_t)s * XSTEP, sbase + (wave * TM + c) * 1024);
        else if constexpr (c < TM + 2) copy(voff, ws[c - TM] + so, sbase + (XB + wave + 4 * (c - TM)) * 1024);
        else copy_1k_if(wave == 0 && on, voff, ws8 + so, sbase + (XB + 8) * 1024);
    };
    auto issue = [&](int s, int st) {
        static_for_n<TM + 3>([&](auto c) { issue_one(c, s, st, std::integral_constant<bool, false>{}); });
    };

    // epilogue operands first (older than every tile copy, so the first wait covers them):
    // wave 0 the 144 channel scales, wave 1 the biases, wave 2 the BM token scales
    {
        const uint32_t par = lds0 + kParOff;
        const uint32_t v36 = (uint32_t)((lane < kBN / 4 ? lane : kBN / 4 - 1) * 16);
        const uint32_t vsx = (uint32_t)((lane < BM / 4 ? lane : BM / 4 - 1) * 16);
        copy_1k_if(wave == 0, v36, g.sw + n0, par + kParSw);
        copy_1k_if(wave == 1 && g.bias != nullptr, v36, g.bias ? g.bias + n0 : g.sw, par + kParBias);
        if (wave == 1 && g.bias == nullptr)           // no bias: zeros, so that the epilogue needs no branch
            *reinterpret_cast<uint4 *>(smem + kParOff + kParBias + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (FORM == kBlocks) {
            copy_1k_if(wave == 2, vsx, g.sx + m0, par + kParSx);
        } else {                                      // any token may be the tile's first: four-byte pieces
            copy_256_if(wave < BM / 64, (uint32_t)(lane * 4), g.sx + m0 + wave * 64, par + kParSx + wave * 256);
            if constexpr (FORM == kRowsAsym) {
                copy_256_if(wave < BM / 64, (uint32_t)(lane * 4), g.zc + m0 + wave * 64, par + kParZc + wave * 256);
                copy_1k_if(wave == 3, v36, g.colsum + n0, par + kParCs);
            }
        }
    }
    // KT is even and at least 2 (K is a multiple of 128)
    issue(0, 0);
    issue(1, 1);
    if (KT >= 4) {
        issue(2, 2);
        wait_vmcnt<2 * PMIN>();
    } else {
        wait_vmcnt<PMIN>();
    }
    __syncthreads();

#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c1 = __builtin_readcyclecounter();
    const uint64_t clk_t1 = wall_clock64();
#endif
    const int fro = blk_off(l16, lg);                 // the lane's piece of a fragment block
    const int frox = x_frag_off<FORM>(l16, lg);       // ... of an activation block
    v4i acc[kTN][TM];
#pragma unroll
    for (int a = 0; a < kTN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    v4i af[kTN], bf[2][TM];
#pragma unroll
    for (int a = 0; a < kTN; ++a) af[a] = *reinterpret_cast<const v4i *>(smem + (XB + a) * 1024 + fro);
#pragma unroll
    for (int b = 0; b < TM; ++b) bf[0][b] = *reinterpret_cast<const v4i *>(smem + (wave * TM + b) * 1024 + frox);

    int st = 0;
    // WHOLE: the loop takes all but the last two steps, its last odd one requesting nothing.  Otherwise the last pair in which
    // only the even step requests stands behind the loop, where tall tiles of row-major activations ran out of registers: 14
    // spilled, 35 with zero points, behind full waits.  us, rows 1152 -> 3456 / 4608 at 4096 tokens 21.7 / 27.4 -> 21.2 / 26.4, 4608 at
    // 16384 103 -> 98; the question on every odd copy makes it the slower one elsewhere (block-tiled 18.6 / 23.8 -> 19.1 / 24.7,
    // short tiles 6.7 -> 7.1 at 1000 x 768 -> 2304).
    constexpr bool WHOLE = BM == 256 && FORM != kBlocks;
    // One k-step on activation fragment set PAR.  REFILL: the next step exists; its fragments are read
    // while this step's matrix instructions run (after waiting for vmcnt(WAITN) and the barrier).
    // ISSUE: the step three ahead exists and is requested into this step's stage.
    // The order below is the order of issue: the scheduling fences keep the compiler from bunching
    // the LDS reads at the end of the step, where nothing would cover their latency.
    auto step = [&](auto par_tag, auto refill_tag, auto issue_tag, auto wait_tag, int kt) {
        constexpr int PAR = decltype(par_tag)::value;
        constexpr bool REFILL = decltype(refill_tag)::value;
        constexpr bool ISSUE = decltype(issue_tag)::value;
        constexpr int WAITN = decltype(wait_tag)::value;
        const int nst = (st + 1 == kNS) ? 0 : st + 1;
        const int8_t *const nxt = smem + nst * STAGE + fro;
        const int8_t *const nxtx = smem + nst * STAGE + frox;
        if constexpr (REFILL) {
            wait_vmcnt<WAITN>();                               // step kt+1 has landed (this wave's share)
            __syncthreads();                                   // ... everyone's; step kt's stage is retired
#pragma unroll
            for (int b = 0; b < TM; ++b)
                bf[1 - PAR][b] = *reinterpret_cast<const v4i *>(nxtx + (wave * TM + b) * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for_n<kTN>([&](auto a_tag) {
            constexpr int a = decltype(a_tag)::value;
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[PAR][b], acc[a][b], 0, 0, 0);
            if constexpr (REFILL) af[a] = *reinterpret_cast<const v4i *>(nxt + (XB + a) * 1024);
            // the copies of the step three ahead go out one at a time between the matrix instructions
            // (bunched, they stall the wave at the compute unit's copy path)
            if constexpr (ISSUE && a < TM + 3)
                issue_one(std::integral_constant<int, a>{}, kt + kNS, st, std::integral_constant<bool, WHOLE && PAR == 1>{},
                          !(WHOLE && PAR == 1) || kt + kNS < KT);
            if constexpr (REFILL) __builtin_amdgcn_sched_barrier(0);
        });
        st = nst;
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    using WP = std::integral_constant<int, PMIN>;
    if constexpr (WHOLE) {
        for (int kt = 0; kt + 2 < KT; kt += 2) {
            step(I0{}, Yes{}, Yes{}, WP{}, kt);
            step(I1{}, Yes{}, Yes{}, WP{}, kt + 1);
        }
    } else if (KT >= 4) {
        int kt = 0;
        for (; kt + 4 < KT; kt += 2) {
            step(I0{}, Yes{}, Yes{}, WP{}, kt);
            step(I1{}, Yes{}, Yes{}, WP{}, kt + 1);
        }
        step(I0{}, Yes{}, Yes{}, WP{}, kt);           // kt = KT - 4: requests the last step
        step(I1{}, Yes{}, No{}, WP{}, kt + 1);
    }
    step(I0{}, Yes{}, No{}, I0{}, KT - 2);            // the last step's blocks: nothing younger is in flight
    step(I1{}, No{}, No{}, I0{}, KT - 1);

#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c2 = __builtin_readcyclecounter();
    const uint64_t clk_t2 = wall_clock64();
#endif
    // ---- epilogue: y = float(acc) * s_x[m] * s_w[n] + bias[n] -> bf16.  One token tile (16 tokens x
    // 144 channels) at a time is laid out in the wave's part of the idle ring and read back row by
    // row, so that a store instruction writes whole 288-byte row segments, 16 bytes per lane.
    // (Laying out the wave's whole 64 x 144 block first and storing three rows per instruction cost
    // registers in the k-loop and was slower; the store phase is bound by the memory write rate.)
    __syncthreads();                                  // every wave has read its last fragments
    const float *const par = reinterpret_cast<const float *>(smem + kParOff);
    constexpr int ROWB = kBN * 2 + 16;
    int8_t *const stg = smem + wave * (16 * ROWB);
    const int64_t m_wave = m0 + wave * (BM / 4);
    // The lane's channel scales and biases are read one channel tile ahead of their use: read where
    // they are used, every one of the 9 x TM reads waits out an LDS round trip with nothing else to issue.
    const float *const psw = par + kParSw / 4 + lg * 4, *const pbi = par + kParBias / 4 + lg * 4;
    float4 s_nxt = *reinterpret_cast<const float4 *>(psw), bi_nxt = *reinterpret_cast<const float4 *>(pbi);
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const float sxm = par[kParSx / 4 + wave * (BM / 4) + b * 16 + l16];
        int zc = 0;
        if constexpr (FORM == kRowsAsym) zc = reinterpret_cast<const int *>(par)[kParZc / 4 + wave * (BM / 4) + b * 16 + l16];
#pragma unroll
        for (int a = 0; a < kTN; ++a) {
            const float4 s = s_nxt, bi = bi_nxt;
            if constexpr (FORM == kRowsAsym) {
                if (a == 0) asm volatile("" ::: "memory");            // re-read per token tile: 36 registers if kept
                acc[a][b] += zc * *reinterpret_cast<const v4i *>(par + kParCs / 4 + a * 16 + lg * 4);
            }
            {
                const int an = (a + 1) % kTN;         // wraps to the first tile for the next token tile
                s_nxt = *reinterpret_cast<const float4 *>(psw + an * 16);
                bi_nxt = *reinterpret_cast<const float4 *>(pbi + an * 16);
            }
            if constexpr (DEBUG) {
                const int64_t m = m_wave + b * 16 + l16;
                *reinterpret_cast<int4 *>(g.acc_debug + m * g.N + n0 + a * 16 + lg * 4) =
                    make_int4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]);
            }
            uint2 o;
            o.x = pack_bf16x2((float)acc[a][b][0] * sxm * s.x + bi.x, (float)acc[a][b][1] * sxm * s.y + bi.y);
            o.y = pack_bf16x2((float)acc[a][b][2] * sxm * s.z + bi.z, (float)acc[a][b][3] * sxm * s.w + bi.w);
            *reinterpret_cast<uint2 *>(stg + l16 * ROWB + (a * 16 + lg * 4) * 2) = o;
        }
        __builtin_amdgcn_wave_barrier();
        constexpr int LPR = kBN / 8;
#pragma unroll
        for (int i = 0; i < (16 * LPR + 63) / 64; ++i) {
            const int id = i * 64 + lane;
            if (id < 16 * LPR) {
                const int row = id / LPR, c = id - row * LPR;
                const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * ROWB + c * 16);
                store_piece<kBN * 2, LINES>(g.Y + (m_wave + b * 16 + row) * g.ldy + n0, c, v);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
#ifdef TRDQ_PROBE_PHASES
    if (tid == 0 && g.acc_debug) {
        const uint64_t clk_c3 = __builtin_readcyclecounter();
        uint32_t hw, xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        uint64_t *o = reinterpret_cast<uint64_t *>(g.acc_debug) + (int64_t)blockIdx.x * 16;
        o[0] = clk_t0; o[1] = clk_t1; o[2] = clk_t2; o[3] = wall_clock64();
        o[4] = clk_c0; o[5] = clk_c1; o[6] = clk_c2; o[7] = clk_c3;
        o[8] = hw; o[9] = xcc; o[10] = BM; o[11] = 1;
    }
#endif
}

template <bool DEBUG, int FORM, int LINES>
__global__ __launch_bounds__(kThreads, 2) void qgemm8_tiled_kernel(GemmArgs g, int n_big, int nbn)
{
    extern __shared__ __align__(16) int8_t smem[];
    const int id = blockIdx.x;
    const int tiles_n = (g.N + kBN - 1) / kBN;        // kBlocks: whole tiles
    int tm, tn;
    if (id < n_big) {
        tile_map(id, (int)((g.M + 255) / 256), nbn, tm, tn);
        run_tile<256, DEBUG, FORM, LINES>(g, tm, tn, smem);
    } else {
        tile_map(id - n_big, (int)((g.M + 127) / 128), tiles_n - nbn, tm, tn);
        run_tile<128, DEBUG, FORM, LINES>(g, tm, tn + nbn, smem);
    }
}

// ---- one tile per compute unit: K split over two wave pairs --------------------------------------
// A launch with no more 128 x 144 tiles than compute units has nothing to put beside a tile, and a
// 128-token tile run by four waves as above means wave tiles of 32 x 144, whose fragment reads
// (0.6 KB per matrix instruction) bound the loop.  Here the four waves share the tile as two token
// halves x two halves of K: every wave keeps the 64 x 144 wave tile, each pair walks its half of
// the k-steps on a ring of its own (NS stages of 17 KB: 8 activation + 9 weight blocks), and all
// four meet at one barrier per k-step.  Such a tile pulls 17 KB through the compute unit's copy
// path per 72 matrix instructions, and that path delivers about 120 KB/us with nothing else going
// on (measured), so the loop runs at the rate of the copies and what counts is how many of them
// are in flight: two pairs x four stages keep three quarters of a 136 KB ring in flight (four
// pairs x two stages, eight waves, kept half of it and was 20 % slower; whether the blocks came
// from L2 or from behind it made no difference).
// At the end the two partial sums of each token sub-tile (16 tokens x 144 channels) meet in LDS,
// each pair adding up and finishing two of the four sub-tiles of both token halves.
// Needs K % 128 == 0 (the same number of k-steps for both pairs) and at least NS k-steps per pair;
// NS is 4, or 3 where the number of k-steps per pair is odd (the main loop takes two at a time).
constexpr int kKsStage = (8 + kTN) * 1024;
constexpr int kKsCopies = 9;                         // per wave and k-step
constexpr int kKsPairs = 2;
template <int NS> constexpr int ks_par_off() { return kKsPairs * NS * kKsStage; }
// The output, 9.4 MB at most, of block-tiled codes is stored non-temporally, all lines, that of row-major ones ordinarily.  us, none / all, pass
// and product on inputs of their own, and with a pass behind them that reads the output: block-tiled 1152 -> 1152 at 4096 tokens 17.4 / 16.5
// and 21.5 / 21.5, 4608 -> 1152 35.7 / 34.4 and 40.2 / 39.6, 2304 -> 1152 at 3072 21.0 / 20.2 and 24.1 / 24.1; row-major 1152 -> 2304 at 1900
// 16.4 / 16.3 and 21.3 / 23.3, 1152 -> 3456 at 1000 15.3 / 15.2 and 19.8 / 21.5, 4608 -> 1152 at 3000 34.5 / 33.8 and 38.8 / 39.6, at 4000
// 39.5 / 38.8 and 43.9 / 44.0; a block of width 1152 whose outputs are read at 1500 tokens, none / all, 112 / 113, at 4000 170 / 171.  Either by the
// size of the output: two kernels in a block, whose instructions are fetched in turn (1000 tokens 97.0, with one 95.6).
template <int FORM> constexpr int kKsLines = FORM == kBlocks ? kAllLines : kNoLines;
template <int NS> constexpr int ks_lds(bool asym) { return ks_par_off<NS>() + par_bytes(asym); }

template <int NS, bool DEBUG, int FORM>
__global__ __launch_bounds__(128 * kKsPairs) void qgemm8_tiled_ksplit_kernel(GemmArgs g)
{
    constexpr int NG = kKsPairs;
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int TM = 4;
    constexpr int P = kKsCopies;
    constexpr int RING = NS * kKsStage;
    constexpr int PAROFF = ks_par_off<NS>();
    static_assert((NS - 1) * P < 64, "vmcnt is a 6-bit counter");
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)smem;
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c0 = __builtin_readcyclecounter();
    const uint64_t clk_t0 = wall_clock64();
#endif
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mw = wave & 1, kg = wave >> 1;         // token half, part of K
    const int l16 = lane & 15, lg = lane >> 4;
    int tm, tn;
    tile_map(blockIdx.x, (int)((g.M + 127) / 128), (g.N + kBN - 1) / kBN, tm, tn);
    const int KT = g.K >> 6;                          // k-steps of the product
    const int KTg = KT / NG;                          // of one pair: even, at least NS
    const int64_t m0 = tile_m0(g, tm, 128);
    const int n0 = tile_n0<FORM>(g, tn);

    const int64_t gstride = (int64_t)KT * 1024;      // bytes from one 16-row group to the next
    const int64_t kofs = (int64_t)kg * KTg * 1024;   // this pair's first k-step
    constexpr int XSTEP = FORM == kBlocks ? 1024 : 64;  // bytes from one k-step of the activations to the next
    const int8_t *const xsrc = g.Xq + (m0 + mw * TM * 16) * g.K + (int64_t)kg * KTg * XSTEP;
    const int8_t *const wsrc = static_cast<const int8_t *>(g.Wc) + (int64_t)(n0 / 16) * gstride + kofs;
    const uint32_t voff = (uint32_t)(lane * 16);        // copies keep the block's order
    const uint32_t voffx = x_copy_off<FORM>(lane, g.K);
    int8_t *const ring = smem + kg * RING;
    const uint32_t ring0 = lds0 + kg * RING;

    // this wave's nine copies of a k-step: its own four activation blocks, and weight blocks 0..4
    // (first wave of the pair) or 5..8 and 8 once more (second wave: equal counts keep the waits uniform)
    const int8_t *src[P];
    uint32_t dst[P];
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        src[b] = xsrc + b * gstride;
        dst[b] = (uint32_t)((mw * TM + b) * 1024);
    }
#pragma unroll
    for (int i = 0; i < P - TM; ++i) {
        const int blk = mw == 0 ? i : (5 + i < kTN ? 5 + i : kTN - 1);
        src[TM + i] = wsrc + blk * gstride;
        dst[TM + i] = (uint32_t)((8 + blk) * 1024);
    }
    auto issue_one = [&](auto c_tag, int s, int st) {
        constexpr int c = decltype(c_tag)::value;
        if constexpr (c < TM) dma_1k(voffx, src[c] + (int64_t)s * XSTEP, ring0 + st * kKsStage + dst[c]);
        else dma_1k(voff, src[c] + (int64_t)s * 1024, ring0 + st * kKsStage + dst[c]);
    };
    auto issue = [&](int s, int st) {
        static_for_n<P>([&](auto c) { issue_one(c, s, st); });
    };

    // epilogue operands first (older than every tile copy, so the first wait covers them)
    {
        const uint32_t par = lds0 + PAROFF;
        const uint32_t v36 = (uint32_t)((lane < kBN / 4 ? lane : kBN / 4 - 1) * 16);
        const uint32_t vsx = (uint32_t)((lane < 128 / 4 ? lane : 128 / 4 - 1) * 16);
        copy_1k_if(wave == 0, v36, g.sw + n0, par + kParSw);
        copy_1k_if(wave == 1 && g.bias != nullptr, v36, g.bias ? g.bias + n0 : g.sw, par + kParBias);
        if (wave == 1 && g.bias == nullptr)
            *reinterpret_cast<uint4 *>(smem + PAROFF + kParBias + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (FORM == kBlocks) {
            copy_1k_if(wave == 2, vsx, g.sx + m0, par + kParSx);
        } else {
            copy_256_if(wave < 2, (uint32_t)(lane * 4), g.sx + m0 + mw * 64, par + kParSx + mw * 256);
            if constexpr (FORM == kRowsAsym) {
                copy_256_if(wave < 2, (uint32_t)(lane * 4), g.zc + m0 + mw * 64, par + kParZc + mw * 256);
                copy_1k_if(wave == 3, v36, g.colsum + n0, par + kParCs);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) issue(s, s);
    wait_vmcnt<(NS - 1) * P>();                       // step 0 and the operands above
    __syncthreads();
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c1 = __builtin_readcyclecounter();
    const uint64_t clk_t1 = wall_clock64();
#endif

    const int fro = blk_off(l16, lg), frox = x_frag_off<FORM>(l16, lg);
    v4i acc[kTN][TM];
#pragma unroll
    for (int a = 0; a < kTN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    v4i af[kTN], bf[2][TM];
#pragma unroll
    for (int a = 0; a < kTN; ++a) af[a] = *reinterpret_cast<const v4i *>(ring + (8 + a) * 1024 + fro);
#pragma unroll
    for (int b = 0; b < TM; ++b) bf[0][b] = *reinterpret_cast<const v4i *>(ring + (mw * TM + b) * 1024 + frox);

    int st = 0;
    // One k-step on activation fragment set PAR.  REFILL: the next step exists: wait until at most
    // WAITN younger copies are in flight (then it has landed), barrier, and read its fragments while
    // this step's matrix instructions run.  ISSUE: the step NS ahead exists and is requested into
    // this step's stage, whose fragments are all in registers by now.
    auto step = [&](auto par_tag, auto refill_tag, auto issue_tag, auto wait_tag, int kt) {
        constexpr int PAR = decltype(par_tag)::value;
        constexpr bool REFILL = decltype(refill_tag)::value;
        constexpr bool ISSUE = decltype(issue_tag)::value;
        constexpr int WAITN = decltype(wait_tag)::value;
        const int nst = (st + 1 == NS) ? 0 : st + 1;
        const int8_t *const nxt = ring + nst * kKsStage + fro;
        const int8_t *const nxtx = ring + nst * kKsStage + frox;
        if constexpr (REFILL) {
            wait_vmcnt<WAITN>();
            __syncthreads();
#pragma unroll
            for (int b = 0; b < TM; ++b)
                bf[1 - PAR][b] = *reinterpret_cast<const v4i *>(nxtx + (mw * TM + b) * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for_n<kTN>([&](auto a_tag) {
            constexpr int a = decltype(a_tag)::value;
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[PAR][b], acc[a][b], 0, 0, 0);
            if constexpr (REFILL) af[a] = *reinterpret_cast<const v4i *>(nxt + (8 + a) * 1024);
            if constexpr (ISSUE && a < P) issue_one(std::integral_constant<int, a>{}, kt + NS, st);
            if constexpr (REFILL) __builtin_amdgcn_sched_barrier(0);
        });
        st = nst;
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    using WFull = std::integral_constant<int, (NS - 2) * P>;
    int kt = 0;
    for (; kt + NS < KTg; kt += 2) {                  // KTg - NS is even (the launcher picks NS by the parity of KTg)
        step(I0{}, Yes{}, Yes{}, WFull{}, kt);
        step(I1{}, Yes{}, Yes{}, WFull{}, kt + 1);
    }
    // the last NS steps request nothing; step j of them leaves NS - 2 - j younger steps in flight
    static_for_n<NS>([&](auto j_tag) {
        constexpr int j = decltype(j_tag)::value;
        using Par = std::integral_constant<int, j & 1>;
        if constexpr (j + 1 < NS) step(Par{}, Yes{}, No{}, std::integral_constant<int, (NS - 2 - j) * P>{}, kt + j);
        else step(Par{}, No{}, No{}, I0{}, kt + j);
    });

#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c2 = __builtin_readcyclecounter();
    const uint64_t clk_t2 = wall_clock64();
#endif
    // ---- the partial sums of every token sub-tile meet in LDS ------------------------------------
    __syncthreads();                                  // every wave has read its last fragments
    v4i *const xch = reinterpret_cast<v4i *>(smem);
    constexpr int ROWB = kBN * 2 + 16;
    int8_t *stg;
    {
        // Pair q finishes sub-tiles 2q, 2q + 1: each wave lays down the two it does not finish
        // ([4 waves][2][9][64]) and adds what the other pair's wave of its token half left for it.
        {
            v4i *const out = xch + (wave * 2 * kTN) * 64 + lane;
#pragma unroll
            for (int a = 0; a < kTN; ++a) {
                out[a * 64] = kg == 0 ? acc[a][2] : acc[a][0];
                out[(kTN + a) * 64] = kg == 0 ? acc[a][3] : acc[a][1];
            }
        }
        __syncthreads();
        {
            const v4i *const in = xch + (((1 - kg) * 2 + mw) * 2 * kTN) * 64 + lane;
#pragma unroll
            for (int a = 0; a < kTN; ++a) {
                const v4i p0 = in[a * 64], p1 = in[(kTN + a) * 64];
                if (kg == 0) { acc[a][0] += p0; acc[a][1] += p1; }
                else { acc[a][2] += p0; acc[a][3] += p1; }
            }
        }
        stg = smem + 4 * 2 * kTN * 1024 + wave * (16 * ROWB);   // behind the exchange area
    }

    // ---- epilogue of this wave's sub-tiles: 16 tokens x all 144 channels each ---------------------
    const float *const par = reinterpret_cast<const float *>(smem + PAROFF);
    float4 sw_r[kTN], bi_r[kTN];                      // the lane's channel scales and biases, read once
#pragma unroll
    for (int a = 0; a < kTN; ++a) {
        sw_r[a] = *reinterpret_cast<const float4 *>(par + kParSw / 4 + a * 16 + lg * 4);
        bi_r[a] = *reinterpret_cast<const float4 *>(par + kParBias / 4 + a * 16 + lg * 4);
    }
    static_for_n<TM>([&](auto b_tag) {
        constexpr int b = decltype(b_tag)::value;
        if (b * NG / TM == kg) {                      // wave-uniform
            const int64_t m_own = m0 + mw * 64 + b * 16;
            const float sxm = par[kParSx / 4 + mw * 64 + b * 16 + l16];
            int zc = 0;
            if constexpr (FORM == kRowsAsym) zc = reinterpret_cast<const int *>(par)[kParZc / 4 + mw * 64 + b * 16 + l16];
#pragma unroll
            for (int a = 0; a < kTN; ++a) {
                const float4 s = sw_r[a];
                const float4 bi = bi_r[a];
                if constexpr (FORM == kRowsAsym)
                    acc[a][b] += zc * *reinterpret_cast<const v4i *>(par + kParCs / 4 + a * 16 + lg * 4);
                if constexpr (DEBUG) {
                    *reinterpret_cast<int4 *>(g.acc_debug + (m_own + l16) * g.N + n0 + a * 16 + lg * 4) =
                        make_int4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]);
                }
                uint2 o;
                o.x = pack_bf16x2((float)acc[a][b][0] * sxm * s.x + bi.x, (float)acc[a][b][1] * sxm * s.y + bi.y);
                o.y = pack_bf16x2((float)acc[a][b][2] * sxm * s.z + bi.z, (float)acc[a][b][3] * sxm * s.w + bi.w);
                *reinterpret_cast<uint2 *>(stg + l16 * ROWB + (a * 16 + lg * 4) * 2) = o;
            }
            __builtin_amdgcn_wave_barrier();
            constexpr int LPR = kBN / 8;
#pragma unroll
            for (int i = 0; i < (16 * LPR + 63) / 64; ++i) {
                const int id = i * 64 + lane;
                if (id < 16 * LPR) {
                    const int row = id / LPR, c = id - row * LPR;
                    const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * ROWB + c * 16);
                    store_piece<kBN * 2, kKsLines<FORM>>(g.Y + (m_own + row) * g.ldy + n0, c, v);
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    });
#ifdef TRDQ_PROBE_PHASES
    if (tid == 0 && g.acc_debug) {
        const uint64_t clk_c3 = __builtin_readcyclecounter();
        uint32_t hw, xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        uint64_t *o = reinterpret_cast<uint64_t *>(g.acc_debug) + (int64_t)blockIdx.x * 16;
        o[0] = clk_t0; o[1] = clk_t1; o[2] = clk_t2; o[3] = wall_clock64();
        o[4] = clk_c0; o[5] = clk_c1; o[6] = clk_c2; o[7] = clk_c3;
        o[8] = hw; o[9] = xcc; o[10] = 128; o[11] = 2;                 // 2: the K-split kernel
    }
#endif
}

// ---- int4 weights on block-tiled operands ---------------------------------------------------------
// Eq. 10's product with 4-bit weight codes and one scale per 128 input channels and output channel.
// Activations as above (1 KB blocks).  Weights: 16 * code, one byte each, in the 1 KB blocks of the int8 form (the packed codes,
// widened when the set is prepared: K * N more bytes per set), so that the operands are those of the int8 kernels; PACKED: the
// packed codes in blocks of 16 channels x 64 k (512 bytes): the 8 bytes that hold 16 consecutive k of a channel (byte j of a 4-byte
// word = code(k0 + j) | code(k0 + 4 + j) << 4) are the unit, unit (n, q = k / 16) at ((n / 16) * (K / 64) + q / 4) * 512 + (q % 4) * 128 +
// (n % 16) * 8, which a lane widens in registers (one shift-and-mask and one mask per word).  After the
// two k-steps of a scale group the int32 sums are folded into float accumulators with the group's scales; the factor 16 leaves
// with the token scale in the epilogue.
//
// 128 x 128 tiles, four waves as 2 x 2 (64 x 64 wave tiles: 64 + 64 accumulator registers), two
// workgroups per compute unit, a ring of four stages of 16.5 KB (8 activation blocks, 8 weight blocks, the
// group's 128 scales).  Per wave and k-step five copies: two activation blocks, two weight blocks, 256 bytes of scales
// (waves 2 and 3 copy the same scales as 0 and 1, and they travel with both k-steps of their group, so that every wave
// issues the same number of requests per step; past the last k-step the last one is copied again, for the same reason).
// The fold of group g is spread over the first k-step of group g + 1: channel tile by channel tile, the vector
// instructions of the tile's four sums in one run before the matrix instructions that start the next sums from zero.
// Packed (64-token tiles only): a ring of five stages of 8.5 KB, three copies per wave and k-step, and each sum's fold right before
// the matrix instruction that starts it again, under the ones before (in runs 1 to 10 % slower there).
//
// What bounds it is vector issue, two instructions per sum and group, and beyond 8192 tokens the power that sets the clock
// (1.73 GHz in the loop).  Widening in the loop cost 1.5 vector instructions per matrix instruction: with packed codes in LDS,
// and the folds between single matrix instructions, a workgroup's loop took 19100 cycles at K = 1152, now 17000.  us,
// before and after: 1152 -> 3456 at 4096 / 16384 tokens 26.8 / 88.6 -> 26.0 / 84.5, 1152 -> 4608 at 16384 115.4 -> 110.7, 4608 ->
// 1152 at 16384 106.1 -> 99.9, 768 -> 2304 at 2048 11.2 -> 10.2; 64-token tiles: see tiled4_rows_reads_wide.
constexpr int kW4BM = 128, kW4BN = 128;
constexpr int kW4XOff = 0;
constexpr int w4_stages(bool packed) { return packed ? 5 : 4; }
constexpr int kW4MinK = 384;                          // a k-step more than the ring has stages, whole groups
constexpr int w4_woff(int bm) { return bm * 64; }
constexpr int w4_soff(int bm, bool packed) { return bm * 64 + (packed ? 4096 : 8192); }
constexpr int w4_stage(int bm, bool packed) { return w4_soff(bm, packed) + 512; }
constexpr int w4_par_off(int bm, bool packed) { return w4_stages(packed) * w4_stage(bm, packed); }   // epilogue operands: [128 bias][pad][BM s_x]
constexpr int w4_lds(int bm, bool packed) { return w4_par_off(bm, packed) + 2048; }     // 69632 B; with 64 tokens 53248, packed 45568 B

template <int BM, bool DEBUG, int FORM, bool PACKED, int LINES>
__global__ __launch_bounds__(kThreads, BM == 64 ? 3 : 2) void qgemm4_tiled_kernel(GemmArgs g)
{
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int TM = BM / 32, TN = 4, NS = w4_stages(PACKED);
    constexpr int XC = BM / 64;                       // activation blocks a wave copies per k-step
    constexpr int WC = PACKED ? 1 : 2;                // weight copies: two blocks, in one copy or two
    constexpr int P = XC + WC + 1;                    // copies per wave and k-step
    constexpr int WBLOCK = PACKED ? 512 : 1024;       // bytes of a weight block, 16 channels x 64 k
    constexpr int kW4WOff = w4_woff(BM), kW4SOff = w4_soff(BM, PACKED), kW4Stage = w4_stage(BM, PACKED), kW4ParOff = w4_par_off(BM, PACKED);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)smem;
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c0 = __builtin_readcyclecounter();
    const uint64_t clk_t0 = wall_clock64();
#endif
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lg = lane >> 4;
    int tm, tn;
    tile_map(blockIdx.x, (int)((g.M + BM - 1) / BM), (g.N + kW4BN - 1) / kW4BN, tm, tn);
    const int KT = g.K >> 6;                          // k-steps: even, more than NS
    const int64_t m0 = tile_m0(g, tm, BM);
    const int n0 = tile_n0<FORM>(g, tn, kW4BN);

    const int64_t xstride = (int64_t)KT * 1024;      // bytes from one 16-token group to the next
    constexpr int XSTEP = FORM == kBlocks ? 1024 : 64;  // bytes from one k-step of the activations to the next
    const int8_t *const xsrc = g.Xq + (m0 + 16 * XC * wave) * g.K;
    const int64_t wstride = (int64_t)KT * WBLOCK;     // ... one 16-channel group to the next
    const int8_t *const wsrc = static_cast<const int8_t *>(g.Wc) + (int64_t)(n0 / 16 + 2 * wave) * wstride;
    const uint32_t voffx = x_copy_off<FORM>(lane, g.K);
    // a packed copy moves two blocks: lanes 0-31 the first, lanes 32-63 the one a channel group further
    const uint32_t voffw = PACKED ? (uint32_t)((lane & 31) * 16) + (lane >= 32 ? (uint32_t)wstride : 0u) : (uint32_t)(lane * 16);
    const float *const ssrc = g.sw + n0 + (wave & 1) * 64;
    const uint32_t voffs = (uint32_t)(lane * 4);
    auto issue_one = [&](auto c_tag, int s, int st) {
        constexpr int c = decltype(c_tag)::value;
        const uint32_t sbase = lds0 + st * kW4Stage;
        if constexpr (c < XC) dma_1k(voffx, xsrc + c * xstride + (int64_t)s * XSTEP, sbase + kW4XOff + (XC * wave + c) * 1024);
        else if constexpr (c < XC + WC) dma_1k(voffw, wsrc + (c - XC) * wstride + (int64_t)s * WBLOCK, sbase + kW4WOff + (WC * wave + c - XC) * 1024);
        else copy_256_if(1, voffs, ssrc + (int64_t)(s >> 1) * g.N, sbase + kW4SOff + (wave & 1) * 256);
    };
    auto issue = [&](int s, int st) {
        static_for_n<P>([&](auto c) { issue_one(c, s, st); });
    };

    // epilogue operands first: wave 0 the biases, wave 1 the token scales (half a copy each)
    {
        const uint32_t par = lds0 + kW4ParOff;
        const uint32_t v32 = (uint32_t)((lane & 31) * 16);
        copy_1k_if(wave == 0 && g.bias != nullptr, v32, g.bias ? g.bias + n0 : g.sw, par);
        if (wave == 0 && g.bias == nullptr)
            *reinterpret_cast<uint4 *>(smem + kW4ParOff + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (FORM == kBlocks) copy_1k_if(wave == 1, v32, g.sx + m0, par + 1024);
        else copy_256_if(wave < BM / 64, (uint32_t)(lane * 4), g.sx + m0 + wave * 64, par + 1024 + wave * 256);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) issue(s, s);
    wait_vmcnt<(NS - 1) * P>();
    __syncthreads();
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c1 = __builtin_readcyclecounter();
    const uint64_t clk_t1 = wall_clock64();
#endif

    const int xfr = kW4XOff + (wm * TM) * 1024 + (FORM == kBlocks ? lane * 16 : x_frag_off<FORM>(l16, lg));
    const int wfr = kW4WOff + (wn * TN) * WBLOCK + lane * (WBLOCK / 64);
    const int sfr = kW4SOff + (wn * 64 + lg * 4) * 4;
    auto widen = [](uint2 p) {
        return v4i{(int)((p.x << 4) & 0xF0F0F0F0u), (int)(p.x & 0xF0F0F0F0u), (int)((p.y << 4) & 0xF0F0F0F0u), (int)(p.y & 0xF0F0F0F0u)};
    };
    v4i acc[TN][TM];
    v4f facc[TN][TM];
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) { acc[a][b] = v4i{0, 0, 0, 0}; facc[a][b] = v4f{0.f, 0.f, 0.f, 0.f}; }
    v4i af[TN], bf[2][TM];
    uint2 raw[PACKED ? TN : 1];                       // the next k-step's codes, widened where the ones before are used up
    float4 sc[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) {
        if constexpr (PACKED) af[a] = widen(*reinterpret_cast<const uint2 *>(smem + wfr + a * WBLOCK));
        else af[a] = *reinterpret_cast<const v4i *>(smem + wfr + a * WBLOCK);
        sc[a] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int b = 0; b < TM; ++b) bf[0][b] = *reinterpret_cast<const v4i *>(smem + xfr + b * 1024);

    const int n_lane = n0 + wn * 64 + lg * 4;
    const int64_t m_lane0 = m0 + wm * (BM / 2) + l16;
    int st = 0;
    // One k-step.  HALF 0 starts the sums of a scale group (folding the group before, tile by tile, with
    // the scales read one group earlier) and ends by reading the new group's scales; HALF 1 continues the sums.
    auto step = [&](auto half_tag, auto fold_tag, auto next_tag, int kt) {
        constexpr int HALF = decltype(half_tag)::value;
        constexpr bool fold_prev = decltype(fold_tag)::value;     // a group before this one exists
        constexpr bool has_next = decltype(next_tag)::value;      // a k-step after this one exists
        const int nst = (st + 1 == NS) ? 0 : st + 1;
        const int8_t *const nxt = smem + nst * kW4Stage;
        wait_vmcnt<(NS - 2) * P>();
        __syncthreads();
        if constexpr (has_next) {
#pragma unroll
            for (int b = 0; b < TM; ++b) bf[1 - HALF][b] = *reinterpret_cast<const v4i *>(nxt + xfr + b * 1024);
            if constexpr (PACKED) {
#pragma unroll
                for (int a = 0; a < TN; ++a) raw[a] = *reinterpret_cast<const uint2 *>(nxt + wfr + a * WBLOCK);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for_n<TN>([&](auto a_tag) {
            constexpr int a = decltype(a_tag)::value;
            auto fold = [&](int b) {
                if constexpr (HALF == 0 && fold_prev) {
                    if constexpr (DEBUG) {
                        const int64_t m = m_lane0 + b * 16;
                        *reinterpret_cast<int4 *>(g.acc_debug + ((int64_t)((kt >> 1) - 1) * g.M + m) * g.N + n_lane + a * 16) =
                            make_int4(acc[a][b][0] >> 4, acc[a][b][1] >> 4, acc[a][b][2] >> 4, acc[a][b][3] >> 4);
                    }
                    facc[a][b][0] += sc[a].x * (float)acc[a][b][0];
                    facc[a][b][1] += sc[a].y * (float)acc[a][b][1];
                    facc[a][b][2] += sc[a].z * (float)acc[a][b][2];
                    facc[a][b][3] += sc[a].w * (float)acc[a][b][3];
                }
            };
            if constexpr (!PACKED) {
#pragma unroll
                for (int b = 0; b < TM; ++b) fold(b);
                if constexpr (HALF == 0) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int bb = 0; bb < TM; ++bb) {
                const int b = !PACKED && (a & 1) ? TM - 1 - bb : bb;
                if constexpr (PACKED) fold(b);
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[HALF][b], HALF == 0 ? v4i{0, 0, 0, 0} : acc[a][b], 0, 0, 0);
            }
            if constexpr (has_next && PACKED) af[a] = widen(raw[a]);
            else if constexpr (has_next) af[a] = *reinterpret_cast<const v4i *>(nxt + wfr + a * WBLOCK);
            if constexpr (a < P) issue_one(std::integral_constant<int, a>{}, kt + NS < KT ? kt + NS : KT - 1, st);
            if constexpr (a == TN - 1 && P > TN) issue_one(std::integral_constant<int, P - 1>{}, kt + NS < KT ? kt + NS : KT - 1, st);
            __builtin_amdgcn_sched_barrier(0);
        });
        // The group's scales, once the fold of the group before is done, from the NEXT step's stage (they
        // travel with both steps of the group): that stage is not given away before the next barrier,
        // this step's is being refilled by the other waves already.
        if constexpr (HALF == 0) {
#pragma unroll
            for (int a = 0; a < TN; ++a) sc[a] = *reinterpret_cast<const float4 *>(nxt + sfr + a * 64);
        }
        st = nst;
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    step(H0{}, No{}, Yes{}, 0);                       // at least three groups (the launcher checks)
    step(H1{}, No{}, Yes{}, 1);
    int kt = 2;
    for (; kt + 2 < KT; kt += 2) {
        step(H0{}, Yes{}, Yes{}, kt);
        step(H1{}, No{}, Yes{}, kt + 1);
    }
    step(H0{}, Yes{}, Yes{}, kt);
    step(H1{}, No{}, No{}, kt + 1);
    wait_vmcnt<0>();                                  // the repeated copies of the last steps
#ifdef TRDQ_PROBE_PHASES
    const uint64_t clk_c2 = __builtin_readcyclecounter();
    const uint64_t clk_t2 = wall_clock64();
#endif
    // the last group's fold
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            if constexpr (DEBUG) {
                const int64_t m = m_lane0 + b * 16;
                *reinterpret_cast<int4 *>(g.acc_debug + ((int64_t)((KT >> 1) - 1) * g.M + m) * g.N + n_lane + a * 16) =
                    make_int4(acc[a][b][0] >> 4, acc[a][b][1] >> 4, acc[a][b][2] >> 4, acc[a][b][3] >> 4);
            }
            facc[a][b][0] += sc[a].x * (float)acc[a][b][0];
            facc[a][b][1] += sc[a].y * (float)acc[a][b][1];
            facc[a][b][2] += sc[a].z * (float)acc[a][b][2];
            facc[a][b][3] += sc[a].w * (float)acc[a][b][3];
        }

    // ---- epilogue: y = (s_x / 16) * facc + bias -> bf16, one 16-token tile at a time through the idle ring
    __syncthreads();
    const float *const par = reinterpret_cast<const float *>(smem + kW4ParOff);
    constexpr int ROWB = 64 * 2 + 16;                 // a wave's 64 channels of one token, padded
    int8_t *const stg = smem + wave * (16 * ROWB);
    float4 bi_r[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) bi_r[a] = *reinterpret_cast<const float4 *>(par + wn * 64 + a * 16 + lg * 4);
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        const float sxm = par[256 + wm * (BM / 2) + b * 16 + l16] * 0.0625f;
#pragma unroll
        for (int a = 0; a < TN; ++a) {
            uint2 o;
            o.x = pack_bf16x2(sxm * facc[a][b][0] + bi_r[a].x, sxm * facc[a][b][1] + bi_r[a].y);
            o.y = pack_bf16x2(sxm * facc[a][b][2] + bi_r[a].z, sxm * facc[a][b][3] + bi_r[a].w);
            *reinterpret_cast<uint2 *>(stg + l16 * ROWB + (a * 16 + lg * 4) * 2) = o;
        }
        __builtin_amdgcn_wave_barrier();
        // 16 rows x 128 bytes = 128 pieces of 16 bytes: two per lane
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int id = i * 64 + lane;
            const int row = id >> 3, c = id & 7;
            const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * ROWB + c * 16);
            store_piece<128, LINES>(g.Y + (m0 + wm * (BM / 2) + b * 16 + row) * g.ldy + n0 + wn * 64, c, v);
        }
        __builtin_amdgcn_wave_barrier();
    }
#ifdef TRDQ_PROBE_PHASES
    if (tid == 0 && g.acc_debug) {
        const uint64_t clk_c3 = __builtin_readcyclecounter();
        uint32_t hw, xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        uint64_t *o = reinterpret_cast<uint64_t *>(g.acc_debug) + (int64_t)blockIdx.x * 16;
        o[0] = clk_t0; o[1] = clk_t1; o[2] = clk_t2; o[3] = wall_clock64();
        o[4] = clk_c0; o[5] = clk_c1; o[6] = clk_c2; o[7] = clk_c3;
        o[8] = hw; o[9] = xcc; o[10] = BM; o[11] = 4;                 // 4: the int4 kernel
    }
#endif
}

// ---- more than one round of 128 x 128 tiles: a workgroup walks a list of them --------------------
// The loop and the arithmetic of qgemm4_tiled_kernel.  With a workgroup per tile a slot of a compute unit stands 0.7 us without one
// between two tiles, and the new one waits 2 us for its first operands, of 14 us at K = 1152 (time stamps, 16384 tokens 1152 ->
// 4608).  Here the ring never drains: the last k-steps of a tile request the first ones of the next, which land under the
// epilogue; the output is laid out beside the ring, so that no barrier stands between two tiles.  Stages, copies and fragments as
// above.  What bounds it is the loop: without copies 3 % faster, without LDS reads or stores not at all, without folds 17 %.
// us, before and after: 1152 -> 1152 / 3456 / 4608 at 16384 tokens 33.3 / 86.9 / 110.9 -> 31.2 / 86.6 / 109.7, 4608 -> 1152 101.3 ->
// 98.0, 768 -> 3072 at 8192 29.1 -> 27.9, 384 -> 1536 at 32768 36.8 -> 33.7.  Up to one round it is the slower form: the next tile's
// place and the wait for its unused copies cost 0.6 us (4096 tokens 1152 -> 1152 14.1 -> 14.6, 384 -> 1152 7.6 -> 8.3).
// (The same for the int8 kernel, tall tiles: 2 to 6 % slower.  Its lists drift apart, and with them what a die's L2 shares.)
constexpr int kW4ListStage = 8192 + 8192 + 512;       // 8 activation blocks, 8 weight blocks, the group's 128 scales
constexpr int kW4ListStages = 4;
constexpr int kW4ListPar = kW4ListStages * kW4ListStage;          // [128 bias][pad][128 s_x][pad]
constexpr int kW4ListRow = 64 * 2 + 16;               // a wave's 64 channels of one token, padded
constexpr int kW4ListStg = kW4ListPar + 2048;
constexpr int kW4ListLds = kW4ListStg + 4 * 16 * kW4ListRow;      // 78848 B: two workgroups per compute unit

template <bool DEBUG, int LINES>
__global__ __launch_bounds__(kThreads, 2) void qgemm4_list_kernel(GemmArgs g, int stride)
{
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int TM = 4, TN = 4, NS = kW4ListStages;
    constexpr int P = 5;                              // copies per wave and k-step: two activation blocks, two weight blocks, scales
    constexpr int XOFF = 0, WOFF = 8192, SOFF = 16384;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)smem;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lg = lane >> 4;
    const int tiles_m = (int)(g.M / kW4BM), tiles_n = g.N / kW4BN, ntiles = tiles_m * tiles_n;
    const int KT = g.K >> 6;                          // k-steps: even, more than NS
    auto locate = [&](int id, int64_t &m, int &n) {
        int tm, tn, rows = tiles_m, cols = tiles_n;
        asm volatile("" : "+s"(rows), "+s"(cols));    // the map's divisors anew for every tile: kept, they take the sums' registers
        tile_map(id, rows, cols, tm, tn);
        m = (int64_t)__builtin_amdgcn_readfirstlane(tm) * kW4BM;
        n = __builtin_amdgcn_readfirstlane(tn) * kW4BN;
    };
    int id = blockIdx.x;
    int64_t m0, m1;                                   // first token and channel of this tile and of the next one
    int n0, n1;
    locate(id, m0, n0);

    // The copies run ahead of the products, over the end of a tile into the next one: where the next k-step to be copied
    // lies, and how many of its tile are left.
    const int64_t gstride = (int64_t)KT * 1024;       // bytes from one 16-row group to the next
    const int8_t *xp, *wp, *xnext, *wnext;                  // ... and the tile after it
    const float *sp, *snext;
    int left = KT;
    auto aim = [&](int64_t m, int n) {
        xnext = g.Xq + (m / 16 + 2 * wave) * gstride;
        wnext = static_cast<const int8_t *>(g.Wc) + (int64_t)(n / 16 + 2 * wave) * gstride;
        snext = g.sw + n + (wave & 1) * 64;
    };
    const uint32_t voff = (uint32_t)(lane * 16), voffs = (uint32_t)(lane * 4);
    auto copy = [&](auto c_tag, int stage) {          // stage: byte offset in the ring
        constexpr int c = decltype(c_tag)::value;
        const uint32_t to = lds0 + stage;
        if constexpr (c < 2) dma_1k(voff, xp + c * gstride, to + XOFF + (2 * wave + c) * 1024);
        else if constexpr (c < 4) dma_1k(voff, wp + (c - 2) * gstride, to + WOFF + (2 * wave + c - 2) * 1024);
        else copy_256_if(1, voffs, sp, to + SOFF + (wave & 1) * 256);
    };
    auto advance = [&]() {
        xp += 1024;
        wp += 1024;
        sp += (int64_t)(left & 1) * g.N;              // both steps of a group bring its scales
        // (selects that stay selects: with a branch in the step the compiler moves the folds behind it)
        asm("s_cmp_eq_u32 %3, 1\n\ts_cselect_b64 %0, %4, %0\n\ts_cselect_b64 %1, %5, %1\n\t"
            "s_cselect_b64 %2, %6, %2\n\ts_cselect_b32 %3, %7, %3\n\ts_sub_i32 %3, %3, 1"
            : "+&s"(xp), "+&s"(wp), "+&s"(sp), "+&s"(left) : "s"(xnext), "s"(wnext), "s"(snext), "s"(KT + 1) : "scc");
    };

    if (wave == 0 && g.bias == nullptr)               // no bias: zeros, so that the epilogue needs no branch
        *reinterpret_cast<uint4 *>(smem + kW4ListPar + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
    aim(m0, n0);
    xp = xnext;
    wp = wnext;
    sp = snext;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        static_for_n<P>([&](auto c) { copy(c, s * kW4ListStage); });
        advance();
    }
    wait_vmcnt<(NS - 1) * P>();
    __syncthreads();

    const int xfr = XOFF + wm * TM * 1024 + lane * 16;
    const int wfr = WOFF + wn * TN * 1024 + lane * 16;
    const int sfr = SOFF + (wn * 64 + lg * 4) * 4;
    v4i af[TN], bf[2][TM];
    float4 sc[TN];
#pragma unroll
    for (int a = 0; a < TN; ++a) {
        af[a] = *reinterpret_cast<const v4i *>(smem + wfr + a * 1024);
        sc[a] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int b = 0; b < TM; ++b) bf[0][b] = *reinterpret_cast<const v4i *>(smem + xfr + b * 1024);

    int st = 0;                                       // byte offset of this step's stage
    bool first = true;                                // no tile before: no stores among the requests
    for (;;) {
        const bool more = id + stride < ntiles;
        v4i acc[TN][TM];
        v4f facc[TN][TM];
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) facc[a][b] = v4f{0.f, 0.f, 0.f, 0.f};
        auto fold = [&](int a, int b, int group) {
            asm volatile("" : "+v"(acc[a][b]));       // folds stay where they are written: the compiler moves them into the step before
            if constexpr (DEBUG) {
                const int64_t m = m0 + wm * 64 + b * 16 + l16;
                *reinterpret_cast<int4 *>(g.acc_debug + ((int64_t)group * g.M + m) * g.N + n0 + wn * 64 + a * 16 + lg * 4) =
                    make_int4(acc[a][b][0] >> 4, acc[a][b][1] >> 4, acc[a][b][2] >> 4, acc[a][b][3] >> 4);
            }
            facc[a][b][0] += sc[a].x * (float)acc[a][b][0];
            facc[a][b][1] += sc[a].y * (float)acc[a][b][1];
            facc[a][b][2] += sc[a].z * (float)acc[a][b][2];
            facc[a][b][3] += sc[a].w * (float)acc[a][b][3];
        };
        // One k-step.  HALF 0 starts the sums of a scale group (folding the group before, tile by tile, with
        // the scales read one group earlier) and ends by reading the new group's scales; HALF 1 continues the sums.
        auto step = [&](auto half_tag, auto fold_tag, int kt) {
            constexpr int HALF = decltype(half_tag)::value;
            constexpr bool FOLD = decltype(fold_tag)::value;
            const int nst = st == (NS - 1) * kW4ListStage ? 0 : st + kW4ListStage;
            const int8_t *const nxt = smem + nst;
            // The next step's blocks have landed.  In a tile's first two steps the stores of the tile before are younger
            // than they are (requests retire in order).
            if (!FOLD && kt < 2 && !first) wait_vmcnt<(NS - 2) * P + 2 * TM>();
            else wait_vmcnt<(NS - 2) * P>();
            __syncthreads();
#pragma unroll
            for (int b = 0; b < TM; ++b) bf[1 - HALF][b] = *reinterpret_cast<const v4i *>(nxt + xfr + b * 1024);
            __builtin_amdgcn_sched_barrier(0);
            static_for_n<TN>([&](auto a_tag) {
                constexpr int a = decltype(a_tag)::value;
                if constexpr (FOLD) {
#pragma unroll
                    for (int b = 0; b < TM; ++b) fold(a, b, (kt >> 1) - 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int bb = 0; bb < TM; ++bb) {
                    const int b = a & 1 ? TM - 1 - bb : bb;
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[HALF][b], HALF == 0 ? v4i{0, 0, 0, 0} : acc[a][b], 0, 0, 0);
                }
                af[a] = *reinterpret_cast<const v4i *>(nxt + wfr + a * 1024);
                copy(a_tag, st);
                if constexpr (a == TN - 1) copy(std::integral_constant<int, P - 1>{}, st);
                __builtin_amdgcn_sched_barrier(0);
            });
            advance();
            // The group's scales, once the fold of the group before is done, from the NEXT step's stage (they
            // travel with both steps of the group): that stage is not given away before the next barrier,
            // this step's is being refilled by the other waves already.
            if constexpr (HALF == 0) {
#pragma unroll
                for (int a = 0; a < TN; ++a) sc[a] = *reinterpret_cast<const float4 *>(nxt + sfr + a * 64);
            }
            st = nst;
        };
        using H0 = std::integral_constant<int, 0>;
        using H1 = std::integral_constant<int, 1>;
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
        step(H0{}, No{}, 0);
        // Every wave is past the epilogue of the tile before: wave 0 requests this tile's biases, wave 1 its token scales
        // (half a copy each).  They are there long before the last of at least six k-steps.
        {
            const uint32_t v32 = (uint32_t)((lane & 31) * 16);
            copy_1k_if(wave == 0 && g.bias != nullptr, v32, g.bias ? g.bias + n0 : g.sw, lds0 + kW4ListPar);
            copy_1k_if(wave == 1, v32, g.sx + m0, lds0 + kW4ListPar + 1024);
        }
        locate(more ? id + stride : id, m1, n1);          // past the end: the last tile again, unused
        aim(m1, n1);
        step(H1{}, No{}, 1);
        int kt = 2;
        do {
            step(H0{}, Yes{}, kt);
            step(H1{}, No{}, kt + 1);
            kt += 2;
        } while (kt < KT);
        if (!more) wait_vmcnt<0>();                   // the unused copies: nobody may get their part of the LDS before
        // the last group's fold
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) fold(a, b, (KT >> 1) - 1);

        // ---- epilogue: y = (s_x / 16) * facc + bias -> bf16, one 16-token tile at a time through the wave's staging rows
        // (the lane index anew: kept over the loop, what follows from it takes the registers of the sums)
        int zero = 0;
        asm volatile("" : "+s"(zero));
        const int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (uint32_t)zero));
        const int l16_e = lane_e & 15, lg_e = lane_e >> 4;
        const float *const par = reinterpret_cast<const float *>(smem + kW4ListPar);
        int8_t *const stg = smem + kW4ListStg + wave * (16 * kW4ListRow);
        float4 bi_r[TN];
#pragma unroll
        for (int a = 0; a < TN; ++a) bi_r[a] = *reinterpret_cast<const float4 *>(par + wn * 64 + a * 16 + lg_e * 4);
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            const float sxm = par[256 + wm * 64 + b * 16 + l16_e] * 0.0625f;
#pragma unroll
            for (int a = 0; a < TN; ++a) {
                uint2 o;
                o.x = pack_bf16x2(sxm * facc[a][b][0] + bi_r[a].x, sxm * facc[a][b][1] + bi_r[a].y);
                o.y = pack_bf16x2(sxm * facc[a][b][2] + bi_r[a].z, sxm * facc[a][b][3] + bi_r[a].w);
                *reinterpret_cast<uint2 *>(stg + l16_e * kW4ListRow + (a * 16 + lg_e * 4) * 2) = o;
            }
            __builtin_amdgcn_wave_barrier();
            // 16 rows x 128 bytes = 128 pieces of 16 bytes: two per lane
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int q = i * 64 + lane_e;
                const int row = q >> 3, c = q & 7;
                const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * kW4ListRow + c * 16);
                store_piece<128, LINES>(g.Y + (m0 + wm * 64 + b * 16 + row) * g.ldy + n0 + wn * 64, c, v);
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (!more) break;
        id += stride;
        m0 = m1;
        n0 = n1;
        first = false;
    }
}

// 16 bytes per thread from the block form to the row-major form [M, K]
__global__ void untile_kernel(const int8_t *__restrict__ Xt, int8_t *__restrict__ Xq, int64_t M, int K)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int cpr = K >> 4;                           // 16-byte pieces per row
    if (idx >= M * cpr) return;
    const int64_t row = idx / cpr;
    const int c = (int)(idx - row * cpr);
    const int64_t t = ((row >> 4) * (K >> 6) + (c >> 2)) * 1024 + (c & 3) * 256 + (row & 15) * 16;
    *reinterpret_cast<uint4 *>(Xq + row * K + (int64_t)c * 16) = *reinterpret_cast<const uint4 *>(Xt + t);
}

}  // namespace

bool tiled_supports(const GemmArgs &a)
{
    return a.M > 0 && a.M % 128 == 0 && a.N % kBN == 0 && a.K % 128 == 0 && a.K >= 128 && a.ldy % 8 == 0 &&
           reinterpret_cast<uintptr_t>(a.Y) % 16 == 0 && !a.zc;
}

// How a launch splits the channel tiles between 256-token and 128-token workgroup tiles: the
// first nbn channel tiles go to tall tiles.  One round of two workgroups per compute unit if the
// short tiles alone would need more; all tall tiles when even those need more than one round.
void tiled_split(int64_t M, int N, int &n_big, int &nbn)
{
    const int T = (N + kBN - 1) / kBN;
    const int64_t slots = 2 * (int64_t)num_cus();
    const int64_t p128 = (M + 127) / 128, p256 = (M + 255) / 256;
    n_big = 0; nbn = 0;
    if (M < 256 || p128 * T <= slots) return;
    // tiles(nbn) = p256 * nbn + p128 * (T - nbn) <= slots
    const int64_t need = p128 > p256 ? (p128 * T - slots + (p128 - p256) - 1) / (p128 - p256) : T;
    nbn = (int)(need > T ? T : need);
    n_big = (int)(p256 * nbn);
}

// Which lines of its segments of 288 bytes a workgroup stores non-temporally (gemm_common.h).  A product alone gains 2 to 8 % by it nearly
// everywhere, but outputs are read, and then it gains nothing or loses.  So the choice is the one with which whole blocks do best whose every
// output is read by the next pass (four blocks with weights of their own, elementwise kernels between, buffers used again; us a block, no lines / all
// from 8 MB on / this rule and pipe144_lines): width 1152 at 4096 tokens 159 / 162 / 159, at 6144 225 / 221 / 222, at 32768 945 / 928 /
// 928; row-major codes at 3000 146 / 148 / 147, at 4096 161 / 164 / 162, width 768 at 6000 156 / 159 / 156, at 12000 251 / 255 / 250; with
// zero points at 8192 286 / 292 / 284, at 16384 531 / 545 / 529.  Of 35 such blocks those with all lines took 0.3 % longer than with
// none, at most 2.5 %, those with this rule 0.1 % less, at most 1.4 % longer.
// By size, us, none / all / whole lines, pass and product on inputs of their own, and the mean of three forms with a reader behind:
//   - below 8 MB none (256 -> 288 at 6000 / 9368 tokens, alone, 8.9 / 10.0 none, 9.1 / 10.3 all);
//   - to 20 MB all: 768 -> 1152 at 5120 17.3 / 15.6 / 16.7 and 22.9 / 21.8 / 22.3, 1152 -> 2304 at 2560 18.8 / 17.2 / 18.2 and 23.5 / 22.9 / 23.5;
//     from 16 MB on whole ones for fewer than 640 input channels (512 -> 2304 at 4096 16.4 / 16.1 / 15.6 and 24.1 / 24.8 / 23.9);
//   - to 64 MB none: 1152 -> 4608 at 4096 32.5 / 31.5 / 31.8 and 42.0 / 43.0 / 42.6, 768 -> 2304 at 8192 30.4 / 30.6 / 29.7 and 39.4 / 41.2 / 40.1;
//     for 1024 to 1151 input channels up to 128 MB (1024 -> 4608 at 8192 54.5 / 53.1 / 53.3 and 72.6 / 74.4 / 74.4), for fewer up to 192 MB
//     (896 -> 2304 at 16384 53.6 / 52.3 / 52.8 and 73.1 / 75.2 / 74.6);
//   - then all (1152 -> 3456 at 16384 82.3 / 77.2 / 80.7 and 111 / 110 / 111, 1024 -> 4608 96.5 / 90.7 / 95.6 and 141 / 138 / 139), for fewer
//     than 768 input channels whole ones (512 -> 4608 at 32768 128 / 135 / 126 and 213 / 225 / 208).
int tiled_lines(int64_t M, int K, int N)
{
    const int64_t mi = M * N >> 20;
    if (mi < 4) return kNoLines;
    if (mi < 10) return K < 640 && mi >= 8 ? kWholeLines : kAllLines;
    if (mi < (K >= 1152 ? 32 : K >= 1024 ? 64 : 96)) return kNoLines;
    return K >= 768 ? kAllLines : kWholeLines;
}

// The kernel that splits K inside the workgroup: two pairs, four stages for an even number of
// k-steps per pair and three for an odd one (the main loop takes the steps two at a time).
bool tiled_ksplit_applies(const GemmArgs &a)
{
    return a.K % 128 == 0 && a.K >= 1024 && ((a.M + 127) / 128) * (int64_t)((a.N + kBN - 1) / kBN) <= num_cus();
}

template <int NS, int FORM>
hipError_t launch_ksplit(const GemmArgs &a, bool debug, hipStream_t st)
{
    GemmArgs g = a;
    constexpr int lds = ks_lds<NS>(FORM == kRowsAsym);
    auto go = [&](auto kern) -> hipError_t {
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(((a.M + 127) / 128) * ((a.N + kBN - 1) / kBN))), dim3(256), lds, st, g);
        return hipGetLastError();
    };
#ifdef TRDQ_PROBE_PHASES
    debug = false;                                    // the debug pointer receives time stamps instead
#endif
    return debug ? go(qgemm8_tiled_ksplit_kernel<NS, true, FORM>) : go(qgemm8_tiled_ksplit_kernel<NS, false, FORM>);
}

template <int FORM>
hipError_t launch_form(const GemmArgs &a, bool debug, hipStream_t st)
{
    if (tiled_ksplit_applies(a)) return ((a.K / 128) & 1) ? launch_ksplit<3, FORM>(a, debug, st) : launch_ksplit<4, FORM>(a, debug, st);
    int n_big, nbn;
    tiled_split(a.M, a.N, n_big, nbn);
    const int64_t total = n_big + ((a.M + 127) / 128) * ((a.N + kBN - 1) / kBN - nbn);
    GemmArgs g = a;
    constexpr int lds = tiled_lds(FORM == kRowsAsym);
    auto go = [&](auto kern) -> hipError_t {
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), lds); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(kThreads), lds, st, g, n_big, nbn);
        return hipGetLastError();
    };
#ifdef TRDQ_PROBE_PHASES
    debug = false;                                    // the debug pointer receives time stamps instead
#endif
    if (debug) return go(qgemm8_tiled_kernel<true, FORM, kAllLines>);
    switch (tiled_lines(a.M, a.K, a.N)) {
        case kAllLines: return go(qgemm8_tiled_kernel<false, FORM, kAllLines>);
        case kWholeLines: return go(qgemm8_tiled_kernel<false, FORM, kWholeLines>);
        default: return go(qgemm8_tiled_kernel<false, FORM, kNoLines>);
    }
}

hipError_t launch_qgemm8_tiled(const GemmArgs &a, bool debug, hipStream_t st)
{
    return tiled_supports(a) ? launch_form<kBlocks>(a, debug, st) : hipErrorInvalidValue;
}

bool tiled_rows_supports(const GemmArgs &a)
{
    return a.M >= 128 && a.M <= (1 << 30) && a.N >= kBN && a.N % 16 == 0 && a.K % 128 == 0 && a.K >= 128 && a.ldy % 8 == 0 &&
           reinterpret_cast<uintptr_t>(a.Y) % 16 == 0 && !a.zcw && (!a.zc || a.colsum);
}

// Where this form is the faster one for row-major codes that the kernel for few tiles leaves (qgemm8_direct_tile < 0);
// both sides measured on ten shapes from 256 -> 512 to 4608 -> 1152 at 130 ... 32768 tokens.  Against the tiled form it
// costs 12 % from 4096 tokens on (1152 -> 3456: 21.2 against 18.7 us; its half-line copies), which puts it near
// the 128 x 144 and 256 x 256 kernels where tokens and channels are whole tiles; it wins where they are not, because the
// others leave the remainder to the any-shape kernel, a second launch (or the whole product, below 1024 tokens or with
// zero points), us, before and after: 1152 -> 3456 at 500 / 1500 / 5000 tokens 11.1 / 18.6 / 30.2 -> 8.4 / 12.6 / 26.3,
// 768 -> 3072 at 1000 tokens 9.6 -> 6.8, 4608 -> 1152 at 3000 tokens 29.3 -> 22.9.
//   - Remainder of tokens: up to where the second launch is a small part: 1100 tiles of 256 x 256 (1152 -> 4608 at 12000
//     tokens, 846 tiles: 82.1 -> 74.9, at 16000, 1134 tiles: 95.3 -> 98.3), and with a width of which the last tile
//     repeats a part 14000 tokens (1024 -> 2048 at 12000 34.6 -> 33.5, at 16000 39.7 -> 42.7).
//   - Whole tiles: up to three quarters of the compute units have one (1152 -> 3456 at 1024 tokens 9.9 -> 9.5, 768 -> 2304 at
//     1024 7.9 -> 6.8; 1152 -> 1152 at 4096, one each, 11.3 -> 11.6 with cold weights), for K < 1024 all of them, for long K
//     half (4608 -> 1152 at 1024 19.6 -> 17.8, at 4096 24.4 -> 25.0).  (Not at every shape: 2048 -> 2304 at 1280 / 1536 tokens
//     13.5 / 13.7 -> 13.9 / 14.1, -> 1152 at 2560 / 3072 12.7 / 13.1 -> 11.4 / 12.2.)  Below K = 512, where the width is whole 128-channel
//     tiles too, the 128 x 128 kernel is the other one and has no K to walk: only at nearly one tile each (256 -> 2304 at
//     512 / 1536 / 2048 tokens 4.5 / 5.4 / 6.3 -> 4.7 / 5.5 / 6.0; 128 -> 1152 at 1024 4.1 -> 4.5).  With zero points K < 1024
//     only (768 -> 2304 at 1024 8.0 -> 7.5, 1152 -> 3456 9.9 -> 10.6).
//     And from more than one to four tiles per compute unit, where a launch is one round of tall and short tiles, if every die
//     gets whole bands of tall ones (M % 2048; with 12 panels at 3072 tokens 1152 -> 3456 / 4608 22.0 / 22.6 -> 20.0 / 25.0), below K =
//     2304: 1152 -> 3456 / 4608 at 4096 tokens 22.3 / 27.8 -> 21.6 / 26.6, 1024 -> 2016 at 6144 20.2 -> 18.5, 640 -> 1296 at 8192 15.5 -> 14.0,
//     1152 -> 1152 at 8192 16.3 -> 16.2, 768 -> 2304 at 4096 12.9 -> 13.0 (2304 -> 2304 at 4096 24.3 -> 25.2).  But not where up to three
//     tiles per compute unit need more tall ones than there are compute units: one with two of them then has the work of four
//     tiles, while the 128 x 144 kernel has three (exactly three each: 768 -> 2304 at 6144 18.6 -> 20.5, 2048 -> 2304 32.6 -> 37.0,
//     1152 -> 1152 at 12288 21.5 -> 24.1).  And where all tiles are short ones (up to two each) only below K = 1792: 1280 -> 2448 at
//     2048 14.1 -> 13.2, 1536 -> 2016 at 4096 17.3 -> 16.8, 1792 -> 2448 at 2048 17.1 -> 17.9, 2176 -> 1152 at 8192 23.7 -> 24.5.
//   - Zero points: the only other kernel that takes them at any shape is the any-shape one (768 -> 3072 at 4096 tokens
//     23.2 -> 19.1, 1152 -> 4608 at 32700 tokens 268 -> 215).
bool tiled_rows_pays(int64_t M, int K, int N, bool asym)
{
    if (M < 128 || N < kBN) return false;
    const bool whole_n = N % kBN == 0;
    if (M % 128 == 0 && whole_n) {
        if (asym && K < 512) return true;
        if (asym && K >= 1024) return false;
        const int64_t tiles = (M / 128) * (int64_t)(N / kBN), cus = num_cus();
        if (K < 512 && N % 128 == 0) return K >= 256 && tiles > cus * 7 / 8 && tiles <= cus;
        if (!asym && K >= 512 && K < 2304 && M % 2048 == 0 && tiles > cus && tiles <= 4 * cus) {
            int n_big, nbn;
            tiled_split(M, N, n_big, nbn);
            return tiles <= 2 * cus ? K < 1792 : tiles > 3 * cus || n_big <= cus;
        }
        return tiles <= (K < 1024 ? cus : K < 2304 ? cus * 3 / 4 : cus / 2);
    }
    if (asym) return true;
    if (M % 128 == 0) return false;
    return whole_n ? ((M + 255) / 256) * ((N + 255) / 256) < 1100 : M < 14000;
}

hipError_t launch_qgemm8_tiled_rows(const GemmArgs &a, bool debug, hipStream_t st)
{
    if (!tiled_rows_supports(a)) return hipErrorInvalidValue;
    return a.zc ? launch_form<kRowsAsym>(a, debug, st) : launch_form<kRows>(a, debug, st);
}

bool tiled4_takes(int K, int N) { return K % 128 == 0 && K >= kW4MinK && N % 16 == 0 && N >= kW4BN; }

bool tiled4_supports(const GemmArgs &a)
{
    return a.M > 0 && a.M % kW4BM == 0 && a.N % kW4BN == 0 && tiled4_takes(a.K, a.N) && a.ldy % 8 == 0 &&
           reinterpret_cast<uintptr_t>(a.Y) % 16 == 0 && !a.zc;
}

namespace {

template <int BM, int FORM, bool PACKED>
hipError_t launch_w4(const GemmArgs &a, bool debug, hipStream_t st)
{
    GemmArgs g = a;
    auto go = [&](auto kern) -> hipError_t {
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), w4_lds(BM, PACKED)); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(((a.M + BM - 1) / BM) * ((a.N + kW4BN - 1) / kW4BN))), dim3(kThreads),
                           w4_lds(BM, PACKED), st, g);
        return hipGetLastError();
    };
#ifdef TRDQ_PROBE_PHASES
    debug = false;                                    // the debug pointer receives time stamps instead
#endif
    if (debug) return go(qgemm4_tiled_kernel<BM, true, FORM, PACKED, kNoLines>);
    return row_lines(a.Y, a.ldy) == kAllLines ? go(qgemm4_tiled_kernel<BM, false, FORM, PACKED, kAllLines>)
                                                   : go(qgemm4_tiled_kernel<BM, false, FORM, PACKED, kNoLines>);
}

}  // namespace

hipError_t launch_qgemm4_tiled(const GemmArgs &a, bool debug, hipStream_t st)
{
    if (!tiled4_supports(a)) return hipErrorInvalidValue;
    const int64_t tiles = (a.M / kW4BM) * (a.N / kW4BN), slots = 2 * (int64_t)num_cus();
#ifdef TRDQ_PROBE_PHASES
    if (debug && tiles > slots) return hipErrorInvalidValue;      // the kernel that takes them records no time stamps
#endif
    if (tiles <= slots || tiles > 0x3fffffff) return launch_w4<kW4BM, kBlocks, false>(a, debug, st);
    auto go = [&](auto kern) -> hipError_t {
        if (hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kern), kW4ListLds); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)slots), dim3(kThreads), kW4ListLds, st, a, (int)slots);
        return hipGetLastError();
    };
    if (debug) return go(qgemm4_list_kernel<true, kNoLines>);
    return row_lines(a.Y, a.ldy) == kAllLines ? go(qgemm4_list_kernel<false, kAllLines>) : go(qgemm4_list_kernel<false, kNoLines>);
}

bool tiled4_rows_supports(const GemmArgs &a)
{
    return a.M >= 64 && a.M <= (1 << 30) && tiled4_takes(a.K, a.N) && a.ldy % 8 == 0 && reinterpret_cast<uintptr_t>(a.Y) % 16 == 0 && !a.zc;
}

hipError_t launch_qgemm4_tiled_rows(const GemmArgs &a, bool debug, hipStream_t st)
{
    if (!tiled4_rows_supports(a)) return hipErrorInvalidValue;
    return tiled4_rows_reads_wide(a.M, a.N) ? launch_w4<64, kRows, false>(a, debug, st) : launch_w4<64, kRows, true>(a, debug, st);
}

// Where the 64-token tiles on row-major codes are the fastest int4 product: up to three workgroups per compute unit, one
// round (beyond, 128-token tiles read less per product: 1152 -> 1152 at 6000 tokens, 846 tiles, 18.0
// against 16.6 us).  With one 128 x 128 tile per compute unit and one wave per SIMD every k-step waits for its barrier,
// its LDS reads and its fold in turn; two or three workgroups of half the height fill those waits.  us, before and
// after: 1024 -> 2048 at 1232 / 2048 / 3000 tokens 10.5 / 10.6 / 15.2 -> 9.1 / 10.2 / 12.9, 1152 -> 4608 at 1000 16.0 -> 13.5,
// 4608 -> 1152 at 1000 31.0 -> 23.2, 768 -> 768 at 3000 9.2 -> 7.8.  Half-line copies of the activations cost
// nothing here, the product being bound by its vector instructions.
bool tiled4_rows_pays(int64_t M, int K, int N)
{
    return M >= 64 && tiled4_takes(K, N) && ((M + 63) / 64) * ((N + kW4BN - 1) / kW4BN) <= 3 * (int64_t)num_cus();
}

// Which copy of the codes they read.  Widened bytes spare a workgroup that shares its compute unit with at most one other the
// instructions, packed ones halve what a die's L2 brings in, which grows with the channel tiles that run side by side and with
// the rounds in which they do.  us, packed / widened: 4608 -> 1152 at 1344 tokens 23.4 / 19.7, at 3584 30.5 / 28.9, 1024 -> 2048 at 1280
// 9.0 / 8.2, 3072 -> 3072 at 512 16.8 / 14.3, 4608 -> 4608 at 320 22.8 / 20.0; but there at 448 23.3 / 24.4, at 1344 45 / 62, 1152 -> 4608
// at 576 9.9 / 11.9, 3072 -> 3072 at 1088 21.2 / 22.8, 1024 -> 2048 at 2048 9.9 / 10.9.  All linears of 24 blocks of width 1024 in turn,
// passes included, at 4096 tokens 2934 / 2824.  Sets that come from memory without a pass that reads them before: 4608 -> 1152 at
// 2304 29.7 / 25.9, 1024 -> 2048 at 1280 9.9 / 9.9, at 1600 10.2 / 10.5, 4608 -> 1152 at 3584 31.1 / 34.5.
bool tiled4_rows_reads_wide(int64_t M, int N)
{
    const int64_t tiles_n = (N + kW4BN - 1) / kW4BN, tiles = (M + 63) / 64 * tiles_n, cus = num_cus();
    return tiles <= 2 * cus && tiles * tiles_n <= 28 * cus;
}

hipError_t launch_untile(const int8_t *Xt, int8_t *Xq, int64_t M, int K, hipStream_t st)
{
    if (M <= 0) return hipSuccess;
    const int64_t n = M * (K / 16);
    hipLaunchKernelGGL(untile_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, Xt, Xq, M, K);
    return hipGetLastError();
}

}  // namespace gemm
}  // namespace trdq
