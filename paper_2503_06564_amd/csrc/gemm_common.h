// Shared pieces of the integer-product kernels: argument block, tile -> die mapping.
#pragma once

#include "device_utils.h"
#include "trdq_internal.h"

namespace trdq {
namespace gemm {

constexpr int kThreads = 256;

struct GemmArgs {
    const int8_t *Xq;      // [M, K]
    const void *Wc;        // codes, see Weights
    const float *sx;       // [M]
    const float *sw;       // [N] or [K/128, N]
    const float *bias;     // [N] or null
    uint16_t *Y;           // [M, ldy]
    int32_t *acc_debug;    // null, [M, N] or [K/128, M, N]
    // asymmetric activations: zc[i] = 128 - z_i per token, and with int8 weights the column sums of the
    // weight codes (the integer sum of a product is acc + zc[i] * colsum[n]), with int4 weights
    // colsumw[n] = 16 * sum_g s_w[g][n] * colsum_g[n] (the scaled term, added in float).  Null otherwise.
    const int32_t *zc = nullptr;
    const int32_t *colsum = nullptr;
    const float *colsumw = nullptr;
    // asymmetric weights: zcw[n] = 128 - z_w[n] and rowsum[i] = sum_k Xq[i][k] of the stored activation codes; the
    // integer sum of the product is acc + zc[i] colsum[n] + zcw[n] (rowsum[i] + K zc[i]).  Null otherwise.
    const int32_t *zcw = nullptr;
    const int32_t *rowsum = nullptr;
    int64_t M, ldy;
    int K, N;
    int tiles_m, tiles_n;
};

// Workgroups are handed to the 8 accelerator dies (XCDs) round-robin by their linear id; give
// each die a contiguous run of tiles so that the panels it re-reads stay in its own L2.
__device__ __forceinline__ int xcd_remap(int bid, int ntiles)
{
    const int q = ntiles >> 3, r = ntiles & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

// Work item id -> tile coordinates.  Each die owns a band of token panels; inside the band the
// tiles are visited in groups of up to 8 token panels, channel tile by channel tile, so the
// ~64 tiles a die has in flight form an 8 x 8 block: 8 activation panels + 8 weight panels fit
// its 4 MB L2, instead of every round streaming the whole weight matrix through it.
// (Needs tiles_m % 8 == 0; otherwise the plain run-per-die order is used.)
// Every die pulls what it touches through its own L2: with 8 bands that is the activations once
// and the weights 8 times.  When the weights are the larger part of that (few token panels, many
// channel tiles) the dies form a 4 x 2 grid instead -- 4 bands, each split between two dies by
// channel halves -- which fetches the activations twice and the weights 4 times.
__device__ __forceinline__ void tile_map(int id, int tiles_m, int tiles_n, int &tm, int &tn)
{
    if ((tiles_m & 7) == 0) {
        const int xcd = id & 7, i = id >> 3;         // i-th work item of this die
        const bool halves = (tiles_n & 1) == 0 && 8 * tiles_n > 3 * tiles_m;
        const int per = halves ? tiles_m >> 2 : tiles_m >> 3;     // token panels per die
        const int cols = halves ? tiles_n >> 1 : tiles_n;          // channel tiles per die
        const int gm = per < 8 ? per : 8;
        const int group = i / (gm * cols);
        const int j = i - group * gm * cols;
        const int rows = (per - group * gm) < gm ? (per - group * gm) : gm;   // last group may be short
        const int c = j / rows;
        tn = (halves ? (xcd >> 2) * cols : 0) + c;
        tm = (halves ? (xcd & 3) : xcd) * per + group * gm + (j - c * rows);
    } else {
        const int t = xcd_remap(id, tiles_m * tiles_n);
        tm = t / tiles_n;
        tn = t - tm * tiles_n;
    }
}

// ---- pieces shared by the direct-to-LDS kernels ---------------------------------------------------

// row -> XOR mask of the 16-byte chunk index, a function of (row mod 16) only so that the
// fragment offsets of different 16-row tiles differ by a constant.
//
// The LDS has 64 four-byte banks (256 B per clock).  A 128-bit read of a wavefront is served
// 16 lanes per clock, and (measured by swapping lane addresses in a conflict-free pattern) the
// lanes served together are the four-lane quads {0,3,5,6}, {1,2,4,7}, {9,10,12,15} and
// {8,11,13,14}.  With the matrix-instruction operand layout (lane = row + 16 * chunk) each of
// those sets holds every row once, rows 0-3 and 12-15 with one chunk of a pair and rows 4-11
// with the other.  The masks below send the 16 lanes of every set to 16 different 16-byte
// bank groups, for row strides of 64 B and 128 B.
template <int BK>
__device__ __forceinline__ int chunk_swizzle(int row)
{
    const int r = row & 15;
    if constexpr (BK == 64) return (r >> 3) << 1;
    else return (r & 2) | ((r >> 1) & 4);
}

__device__ __forceinline__ void dma_1k(uint32_t voff, const void *sbase, uint32_t lds_addr)
{
    // one wait state between the scalar write of M0 and the copy that reads it
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// ---- output rows -----------------------------------------------------------------------------------
// Stored non-temporally, the lines of an output leave a die's L2 while the product runs.  Kept there, up to 32 MB of them are
// written back when the kernel ends, and the next one starts behind that.  A line that two waves share costs memory two partial
// writes then, and whoever reads the output soon finds less of it in the caches.  So each kernel stores all, none or only the whole
// lines of its waves' row segments so, chosen where it is launched.
// Writing through instead (sc1) is slower than either (a block's four linears of width 1152 at 4096 tokens 119 ordinary / 113 / 125),
// and so are non-temporal codes of rotate_quant, in runs of 64 to 128 bytes (117).
enum { kNoLines = 0, kWholeLines = 1, kAllLines = 2 };

// Kernels whose waves store segments of whole lines (128 or 256 bytes): all if the rows of the output begin at lines, else none.
// us, ordinary / all, pass and product on inputs of their own, and with a pass behind them that reads the output.  Rows at lines: int4
// 1152 -> 4608 at 4096 tokens 39.9 / 36.9 and 48.2 / 47.7, at 16384 128 / 122 and 172 / 173, 1024 -> 2048 at 1232 14.1 / 13.5 and 17.5 /
// 17.2; int8 1152 -> 4608 at 16384 107 / 100 and 152 / 152, 512 -> 2064 at 32768 (rows of 2112) 77.1 / 67.4 and 134 / 122.  Rows of 16 bytes
// more, which share their lines: int4 384 -> 1536 at 16384 29.4 / 34.2 and 49.0 / 56.0, 1152 -> 4608 at 4096 41.5 / 40.8 and 52.9 / 55.1; int8
// 768 -> 3072 at 4096 24.8 / 25.8 and 34.8 / 38.5, 1152 -> 4608 at 16384 111 / 112 and 166 / 174, 512 -> 2064 at 32768 80.3 / 89.6 and
// 121 / 138.
inline int row_lines(const void *Y, int64_t ldy)
{
    return ldy % 64 == 0 && reinterpret_cast<uintptr_t>(Y) % 128 == 0 ? kAllLines : kNoLines;
}

// 16 bytes of an output row, non-temporal
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_out16(uint16_t *p, uint4 v)
{
    __builtin_nontemporal_store(u32x4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4_t *>(p));
}
// 16-byte piece c of a row segment of BYTES bytes (whole lines in assembly: the compiler joins two stores that differ by the hint
// only; a vector instruction may write the registers of a 16-byte store two wait states behind it, which the compiler sees to for
// its own stores only)
template <int BYTES, int LINES>
__device__ __forceinline__ void store_piece(uint16_t *seg, int c, uint4 v)
{
    uint16_t *const p = seg + c * 8;
    if constexpr (LINES == kAllLines) {
        store_out16(p, v);
    } else if constexpr (LINES == kWholeLines) {
        const uint32_t line = (uint32_t)(c * 16) - ((uint32_t)(uintptr_t)p & 127u);      // where the piece's line begins in the segment
        const u32x4_t w = {v.x, v.y, v.z, v.w};
        if (line <= (uint32_t)(BYTES - 128)) asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 1" :: "v"(p), "v"(w) : "memory");
        else *reinterpret_cast<u32x4_t *>(p) = w;
    } else {
        *reinterpret_cast<uint4 *>(p) = v;
    }
}

// Direct-to-LDS int8 kernels (qgemm_dma.hip).  variant indexes the table in that file.
int dma_num_variants();
hipError_t launch_qgemm8_dma(const GemmArgs &a, bool debug, int variant, hipStream_t st);
// the kernel for asymmetric activations (a.zc and a.colsum set): 128 x 128 ring kernel, any shape
hipError_t launch_qgemm8_asym(const GemmArgs &a, bool debug, int kind, hipStream_t st);

// int4-weight kernels on the same path (qgemm_dma.hip).
int dma4_num_variants();
hipError_t launch_qgemm4_dma(const GemmArgs &a, bool debug, int variant, hipStream_t st);

// Kernel on block-tiled operands (qgemm_tiled.hip): a.Xq and a.Wc point at the tiled forms.
bool tiled_supports(const GemmArgs &a);
hipError_t launch_qgemm8_tiled(const GemmArgs &a, bool debug, hipStream_t st);
// the same kernels on row-major activation codes, any M >= 128 and N >= 144; a.Wc points at the tiled form, a.zc / a.colsum
// (optional): asymmetric activations
bool tiled_rows_supports(const GemmArgs &a);
bool tiled_rows_pays(int64_t M, int K, int N, bool asym);
hipError_t launch_qgemm8_tiled_rows(const GemmArgs &a, bool debug, hipStream_t st);
hipError_t launch_untile(const int8_t *Xt, int8_t *Xq, int64_t M, int K, hipStream_t st);
// int4 weights on block-tiled operands (qgemm_tiled.hip): a.Wc holds the widened codes
bool tiled4_takes(int K, int N);                      // at some token count, with either tile
bool tiled4_supports(const GemmArgs &a);
hipError_t launch_qgemm4_tiled(const GemmArgs &a, bool debug, hipStream_t st);
// 64-token tiles on row-major activation codes, any M >= 64 and N >= 128; a.Wc holds the widened codes where
// tiled4_rows_reads_wide, the block form of the packed ones elsewhere
bool tiled4_rows_supports(const GemmArgs &a);
bool tiled4_rows_pays(int64_t M, int K, int N);
bool tiled4_rows_reads_wide(int64_t M, int N);
hipError_t launch_qgemm4_tiled_rows(const GemmArgs &a, bool debug, hipStream_t st);

// Small launches, weights straight into registers, activations through LDS areas of the waves' own (qgemm_direct.hip); tile
// indexes the table there.
// qgemm8_direct_tile: the tile for int8 weights where this form is the fastest, else -1.
int qgemm8_direct_tile(int64_t M, int K, int N, bool asym = false);
hipError_t launch_qgemm8_direct(const GemmArgs &a, bool debug, int tile, hipStream_t st);
// the same for int4 weights (a.Wc: the block form of the packed codes)
int qgemm4_direct_tile(int64_t M, int K, int N);
hipError_t launch_qgemm4_direct(const GemmArgs &a, bool debug, int tile, hipStream_t st);

// 256 x 256 tile kernel with a hand-scheduled main loop (qgemm_wide.hip).
bool wide_supports(const GemmArgs &a);
hipError_t launch_qgemm8_wide(const GemmArgs &a, bool debug, hipStream_t st);

}  // namespace gemm
}  // namespace trdq
