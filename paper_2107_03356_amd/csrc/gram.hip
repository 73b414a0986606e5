// Gram matrices K = G G^T on the matrix cores (Section 3.2 initial setup:
// "evaluating G G^T in a straightforward fashion", O(d m^2); Section 3.1
// block-wise precompute, one m x m Gram per block).
//
// Tiling: one work-group (8 waves) per 128 x 128 lower-triangular output tile;
// each wave owns a 32 x 64 piece as 2 x 4 MFMA 16x16x4 tiles. Operands are
// staged through double-buffered LDS in 128 x 32 fp32 panels (row pitch 36
// floats: the 16-row x 4-k read pattern of one MFMA operand is conflict-free).
//
// Window Gram: fp64 MFMA (v_mfma_f64_16x16x4f64) on the fp32 window values
// (exact products, fp64 sums, as in the passes that keep K up to date). The
// column range of the window is split over work-groups and the split
// partials are summed in fp64, in a fixed order, by k_gram_reduce.
// Static blocks: fp64 MFMA (v_mfma_f64_16x16x4f64) over the block's columns
// in 128 x 128 tiles, written straight into the block's padded fp64 matrix
// with m*lambda added on the diagonal, because the keep-mask is decided in fp64.
// When a batch has too few tiles to fill the chip (few, wide blocks; B = d is
// the full-d precompute of Section 3.1) the block's columns are also split
// over work-groups and the fp64 partial tiles are summed in split order by
// k_gram_blocks_reduce.
// The fast static mode's k_gram_blocks32 runs the block Gram in fp32 on the bf16
// matrix cores (see there).
#include <type_traits>

#include "internal.h"
#include "split_mfma.h"
#include "tile_util.h"

namespace mfac {
namespace {

constexpr int KB = 32;     // columns per LDS stage
constexpr int PITCH = 36;  // LDS row pitch (floats)

__device__ __forceinline__ void tile_of(int idx, int& ti, int& tj) {
    int t = (int)((sqrtf(8.0f * (float)idx + 1.0f) - 1.0f) * 0.5f);
    while ((t + 1) * (t + 2) / 2 <= idx) ++t;
    while (t * (t + 1) / 2 > idx) --t;
    ti = t;
    tj = idx - t * (t + 1) / 2;
}

// Wave -> 32 x 64 piece of a 128 x 128 tile (fp64 kernels). Waves w and w + 4
// share a SIMD (round-robin placement): the pieces of a diagonal tile hold 0, 0,
// 3, 3, 7, 7, 8 and 8 parts of 16 x 16 that reach the diagonal, paired here as
// 8 + 0, 8 + 0, 7 + 3, 7 + 3.
__device__ __forceinline__ void lower_piece(int wave, int& wr, int& wc) {
    // (2,0) (3,0) (1,0) (3,1) | (0,1) (1,1) (0,0) (2,1), as 2 wr + wc
    const int code = (0x50317264 >> (4 * wave)) & 15;
    wr = code >> 1;
    wc = code & 1;
}

// The 2 x 4 parts (bit 4 x + y) of a diagonal tile's piece that reach the diagonal.
__device__ __forceinline__ unsigned lower_parts(int wr, int wc) {
    unsigned on = 0;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
            if (wr * 32 + x * 16 >= wc * 64 + y * 16) on |= 1u << (4 * x + y);
    return on;
}

// acc += A B^T over one KB-column chunk of fp32 operands, in fp64, for the parts
// in `on` (the same in every lane; ALL: every part). The caller keeps the two
// forms in loops of their own: one loop with both spills accumulators.
template <bool ALL>
__device__ __forceinline__ void gram_chunk(const float (*Ab)[PITCH], const float (*Bb)[PITCH], int wr, int wc, int lane,
                                           unsigned on, v4d (&acc)[2][4]) {
    const int rl = lane & 15, kl = lane >> 4;
    if constexpr (ALL) {
#pragma unroll
        for (int kk = 0; kk < KB / 4; ++kk) {
            double av[2], bv[4];
#pragma unroll
            for (int x = 0; x < 2; ++x) av[x] = (double)Ab[wr * 32 + x * 16 + rl][kk * 4 + kl];
#pragma unroll
            for (int y = 0; y < 4; ++y) bv[y] = (double)Bb[wc * 64 + y * 16 + rl][kk * 4 + kl];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[x][y], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                if ((on >> (4 * x + y)) & 1u) {
#pragma unroll
                    for (int kk = 0; kk < KB / 4; ++kk)
                        acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            (double)Ab[wr * 32 + x * 16 + rl][kk * 4 + kl],
                            (double)Bb[wc * 64 + y * 16 + rl][kk * 4 + kl], acc[x][y], 0, 0, 0);
                }
    }
}

// Window Gram partials. Grid (ntiles, nsplit): work-group (t, s) computes the
// 128 x 128 lower tile t of K over slabs [s*sps, min(nslab, (s+1)*sps)). Eight
// waves, each owning a 32 x 64 piece as 2 x 4 fp64 MFMA tiles (two waves per
// SIMD hide each other's LDS and memory waits), operands converted from fp32
// as they are read from LDS. The slab's rows stream through double-buffered
// LDS in 32-column chunks (128 x 32 fp32 per operand), the next chunk's global
// loads in flight during the MFMAs. Rows past m load clamped, in-bounds data;
// only rows and columns below m of the partial are ever summed into K.
constexpr int WT = 128;  // window Gram tile

// Two work-groups per CU (4 waves per SIMD).
__global__ __launch_bounds__(512, 4) void k_gram_window(const float* __restrict__ G, int m, int64_t nslab,
                                                     int64_t sps, double* __restrict__ part, int ntiles) {
    __shared__ float As[2][WT][PITCH];
    __shared__ float Bs[2][WT][PITCH];
    int ti, tj;
    tile_of(blockIdx.x, ti, tj);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int wr, wc;  // rows wr*32, columns wc*64
    lower_piece(wave, wr, wc);
    const int rl = lane & 15, kl = lane >> 4;
    // in a diagonal tile only the 16 x 16 parts that reach the diagonal are
    // formed (the reduction reads the lower triangle of such tiles); the waves
    // without any only stage operands
    const unsigned on = ti == tj ? lower_parts(wr, wc) : 255u;
    const int64_t s0 = (int64_t)blockIdx.y * sps;
    const int64_t s1 = min(s0 + sps, nslab);

    // staging: 128 rows x 32 columns per operand, 8 floats per thread and operand
    const int sr = tid >> 2, sc = (tid & 3) * 8;
    const int64_t offa = (int64_t)min(ti * WT + sr, m - 1) * SLAB + sc;
    const int64_t offb = (int64_t)min(tj * WT + sr, m - 1) * SLAB + sc;
    // staged chunk: two float4 per operand, kept in named registers
    float4 pa0, pa1, pb0, pb1;
#define MFAC_GW_LOAD(S_, K0_)                                            \
    {                                                                    \
        const float* base_ = G + (S_) * (int64_t)m * SLAB + (K0_);       \
        const float4* a_ = reinterpret_cast<const float4*>(base_ + offa); \
        const float4* b_ = reinterpret_cast<const float4*>(base_ + offb); \
        pa0 = a_[0];                                                     \
        pa1 = a_[1];                                                     \
        pb0 = b_[0];                                                     \
        pb1 = b_[1];                                                     \
    }
#define MFAC_GW_STORE(BUF_)                                              \
    {                                                                    \
        float4* a_ = reinterpret_cast<float4*>(&As[BUF_][sr][sc]);       \
        float4* b_ = reinterpret_cast<float4*>(&Bs[BUF_][sr][sc]);       \
        a_[0] = pa0;                                                     \
        a_[1] = pa1;                                                     \
        b_[0] = pb0;                                                     \
        b_[1] = pb1;                                                     \
    }

    v4d accd[2][4];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) accd[x][y] = v4d{0.0, 0.0, 0.0, 0.0};
    constexpr int NCH = SLAB / KB;  // chunks per slab
    if (s0 < s1) {
        MFAC_GW_LOAD(s0, 0)
        MFAC_GW_STORE(0)
        __syncthreads();
    }
    auto walk = [&](auto all) {
        int buf = 0;
        for (int64_t s = s0; s < s1; ++s) {
            for (int c = 0; c < NCH; ++c) {
                // next chunk: the following columns of this slab, or the next slab's first
                const bool more = c + 1 < NCH || s + 1 < s1;
                const int64_t sn = c + 1 < NCH ? s : s + 1;
                const int kn = c + 1 < NCH ? (c + 1) * KB : 0;
                if (more) MFAC_GW_LOAD(sn, kn)
                float (*Ab)[PITCH] = As[buf];
                float (*Bb)[PITCH] = Bs[buf];
                gram_chunk<decltype(all)::value>(Ab, Bb, wr, wc, lane, on, accd);
                if (more) MFAC_GW_STORE(buf ^ 1)
                __syncthreads();
                buf ^= 1;
            }
        }
    };
    if (ti == tj)
        walk(std::false_type{});
    else
        walk(std::true_type{});

    if (!on) return;
    double* out = part + ((int64_t)blockIdx.y * ntiles + blockIdx.x) * (WT * WT);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // fp64 MFMA result: lane l register r is row (l/16) + 4r
                const int row = wr * 32 + x * 16 + kl + 4 * r;
                const int col = wc * 64 + y * 16 + rl;
                out[row * WT + col] = accd[x][y][r];
            }
}

#undef MFAC_GW_LOAD
#undef MFAC_GW_STORE

// Sum over the splits of one element of the tile partials (src: split 0, `stride`
// doubles apart), in a fixed order, by TPE threads: 256 / TPE adjacent elements
// a work-group, thread t taking element t % (256 / TPE). Every thread calls it;
// the first 256 / TPE hold the result.
template <int TPE>
__device__ __forceinline__ double sum_splits(const double* __restrict__ src, int64_t stride, int nsplit, bool use) {
    constexpr int EL = 256 / TPE;
    const int el = threadIdx.x % EL, sg = threadIdx.x / EL;
    double s = 0.0;
    if (use)
        for (int k = sg; k < nsplit; k += 8 * TPE) {
            double q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = k + TPE * u < nsplit ? src[(int64_t)(k + TPE * u) * stride] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += q[u];
        }
    if constexpr (TPE > 1) {
        __shared__ double red[TPE][EL];
        red[sg][el] = s;
        __syncthreads();
        s = red[0][el];
#pragma unroll
        for (int u = 1; u < TPE; ++u) s += red[u][el];
    }
    return s;
}

// Whether one thread an element is enough to fill the chip: eight work-groups per
// CU and more. Otherwise (few tiles, whose splits are then many) eight threads share
// an element, each summing every eighth split: one thread walking all splits took
// 12.4 ms for a window's 3 tiles of 683 splits (one work-group per tile). One
// against eight threads, 512 blocks of m = 1024 in 2 splits: 1.2 against 6.0 ms;
// 64 in 8: 0.47 against 1.05; 32 in 16: 0.39 against 0.57; a window of m = 1024
// (2304 work-groups, 57 splits): no difference.
inline bool one_thread_sums(int64_t elements) { return elements >= 2048 * 256; }

// K[row][col] (both triangles) = sum over splits of the tile partials; a diagonal
// tile contributes its lower triangle (mirrored). Bound by reading the partials
// (~2048 tiles of 128 KB, whatever m is). Grid (ntiles, WT * WT * TPE / 256).
template <int TPE>
__global__ __launch_bounds__(256) void k_gram_reduce(const double* __restrict__ part, int nsplit,
                                                     int ntiles, int m, double* __restrict__ K) {
    constexpr int EL = 256 / TPE;
    int ti, tj;
    tile_of(blockIdx.x, ti, tj);
    const int e = blockIdx.y * EL + threadIdx.x % EL;
    const int rr = e / WT, cc = e % WT;
    const int row = ti * WT + rr, col = tj * WT + cc;
    // diagonal tiles: lower triangle (the rest of the partial is not written)
    const bool use = row < m && col < m && !(ti == tj && rr < cc);
    const double v = sum_splits<TPE>(part + (int64_t)blockIdx.x * (WT * WT) + e, (int64_t)ntiles * (WT * WT), nsplit, use);
    if (threadIdx.x < EL && use) {
        K[(int64_t)row * m + col] = v;
        K[(int64_t)col * m + row] = v;
    }
}

// Static blocks, fp64 MFMA. One work-group per 128 x 128 lower-triangular tile
// of one block's Gram matrix and column split (flattened over blocks, splits
// and tiles, XCD-remapped so the tiles of one block and split share an L2);
// the split's columns stream through double-buffered LDS in 32-column chunks,
// the next chunk's loads in flight during the MFMAs.
constexpr int GT = 128;

// Eight waves per 128 x 128 tile, each owning 32 x 64 as 2 x 4 MFMA tiles, and
// two work-groups per CU (4 waves per SIMD hide each other's LDS and memory
// waits). Staged chunk values live in named registers. nsplit == 1: the tile
// goes straight into A (plus mu on the diagonal; with accum, added to what A
// holds instead, no mu); otherwise split s of the block's columns
// [s*kcols, min(B, (s+1)*kcols)) writes its fp64 partial tile to
// part[(block*nsplit + s)*ntiles + tile].
__global__ __launch_bounds__(512, 4) void k_gram_blocks(const float* __restrict__ G, int m, int64_t d, int B,
                                                        int b0, int ntiles, int nsplit, int kcols, double mu,
                                                        int accum, double* __restrict__ A, int mp,
                                                        double* __restrict__ part) {
    __shared__ float As[2][GT][PITCH];
    __shared__ float Bs[2][GT][PITCH];
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int per_block = ntiles * nsplit;
    const int bl = lid / per_block;
    const int rem = lid - bl * per_block;
    const int sp = rem / ntiles;
    const int tile = rem - sp * ntiles;
    int ti, tj;
    tile_of(tile, ti, tj);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int wr, wc;  // rows wr*32, columns wc*64
    lower_piece(wave, wr, wc);
    const int rl = lane & 15, kl = lane >> 4;
    const bool diag_tile = ti == tj;
    // in a diagonal tile the part above the diagonal is never read (the
    // factorization uses the lower triangle): see k_gram_window
    const unsigned on = diag_tile ? lower_parts(wr, wc) : 255u;
    const int cbeg = sp * kcols;
    const int ncols = (B - cbeg) < kcols ? (B - cbeg) : kcols;
    const float* base = G + (int64_t)(b0 + bl) * B + cbeg;
    const int ra0 = ti * GT, rb0 = tj * GT;
    // staging: 128 rows x 32 columns per operand, 8 floats per thread and operand
    const int sr = tid >> 2, sc = (tid & 3) * 8;
    const bool oka = ra0 + sr < m, okb = rb0 + sr < m;
    // loads from clamped, in-bounds addresses (ncols is a positive multiple of
    // 4), the values outside the tile replaced by zeros in registers
    const float* rowa = base + (int64_t)min(ra0 + sr, m - 1) * d;
    const float* rowb = base + (int64_t)min(rb0 + sr, m - 1) * d;
    float4 pa0, pa1, pb0, pb1;
#define MFAC_GB_LOAD(K0_)                                                          \
    {                                                                                    \
        const int c_ = (K0_) + sc;                                                       \
        const int ca_ = min(c_, ncols - 4), cb_ = min(c_ + 4, ncols - 4);                \
        pa0 = *reinterpret_cast<const float4*>(rowa + ca_);                              \
        pa1 = *reinterpret_cast<const float4*>(rowa + cb_);                              \
        if (!diag_tile) {                                                                \
            pb0 = *reinterpret_cast<const float4*>(rowb + ca_);                          \
            pb1 = *reinterpret_cast<const float4*>(rowb + cb_);                          \
        }                                                                                \
    }
#define MFAC_GB_STORE(BUF_, K0_)                                                   \
    {                                                                                    \
        const int c_ = (K0_) + sc;                                                       \
        float4* a_ = reinterpret_cast<float4*>(&As[BUF_][sr][sc]);                       \
        a_[0] = keep4(oka && c_ < ncols, pa0);                                           \
        a_[1] = keep4(oka && c_ + 4 < ncols, pa1);                                       \
        if (!diag_tile) {                                                                \
            float4* b_ = reinterpret_cast<float4*>(&Bs[BUF_][sr][sc]);                   \
            b_[0] = keep4(okb && c_ < ncols, pb0);                                       \
            b_[1] = keep4(okb && c_ + 4 < ncols, pb1);                                   \
        }                                                                                \
    }

    v4d acc[2][4];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = v4d{0.0, 0.0, 0.0, 0.0};
    const int nchunk = (ncols + KB - 1) / KB;
    MFAC_GB_LOAD(0)
    MFAC_GB_STORE(0, 0)
    __syncthreads();
    auto walk = [&](auto all) {
        for (int c = 0; c < nchunk; ++c) {
            const int buf = c & 1;
            if (c + 1 < nchunk) MFAC_GB_LOAD((c + 1) * KB)
            gram_chunk<decltype(all)::value>(As[buf], diag_tile ? As[buf] : Bs[buf], wr, wc, lane, on, acc);
            if (c + 1 < nchunk) MFAC_GB_STORE(buf ^ 1, (c + 1) * KB)
            __syncthreads();
        }
    };
    if (diag_tile)
        walk(std::false_type{});
    else
        walk(std::true_type{});
#undef MFAC_GB_LOAD
#undef MFAC_GB_STORE
    if (!on) return;
    if (nsplit > 1) {
        double* out = part + ((int64_t)bl * nsplit + sp) * ntiles * (GT * GT) + (int64_t)tile * (GT * GT);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[(wr * 32 + x * 16 + kl + 4 * r) * GT + wc * 64 + y * 16 + rl] = acc[x][y][r];
        return;
    }
    double* Ab = A + (int64_t)bl * mp * mp;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // fp64 MFMA result: lane l register r is row (l/16) + 4r
                const int row = ra0 + wr * 32 + x * 16 + kl + 4 * r;
                const int col = rb0 + wc * 64 + y * 16 + rl;
                if (row < mp && col < mp) {
                    double v = acc[x][y][r];
                    if (accum)
                        v += Ab[(int64_t)row * mp + col];
                    else if (row == col)
                        v += (row < m) ? mu : 1.0;
                    Ab[(int64_t)row * mp + col] = v;
                }
            }
}

// A_b (lower triangle of every tile the factorization reads) = sum over the
// column splits of the partial tiles (TS x TS), in a fixed order, plus mu on the
// diagonal (identity on the padding rows); with accum, the sum is added to A_b
// instead. Summed as in k_gram_reduce: one wide block of m <= 128 rows is a single
// tile of up to 2048 splits, a batch of 512 blocks of 4096 columns in the fast
// mode is 5120 tiles of two. One thread an element takes four elements, 256 apart
// (1.5 -> 1.2 ms there). Grid (ntiles, nb, TS * TS / 1024), or TS * TS / 32 with eight threads.
template <typename OT, int TS, int TPE>
__global__ __launch_bounds__(256) void k_gram_blocks_reduce(const double* __restrict__ part, int nsplit, int ntiles,
                                                            int m, double mu, int accum, OT* __restrict__ A,
                                                            int mp) {
    constexpr int EL = 256 / TPE;
    const int tile = blockIdx.x, bl = blockIdx.y;
    int ti, tj;
    tile_of(tile, ti, tj);
    const int64_t sstride = (int64_t)ntiles * (TS * TS);
    const double* src = part + (int64_t)bl * nsplit * sstride + (int64_t)tile * (TS * TS);
#pragma unroll
    for (int q = 0; q < (TPE == 1 ? 4 : 1); ++q) {
        const int e = (TPE == 1 ? blockIdx.z * 4 + q : blockIdx.z) * EL + threadIdx.x % EL;
        const int rr = e / TS, cc = e % TS;
        const int row = ti * TS + rr, col = tj * TS + cc;
        const bool use = row < mp && col < mp && !(ti == tj && rr < cc);
        double v = sum_splits<TPE>(src + e, sstride, nsplit, use);
        if (threadIdx.x < EL && use) {
            OT* dst = A + (int64_t)bl * mp * mp + (int64_t)row * mp + col;
            if (accum)
                v += (double)*dst;
            else if (row == col)
                v += (row < m) ? mu : 1.0;
            *dst = (OT)v;
        }
    }
}

// Static blocks of the fast mode: fp32 products on the bf16 matrix cores
// (split_mfma.h), fp32 sums over at most SPLIT32 columns; wider blocks are split
// and the splits summed in fp64 (k_gram_blocks_reduce). One work-group per
// BM x BM lower tile and column split, waves of WM x WN, the columns in 16-wide
// chunks double-buffered in LDS, converted as they are staged, the next chunk's
// loads in flight during the MFMAs. 32 x 32 pieces wholly above the diagonal or
// past row m are skipped, and the waves of a diagonal 256-tile are placed so
// that the four SIMDs (waves go to them round-robin) hold 8, 8, 10 and 10 of its
// 36 pieces.
constexpr int SPLIT32 = 2048;

template <int BM, int WM, int WN>
__global__ __launch_bounds__((BM / WM) * (BM / WN) * 64, BM == 128 ? 4 : 2) void k_gram_blocks32(
    const float* __restrict__ G, int m, int64_t d, int B, int b0, int ntiles, int nsplit, int kcols, double mu,
    float* __restrict__ A, int mp, double* __restrict__ part) {
    constexpr int NX = WM / 32, NY = WN / 32, NT = (BM / WM) * (BM / WN) * 64;
    constexpr int RPT = BM * 4 / NT;  // rows (4 columns each) a thread stages per operand and chunk
    __shared__ SplitChunk<BM> As[2], Bs[2];
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int per_block = ntiles * nsplit;
    const int bl = lid / per_block;
    const int rem = lid - bl * per_block;
    const int sp = rem / ntiles;
    const int tile = rem - sp * ntiles;
    int ti, tj;
    tile_of(tile, ti, tj);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // wave -> piece (rows wr * WM, columns wc * WN)
    int wr, wc;
    if constexpr (BM == 256) {
        // waves w and w + 4 share a SIMD: (1,0)+(0,2), (1,1)+(0,3), (0,0)+(0,1), (1,2)+(1,3)
        const int code = (0x71326054 >> (4 * wave)) & 15;
        wr = code >> 2;
        wc = code & 3;
    } else {
        wr = wave / (BM / WN);
        wc = wave % (BM / WN);
    }
    const bool diag_tile = ti == tj;
    const int cbeg = sp * kcols;
    const int ncols = (B - cbeg) < kcols ? (B - cbeg) : kcols;
    const float* base = G + (int64_t)(b0 + bl) * B + cbeg;
    const int ra0 = ti * BM, rb0 = tj * BM;
    // this wave's 32 x 32 pieces that hold lower-triangle entries of rows below m
    unsigned on = 0;
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y) {
            const int r = ra0 + wr * WM + 32 * x, c = rb0 + wc * WN + 32 * y;
            if (r < m && c < m && r >= c) on |= 1u << (x * NY + y);
        }
    // staging: thread t moves 4 columns of rows t / 4 + i NT / 4 of each operand
    // (four lanes read one row's 64 bytes), from clamped, in-bounds addresses
    // (ncols is a positive multiple of 4); columns past ncols become zeros, rows
    // past m are dropped when A is written
    const int sr = tid >> 2, sq = tid & 3;
    const float* row[2 * RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        row[i] = base + (int64_t)min(ra0 + sr + i * (NT / 4), m - 1) * d;
        row[RPT + i] = base + (int64_t)min(rb0 + sr + i * (NT / 4), m - 1) * d;
    }
    float4 q[2 * RPT] = {};
    auto load = [&](int k0) {
        const int c = min(k0 + sq * 4, ncols - 4);
#pragma unroll
        for (int i = 0; i < RPT; ++i) q[i] = *reinterpret_cast<const float4*>(row[i] + c);
        if (!diag_tile) {
#pragma unroll
            for (int i = RPT; i < 2 * RPT; ++i) q[i] = *reinterpret_cast<const float4*>(row[i] + c);
        }
    };
    auto store = [&](int buf, int k0) {
        if (k0 + SPLIT_KC > ncols) {
#pragma unroll
            for (int i = 0; i < 2 * RPT; ++i) q[i] = keep4(k0 + sq * 4 < ncols, q[i]);
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) As[buf].put4(sr + i * (NT / 4), sq, q[i]);
        if (!diag_tile) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) Bs[buf].put4(sr + i * (NT / 4), sq, q[RPT + i]);
        }
    };

    v16f acc[NX][NY];
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
    load(0);
    store(0, 0);
    load(SPLIT_KC);
    __syncthreads();
    // Chunks k0 and k0 + 16 (zeros past ncols). The first half of the waves
    // converts the next chunk before its MFMAs, the other half after, so that of
    // the two waves on a SIMD one converts while the other multiplies; each
    // loads the chunk after that at once, a whole step ahead of its conversion.
    const bool early = wave < NT / 128;
    auto walk = [&](auto all) {
        auto step = [&](int buf, int k0) {
            if (early) {
                store(buf ^ 1, k0 + SPLIT_KC);
                load(k0 + 2 * SPLIT_KC);
            }
            split_mma<decltype(all)::value>(As[buf], diag_tile ? As[buf] : Bs[buf], wr * WM, wc * WN, lane, on, acc);
            if (!early) {
                store(buf ^ 1, k0 + SPLIT_KC);
                load(k0 + 2 * SPLIT_KC);
            }
            __syncthreads();
        };
        for (int k0 = 0; k0 < ncols; k0 += 2 * SPLIT_KC) {
            step(0, k0);
            step(1, k0 + SPLIT_KC);
        }
    };
    // the same for the whole work-group
    if (!diag_tile && ra0 + BM <= m)
        walk(std::true_type{});
    else
        walk(std::false_type{});
    double* out = part + (((int64_t)bl * nsplit + sp) * ntiles + tile) * (BM * BM);
    float* Ab = A + (int64_t)bl * mp * mp;
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int y = 0; y < NY; ++y) {
            if (ra0 + wr * WM + 32 * x < rb0 + wc * WN + 32 * y) continue;  // wholly above the diagonal
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = wr * WM + x * 32 + mfma32x32_row(lane, r), cc = wc * WN + y * 32 + (lane & 31);
                const int row = ra0 + rr, col = rb0 + cc;
                if (row >= mp || col >= mp) continue;
                const double v = row < m && col < m ? (double)acc[x][y][r] : 0.0;
                if (nsplit > 1)
                    out[rr * BM + cc] = v;
                else
                    Ab[(int64_t)row * mp + col] = (float)(row == col ? v + (row < m ? mu : 1.0) : v);
            }
        }
}

}  // namespace

namespace {
// splits of the slab range: enough work-groups for ~8 per CU
int64_t gram_window_splits(int m, int64_t nslab, int& ntiles) {
    const int T = (int)ceil_div(m, WT);
    ntiles = T * (T + 1) / 2;
    int64_t nsplit = ceil_div(2048, ntiles);
    if (nsplit > nslab) nsplit = nslab;
    if (nsplit < 1) nsplit = 1;
    const int64_t sps = ceil_div(nslab, nsplit);
    return ceil_div(nslab, sps);
}
}  // namespace

int64_t gram_window_part_doubles(int m, int64_t nslab) {
    int ntiles;
    const int64_t nsplit = gram_window_splits(m, nslab, ntiles);
    return nsplit * ntiles * (int64_t)(WT * WT);
}

hipError_t launch_gram_window(const float* G, int m, int64_t nslab, double* part, double* K,
                              hipStream_t st) {
    int ntiles;
    const int64_t nsplit = gram_window_splits(m, nslab, ntiles);
    const int64_t sps = ceil_div(nslab, nsplit);
    hipLaunchKernelGGL(k_gram_window, dim3(ntiles, (unsigned)nsplit), dim3(512), 0, st, G, m, nslab,
                       sps, part, ntiles);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (one_thread_sums((int64_t)ntiles * (WT * WT)))
        hipLaunchKernelGGL(k_gram_reduce<1>, dim3(ntiles, WT * WT / 256), dim3(256), 0, st, part, (int)nsplit, ntiles,
                           m, K);
    else
        hipLaunchKernelGGL(k_gram_reduce<8>, dim3(ntiles, WT * WT / 32), dim3(256), 0, st, part, (int)nsplit, ntiles,
                           m, K);
    return hipGetLastError();
}

namespace {
// Column splits of a batch of nb blocks: none when the batch has >= 1024
// tiles; otherwise up to 2048 work-groups (four rounds of the 512 that are
// resident at once, two per CU, without a nearly empty fifth), each split
// >= 2048 columns (its fp64 partial tile stays small next to the operand
// reads). kcols is a multiple of the 32-column stage, so every split starts
// 16-byte aligned.
int gram_blocks_splits(int nb, int mp, int B, int& ntiles, int& kcols) {
    const int T = (int)ceil_div(mp, GT);
    ntiles = T * (T + 1) / 2;
    const int64_t wgs = (int64_t)nb * ntiles;
    int64_t ns = 1;
    if (wgs < 1024) {
        ns = 2048 / wgs;
        const int64_t maxs = B / 2048;
        if (ns > maxs) ns = maxs;
        if (ns < 1) ns = 1;
    }
    kcols = (int)round_up(ceil_div(B, ns), KB);
    return (int)ceil_div(B, kcols);
}

// Tile edge of the fast mode's Gram: 256 (one work-group per CU, half the
// operand traffic), or 128 where 256-tiles would be mostly padding.
int gram32_tile(int mp) { return mp <= 128 ? 128 : 256; }

// Column splits of the fast mode's Gram: at most SPLIT32 columns each (fp32
// sums stay short), and more when a batch has fewer tiles than CUs (splits of
// at least SPLIT32 columns, up to ~1024 work-groups).
int gram32_splits(int nb, int mp, int B, int& ntiles, int& kcols) {
    const int T = (int)ceil_div(mp, gram32_tile(mp));
    ntiles = T * (T + 1) / 2;
    const int64_t wgs = (int64_t)nb * ntiles;
    int64_t ns = ceil_div(B, SPLIT32);
    if (wgs < 256) {
        int64_t fill = 1024 / wgs;
        if (fill > B / SPLIT32) fill = B / SPLIT32;
        if (fill > ns) ns = fill;
    }
    if (ns < 1) ns = 1;
    kcols = (int)round_up(ceil_div(B, ns), KB);
    return (int)ceil_div(B, kcols);
}
}  // namespace

int64_t gram_blocks32_part_doubles(int nb, int mp, int B) {
    int ntiles, kcols;
    const int ns = gram32_splits(nb, mp, B, ntiles, kcols), tile = gram32_tile(mp);
    return ns > 1 ? (int64_t)nb * ns * ntiles * (tile * tile) : 0;
}

int64_t gram_blocks_part_doubles(int nb, int mp, int B) {
    int ntiles, kcols;
    const int ns = gram_blocks_splits(nb, mp, B, ntiles, kcols);
    return ns > 1 ? (int64_t)nb * ns * ntiles * (GT * GT) : 0;
}

namespace {
template <typename OT, int TS>
hipError_t gram_blocks_reduce(const double* part, int ns, int ntiles, int nb, int m, double mu, int accum, OT* A, int mp,
                              hipStream_t st) {
    if (one_thread_sums((int64_t)nb * ntiles * (TS * TS)))
        hipLaunchKernelGGL((k_gram_blocks_reduce<OT, TS, 1>), dim3((unsigned)ntiles, (unsigned)nb, TS * TS / 1024),
                           dim3(256), 0, st, part, ns, ntiles, m, mu, accum, A, mp);
    else
        hipLaunchKernelGGL((k_gram_blocks_reduce<OT, TS, 8>), dim3((unsigned)ntiles, (unsigned)nb, TS * TS / 32),
                           dim3(256), 0, st, part, ns, ntiles, m, mu, accum, A, mp);
    return hipGetLastError();
}

template <int BM, int WM, int WN>
hipError_t gram_blocks32_tile(const float* G, int m, int64_t d, int B, int b0, int nb, double mu, float* A, int mp,
                              double* part, hipStream_t st) {
    int ntiles, kcols;
    const int ns = gram32_splits(nb, mp, B, ntiles, kcols);
    hipLaunchKernelGGL((k_gram_blocks32<BM, WM, WN>), dim3((unsigned)(ntiles * ns * nb)),
                       dim3((BM / WM) * (BM / WN) * 64), 0, st, G, m, d,
                       B, b0, ntiles, ns, kcols, mu, A, mp, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ns == 1) return e;
    return gram_blocks_reduce<float, BM>(part, ns, ntiles, nb, m, mu, 0, A, mp, st);
}
}  // namespace

hipError_t launch_gram_blocks32(const float* G, int m, int64_t d, int B, int b0, int nb, double mu, float* A,
                                int mp, double* part, hipStream_t st) {
    if (gram32_tile(mp) == 128) return gram_blocks32_tile<128, 32, 64>(G, m, d, B, b0, nb, mu, A, mp, part, st);
    return gram_blocks32_tile<256, 128, 64>(G, m, d, B, b0, nb, mu, A, mp, part, st);
}

hipError_t launch_gram_blocks(const float* G, int m, int64_t d, int B, int b0, int nb, double mu,
                              double* A, int mp, double* part, hipStream_t st, bool accumulate) {
    int ntiles, kcols;
    const int ns = gram_blocks_splits(nb, mp, B, ntiles, kcols);
    const int acc = accumulate ? 1 : 0;
    hipLaunchKernelGGL(k_gram_blocks, dim3((unsigned)(ntiles * ns * nb)), dim3(512), 0, st, G, m, d, B, b0, ntiles,
                       ns, kcols, mu, acc, A, mp, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ns == 1) return e;
    return gram_blocks_reduce<double, GT>(part, ns, ntiles, nb, m, mu, acc, A, mp, st);
}

}  // namespace mfac
