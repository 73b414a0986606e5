// fp32 matrix products on the bf16 matrix cores, for the fast static mode.
//
// An fp32 value is the sum of three bf16 values (8 significant bits each, rounded
// to nearest: hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid), exactly so from
// 2^-110 up to the largest bf16, 3.39e38. (Below, lo and mid are subnormal and lose
// what lies under 2^-133; above, hi is infinite and the product NaN, where the
// value's square is no fp32 value either.) A product a b is then the sum of nine
// bf16 products, each exact in fp32. Six are formed: the others (mid lo, lo mid, lo
// lo) are together at most 2^-26 of |a b|, a quarter of one fp32 rounding. Six
// v_mfma_f32_32x32x16_bf16 take 6/16 of the time of the fp32 MFMAs for the same
// product. Their sum over 16 k reaches the accumulator in one fp32 addition. Against
// 64 bits the entries of G G^T are off by 2.0e-8 to 2.3e-8 (rms, of sqrt(K_ii K_jj), B
// = 64 to 2048), on the fp32 MFMA by 5.1e-8 to 8.5e-8; what the fast mode makes of
// them is measured where its kernels are described.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mfac {
namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f8v __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int SPLIT_KC = 16;  // k per LDS chunk: one v_mfma_f32_32x32x16_bf16

// Row, within a 32 x 32 MFMA output tile, of accumulator register r of lane l
// (the column is l % 32).
__device__ __forceinline__ int mfma32x32_row(int lane, int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Three bf16 planes of a ROWS x 16 operand chunk; a row is two 8-value pieces
// (one MFMA lane's k values each), swapped in every other group of eight rows,
// so that 16 rows of one piece cover all 64 LDS banks.
template <int ROWS>
struct SplitChunk {
    bf8 v[3][ROWS * 2];
    static __device__ __forceinline__ int at(int row, int half) { return row * 2 + (half ^ ((row >> 3) & 1)); }
    // k 4 q .. 4 q + 3 of row `row`
    __device__ __forceinline__ void put4(int row, int q, float4 t) {
        typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
        typedef float f4 __attribute__((ext_vector_type(4)));
        f4 x = {t.x, t.y, t.z, t.w};
        const int e = at(row, q >> 1);
        const bf4 h = __builtin_convertvector(x, bf4);
        x -= __builtin_convertvector(h, f4);
        const bf4 m = __builtin_convertvector(x, bf4);
        x -= __builtin_convertvector(m, f4);
        reinterpret_cast<bf4*>(&v[0][e])[q & 1] = h;
        reinterpret_cast<bf4*>(&v[1][e])[q & 1] = m;
        reinterpret_cast<bf4*>(&v[2][e])[q & 1] = __builtin_convertvector(x, bf4);
    }
    // k 8 half .. 8 half + 7 of row `row`
    __device__ __forceinline__ void put8(int row, int half, f8v x) {
        const int e = at(row, half);
        const bf8 h = __builtin_convertvector(x, bf8);
        x -= __builtin_convertvector(h, f8v);
        const bf8 m = __builtin_convertvector(x, bf8);
        x -= __builtin_convertvector(m, f8v);
        v[0][e] = h;
        v[1][e] = m;
        v[2][e] = __builtin_convertvector(x, bf8);
    }
};

// acc[x][y] += a b^T over one chunk for this wave's NX x NY tiles of 32 x 32
// (rows ra + 32 x of a, rows rb + 32 y of b). ALL: every tile; else those whose
// bit x * NY + y of `on` is set (the same in every lane). The six products of a
// tile start from zero and are added to acc by the vector ALU: the bf16 MFMA cuts
// what lies below the last bits of a larger accumulator, and sums of 2048 squares
// come out low by 7e-7 to 1.2e-6 (mean over 64 of them). The same cut at the largest of
// a group's 16 products leaves entries of G G^T low by 5e-9 of sqrt(K_ii K_jj);
// negating every other group takes that away for 0.5% of the time and changed no
// error of the diagonal or an IHVP. One tile's additions run under the next tile's
// MFMAs (the scheduling barriers keep it at two tiles in flight, as many as the
// registers hold).
template <bool ALL, int NX, int NY, int RA, int RB>
__device__ __forceinline__ void split_mma(const SplitChunk<RA>& a, const SplitChunk<RB>& b, int ra, int rb, int lane,
                                          unsigned on, v16f (&acc)[NX][NY]) {
    const int rl = lane & 31, h = lane >> 5;
    const int ea = SplitChunk<RA>::at(ra + rl, h), eb = SplitChunk<RB>::at(rb + rl, h);
    bf8 av[3], bv[NY][3];
#pragma unroll
    for (int y = 0; y < NY; ++y)
#pragma unroll
        for (int p = 0; p < 3; ++p) bv[y][p] = b.v[p][eb + 64 * y];
    auto product = [&](int y) {
        constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};  // small products first
        v16f t = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 6; ++q)
            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[PA[q]], bv[y][PB[q]], t, 0, 0, 0);
        return t;
    };
    // acc += t here and not later: left alone, the compiler sinks the additions
    // below the next barrier and keeps every tile's t until then
    auto add = [](v16f& c, const v16f& t) {
        c += t;
        asm volatile("" : "+v"(c));
    };
    v16f prev;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
#pragma unroll
        for (int p = 0; p < 3; ++p) av[p] = a.v[p][ea + 64 * x];
#pragma unroll
        for (int y = 0; y < NY; ++y) {
            if constexpr (ALL) {
                const v16f t = product(y);
                if (x + y > 0) add(acc[y > 0 ? x : x - 1][y > 0 ? y - 1 : NY - 1], prev);
                prev = t;
                __builtin_amdgcn_sched_barrier(0);
            } else if ((on >> (x * NY + y)) & 1u) {
                add(acc[x][y], product(y));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if constexpr (ALL) add(acc[NX - 1][NY - 1], prev);
}

}  // namespace
}  // namespace mfac
