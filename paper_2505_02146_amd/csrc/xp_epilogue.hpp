// Epilogue shared by the MFMA kernels: C = alpha * acc + beta * C for one 32x32 accumulator block.
//
// Accumulator register v of lane l in a 32x32 MFMA block holds row (v/4)*8 + (l>>5)*4 + (v&3),
// column l&31, so one store instruction writes two 128-byte row segments.  Blocks that lie
// completely inside the matrix (the common case) take a branch-free path; beta == 0 never reads C.
#pragma once

#include <hip/hip_runtime.h>

namespace xp {

// The first element of every row of C on a multiple of `bytes`.  Stores that are to leave the L2 at once, non-temporal or
// written through, need rows on 64 bytes: otherwise each row segment ends inside a 64-byte piece of a line that is then written in
// two parts, each a memory access.  Measured, 48 batched 1000 x 1000 x 64 with rows on 32 bytes: written through 93 us, through the
// L2 51; 100 batched 381 x 381 x 64, rows on 4 bytes: non-temporal 33.7, through the L2 15.5.  On 64 bytes (1008 columns) both are even.
template <typename OutT> __device__ __forceinline__ bool rows_aligned(const OutT *C, long long ldc, int bytes)
{
    return (((unsigned long long)C | (unsigned long long)(ldc * (long long)sizeof(OutT))) & (unsigned long long)(bytes - 1)) == 0;
}

// STREAM = true marks the stores non-temporal: for outputs that are written once and not read again
// by the kernel (the store-bound batched shapes) they should not displace operand lines in the caches.
template <bool STREAM, typename T> __device__ __forceinline__ void put(T *dst, T v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, dst);
    else *dst = v;
}

template <bool INT8, bool STREAM = false, typename AccT, typename OutT>
__device__ __forceinline__ void store_block32(const AccT &acc, OutT *C, long long ldc, int blk_row0, int blk_col0,
                                              int lane, int M, int N, float alpha, float beta)
{
    const int col = blk_col0 + (lane & 31);
    const int row0 = blk_row0 + (lane >> 5) * 4;
    OutT *base = C + (long long)row0 * ldc + col;
    const bool interior = blk_row0 + 32 <= M && blk_col0 + 32 <= N;
    if constexpr (INT8) {
        if (interior) {
#pragma unroll
            for (int v = 0; v < 16; ++v) put<STREAM>(base + (long long)((v >> 2) * 8 + (v & 3)) * ldc, (OutT)acc[v]);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (v >> 2) * 8 + (v & 3);
                if (row0 + r < M && col < N) base[(long long)r * ldc] = acc[v];
            }
        }
    } else {
        if (beta == 0.0f) {
            if (interior) {
#pragma unroll
                for (int v = 0; v < 16; ++v) put<STREAM>(base + (long long)((v >> 2) * 8 + (v & 3)) * ldc, alpha * acc[v]);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = (v >> 2) * 8 + (v & 3);
                    if (row0 + r < M && col < N) base[(long long)r * ldc] = alpha * acc[v];
                }
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (v >> 2) * 8 + (v & 3);
                if (row0 + r < M && col < N) {
                    OutT *dst = base + (long long)r * ldc;
                    *dst = __builtin_fmaf(beta, *dst, alpha * acc[v]);
                }
            }
        }
    }
}

// 16x16 block computed transposed (B fragment as the first MFMA operand): accumulator register v
// of lane l holds C(row l&15, column 4*(l>>4) + v), i.e. 4 consecutive columns: one 16-byte store
// per lane wherever the four lie inside the matrix, at any 4-byte aligned address.  Rows off a 16-byte boundary are
// stored through the L2, non-temporal or not: their lines are written in parts, and parts that leave the L2 one by one
// cost a memory access each.  Measured with
// four 4-byte stores for such rows, as before, and with one 16-byte store: bf16 4095 x 4095 x 4096 133 -> 103 us, 96 batched
// 511 x 511 x 128 70 -> 38, convolution 32 x 28 x 28 x 256 -> 255 35 -> 31.
template <bool INT8, bool STREAM = false, typename AccT, typename OutT>
__device__ __forceinline__ void store_block16t(const AccT &acc, OutT *C, long long ldc, int blk_row0, int blk_col0,
                                               int lane, int M, int N, float alpha, float beta)
{
    const int row = blk_row0 + (lane & 15);
    const int col0 = blk_col0 + (lane >> 4) * 4;
    OutT *dst = C + (long long)row * ldc + col0;
    const bool interior = blk_row0 + 16 <= M && blk_col0 + 16 <= N;
    const bool aligned = rows_aligned(C, ldc, STREAM ? 64 : 16) && (blk_col0 & 3) == 0;
    typedef OutT out4 __attribute__((ext_vector_type(4)));
    typedef OutT out4_any __attribute__((ext_vector_type(4), aligned(4)));
    out4 x;
    if constexpr (INT8) x = out4{acc[0], acc[1], acc[2], acc[3]};
    else x = out4{alpha * acc[0], alpha * acc[1], alpha * acc[2], alpha * acc[3]};
    if (!INT8 && beta != 0.0f) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (row < M && col0 + v < N) dst[v] = __builtin_fmaf(beta, dst[v], x[v]);
    } else if (interior && aligned) {
        put<STREAM>((out4 *)dst, x);
    } else if (row < M) {
        if (col0 + 4 <= N) *(out4_any *)dst = x;
        else
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (col0 + v < N) dst[v] = x[v];
    }
}

// The same transposed 16x16 block into a planar output: row i (a pixel) of column j (a channel) lives at
// ((i / plane) * N + j) * plane + i % plane.  For each of a lane's four columns the 16 lanes l&15
// write 16 consecutive rows: one 64-byte run of a plane while the rows stay inside one image.
template <typename AccT, typename OutT>
__device__ __forceinline__ void store_block16t_planar(const AccT &acc, OutT *C, long long plane, int blk_row0, int blk_col0,
                                                      int lane, int M, int N, float alpha)
{
    const int row = blk_row0 + (lane & 15);
    const int col0 = blk_col0 + (lane >> 4) * 4;
    if (row >= M) return;
    // (rows and planes are below 2^31 here: a 32-bit division, a quarter of the instructions of a 64-bit one)
    const unsigned img = (unsigned)row / (unsigned)plane, pix = (unsigned)row - img * (unsigned)plane;
    OutT *dst = C + ((long long)img * N + col0) * plane + pix;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (col0 + v < N) dst[v * plane] = (OutT)(alpha * acc[v]);
}

}  // namespace xp
