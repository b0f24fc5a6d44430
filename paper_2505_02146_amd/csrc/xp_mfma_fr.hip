// Few-rows MFMA kernel: C = X . W^T with at most 64 rows of X against a large matrix W, both contiguous along K -- a linear
// layer over the tokens of one decoding step (Table 5 of the paper: GEMM, GEMV-like cases).  bf16 or int8, any alignment.
//
// Bound: W is read once (16 x 8192 x 8192: 134 MB), so what counts is how fast a compute unit takes loads; the tiles of the
// other kernels are mostly padding here and wait for each K step at a barrier (57 us on that call).  A workgroup owns 8 to 40
// rows of W and all rows of X; its eight waves share out K, each loading its fragments of W and X straight into
// registers, D blocks of 128 bytes ahead, with no barrier before the end.  There the partial sums meet in LDS, in the order
// of the waves.
//
// A load that fetches 64 bytes of each of 16 rows, as a 16-row MFMA fragment wants it, costs a compute unit twice what one
// of eight whole 128-byte lines costs (16 x 8192 x 8192 34 us so).  Here a load is 8 rows x 128 bytes: lane 16g + a holds of row
// a >> 1 chunk 4 (a & 1) + g, that is, the 16 rows of the fragment are 8 rows x 2 halves of the block, for W and X alike.
// Of the 16 x 16 result the pairs of equal halves count, D[2r][2c] + D[2r + 1][2c + 1]; the matrix cores have the time.
#include "xp_internal.hpp"
#include "xp_any_align.hpp"
#include "xp_lds_tr.hpp"

#include <climits>
#include <type_traits>

namespace xp {
namespace {

constexpr int NW = 8;                     // waves per workgroup
constexpr int BLOCKB = 128;               // bytes of K per block
constexpr int ROWS_MAX = 64;              // rows of X

struct FrParams {
    const char *W, *X;
    char *C;
    int N, M, Kb;                         // rows of W, rows of X, K in bytes
    long long ldw_b, ldx_b, w_ext, x_ext; // pitches and extents in bytes
    long long cn, cm;                     // C(n, m) = C[n*cn + m*cm]
    long long strideW_b, strideX_b, strideC;
    float alpha, beta;
};

// WB: blocks of 8 rows of W, MB: of X.  STREAM: the loads of W are marked non-temporal.
template <bool INT8, int WB, int MB, bool STREAM>
__global__ __launch_bounds__(64 * NW) void fr_kernel(FrParams p)
{
    using KD = Kind<INT8>;
    constexpr int ESZ = KD::ESZ, EPC = 16 / ESZ;
    // blocks in flight, by registers: up to 16 rows of X two workgroups share a compute unit (27.5 -> 25.6 us at 16 x 8192 x 8192)
    constexpr int ROOM = ((MB <= 2 ? 118 : WB * MB >= 24 ? 214 : 190) - 4 * WB * MB) / (4 * (WB + MB)), D = ROOM > 8 ? 8 : ROOM;
    static_assert(D >= 1, "at least one block in flight");
    using OutT = typename KD::out_t;
    typedef typename KD::acc_t acc_t;
    __shared__ OutT red[NW][WB * MB][64];

    const int lane = threadIdx.x & 63, a = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * 8 * WB;
    const long long batch = blockIdx.y;
    const char *const X = p.X + batch * p.strideX_b;
    const char *const W = p.W + batch * p.strideW_b, *const W0 = W + (long long)n0 * p.ldw_b;

    // rows past the edge are the last row again; their results are not stored
    const int row = a >> 1, chunk = 16 * (4 * (a & 1) + g);
    unsigned wo[WB], xo[MB];
#pragma unroll
    for (int i = 0; i < WB; ++i) wo[i] = (unsigned)(min(8 * i + row, p.N - 1 - n0) * p.ldw_b) + chunk;
#pragma unroll
    for (int j = 0; j < MB; ++j) xo[j] = (unsigned)(min(8 * j + row, p.M - 1) * p.ldx_b) + chunk;

    acc_t acc[WB][MB];
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

    // the wave's blocks: a contiguous share of those inside K (the waves taking turns block by block: 34 us against 32)
    const int whole = p.Kb / BLOCKB;
    const int first = (int)((long long)whole * wave / NW), mine = (int)((long long)whole * (wave + 1) / NW) - first;
    u32x4 wf[D][WB], xf[D][MB];
    auto load = [&](int block, auto u) {
        const long long at = (long long)(first + block) * BLOCKB;
#pragma unroll
        for (int i = 0; i < WB; ++i) wf[u][i] = STREAM ? load16_stream(W0 + at + wo[i]) : load16(W0 + at + wo[i]);
#pragma unroll
        for (int j = 0; j < MB; ++j) xf[u][j] = load16(X + at + xo[j]);
    };
    auto multiply = [&](auto u) {
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[i][j] = KD::mma(wf[u][i], xf[u][j], acc[i][j]);
    };
    static_for<D>([&](auto u) {
        if (u < mine) load(u, u);
    });
    int i = 0;
    for (; i + 2 * D <= mine; i += D)                            // no condition inside: the waits count the loads of later blocks
        static_for<D>([&](auto u) {
            multiply(u);
            load(i + u + D, u);
        });
    for (; i < mine; i += D)
        static_for<D>([&](auto u) {
            if (i + u < mine) multiply(u);
            if (i + u + D < mine) load(i + u + D, u);
        });
    // the last, partial block: zeros past K, nothing read outside the operands
    if (p.Kb % BLOCKB != 0 && wave == NW - 1) {
        const int at = whole * BLOCKB, n = min(max((p.Kb - at - chunk) / ESZ, 0), EPC);
        const unsigned bits = (1u << n) - 1;
#pragma unroll
        for (int k = 0; k < WB; ++k) wf[0][k] = keep<ESZ>(load16_within(W, n > 0 ? (W0 - W) + wo[k] + at : 0, 0, p.w_ext), bits);
#pragma unroll
        for (int j = 0; j < MB; ++j) xf[0][j] = keep<ESZ>(load16_within(X, n > 0 ? (long long)xo[j] + at : 0, 0, p.x_ext), bits);
        multiply(std::integral_constant<int, 0>{});
    }

    // accumulator register v of lane l: row 4 * (l >> 4) + v of the fragment of W, row l & 15 of that of X.  An even lane
    // keeps the sum for row 2g of W, the odd one beside it that for row 2g + 1.
    const bool odd = (lane & 1) != 0;
#pragma unroll
    for (int k = 0; k < WB; ++k)
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const acc_t d = acc[k][j];
            const OutT s0 = odd ? d[1] : d[0], s1 = odd ? d[3] : d[2];
            const OutT t0 = s0 + __shfl_xor(s0, 1), t1 = s1 + __shfl_xor(s1, 1);
            red[wave][k * MB + j][lane] = odd ? t1 : t0;
        }
    __syncthreads();
    for (int blk = wave; blk < WB * MB; blk += NW) {
        OutT sum = red[0][blk][lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += red[w][blk][lane];
        const int n = n0 + 8 * (blk / MB) + 2 * g + (lane & 1), m = 8 * (blk % MB) + (a >> 1);
        if (n >= p.N || m >= p.M) continue;
        OutT *dst = (OutT *)p.C + batch * p.strideC + n * p.cn + m * p.cm;
        if constexpr (INT8) {
            *dst = sum;
        } else {
            sum *= p.alpha;
            *dst = p.beta != 0.0f ? __builtin_fmaf(p.beta, *dst, sum) : sum;
        }
    }
}

// ------------------------------------------------------------------------------------ host side

// X = A (few rows of C) or X = B (few columns of C, W = A)
bool fr_swapped(const Problem &q) { return q.M > ROWS_MAX || (q.N <= ROWS_MAX && q.N < q.M); }

template <bool INT8>
bool fr_can_run(const Problem &q)
{
    const int64_t esz = INT8 ? 1 : 2;
    if (q.in_type != (INT8 ? XP_I8 : XP_BF16) || q.conv || q.c_plane || q.K <= 0 || q.batch > 65535) return false;
    if (q.a_sk != 1 || q.b_sk != 1) return false;
    if ((fr_swapped(q) ? q.N : q.M) > ROWS_MAX || q.M > 0x3fffffffLL || q.N > 0x3fffffffLL || q.K > 0x3fffffffLL) return false;
    if (((q.M - 1) * q.a_sm + q.K) * esz < 16 || ((q.N - 1) * q.b_sn + q.K) * esz < 16) return false;      // operands of at least one chunk
    // 32-bit offsets of the rows of a workgroup
    return 64 * q.a_sm * esz + q.K * esz < 0x7fffffffLL && 64 * q.b_sn * esz + q.K * esz < 0x7fffffffLL;
}

template <bool INT8, int WB>
hipError_t fr_launch_rows(const FrParams &p, int64_t batch, hipStream_t stream)
{
    const dim3 grid((unsigned)((p.N + 8 * WB - 1) / (8 * WB)), (unsigned)batch);
    // A W that is a quarter of the 256 MB last-level cache or more is marked as streamed: it would not be there the next time
    // anyhow (16 x 8192 x 8192, four matrices in turn: 27.4 -> 25.6 us; a 34 MB one that still is there: 13.0 -> 17.7).
    const bool stream_w = (long long)p.N * p.Kb * batch >= (64LL << 20);
#define XP_FR(MB)                                                                                                  \
    do {                                                                                                           \
        if (stream_w) hipLaunchKernelGGL((fr_kernel<INT8, WB, MB, true>), grid, dim3(64 * NW), 0, stream, p);      \
        else hipLaunchKernelGGL((fr_kernel<INT8, WB, MB, false>), grid, dim3(64 * NW), 0, stream, p);              \
    } while (0)
    if constexpr (WB != 3 && WB != 5) {                          // (see fr_w_blocks)
        if (p.M <= 8) { XP_FR(1); return hipGetLastError(); }
        if (p.M <= 16) { XP_FR(2); return hipGetLastError(); }
    }
    if (p.M <= 24) XP_FR(3);
    else if (p.M <= 32) XP_FR(4);
    else if (p.M <= 48) XP_FR(6);
    else if constexpr (WB <= 4) XP_FR(8);
#undef XP_FR
    return hipGetLastError();
}

// Rows of X as the kernel loads them
int fr_rows(int64_t m) { return m <= 8 ? 8 : m <= 16 ? 16 : m <= 24 ? 24 : m <= 32 ? 32 : m <= 48 ? 48 : 64; }

// Blocks of 8 rows of W per workgroup.  The more, the less often X is read, but every compute unit should have a workgroup, and
// two where they fit (up to 16 rows of X: 32-row workgroups 29.0 us at 16 x 8192 x 8192, 16-row ones 27.4; 8 x 14336 x 4096 27
// and 20).  Above 16 rows of X a compute unit holds one workgroup, and a last round of a few costs as much as a whole one: the fullest
// compute unit's loads of W and X decide (with 32 rows, 42 x 9266 x 11712 would be 290 workgroups; 40 make it 232: 48 us, 80 on
// the 64-row tile; 20 x 10240 x 5120 32 -> 21, 48 x 5435 x 5000 30 -> 19, 32 x 11008 x 4096 30 -> 25).
int fr_w_blocks(int64_t n, int64_t m, int64_t batch)
{
    if (m <= 16) {
        if ((n + 31) / 32 * batch >= 512) return 4;
        return (n + 15) / 16 * batch >= 256 ? 2 : 1;
    }
    int best = 1;
    int64_t least = LLONG_MAX;
    for (int wb = 1; wb <= (m > 48 ? 4 : 5); ++wb) {
        const int64_t loads = ((n + 8 * wb - 1) / (8 * wb) * batch + 255) / 256 * (8 * wb + fr_rows(m));
        if (loads < least) { least = loads; best = wb; }
    }
    return best;
}

template <bool INT8>
hipError_t fr_launch(const Problem &q)
{
    const int64_t esz = INT8 ? 1 : 2;
    FrParams p;
    const bool sw = fr_swapped(q);
    p.W = (const char *)(sw ? q.A : q.B); p.X = (const char *)(sw ? q.B : q.A); p.C = (char *)q.C;
    p.N = (int)(sw ? q.M : q.N); p.M = (int)(sw ? q.N : q.M); p.Kb = (int)(q.K * esz);
    p.ldw_b = (sw ? q.a_sm : q.b_sn) * esz; p.ldx_b = (sw ? q.b_sn : q.a_sm) * esz;
    p.w_ext = (p.N - 1) * p.ldw_b + p.Kb; p.x_ext = (p.M - 1) * p.ldx_b + p.Kb;
    p.cn = sw ? q.ldc : 1; p.cm = sw ? 1 : q.ldc;
    p.strideW_b = (sw ? q.strideA : q.strideB) * esz; p.strideX_b = (sw ? q.strideB : q.strideA) * esz; p.strideC = q.strideC;
    p.alpha = q.alpha; p.beta = q.beta;
    const int wb = fr_w_blocks(p.N, p.M, q.batch);
    if (wb == 5) return fr_launch_rows<INT8, 5>(p, q.batch, q.stream);
    if (wb == 4) return fr_launch_rows<INT8, 4>(p, q.batch, q.stream);
    if (wb == 3) return fr_launch_rows<INT8, 3>(p, q.batch, q.stream);
    if (wb == 2) return fr_launch_rows<INT8, 2>(p, q.batch, q.stream);
    return fr_launch_rows<INT8, 1>(p, q.batch, q.stream);
}

bool fr_aligned(const Problem &q)
{
    const int64_t epc = 16 / elem_size(q.in_type);
    return (((uintptr_t)q.A | (uintptr_t)q.B) & 15) == 0 && q.a_sm % epc == 0 && q.b_sn % epc == 0 && q.K % epc == 0 &&
           q.strideA % epc == 0 && q.strideB % epc == 0;
}

// Chosen by few_rows_preferred, ahead of the table and the estimates: a call that it declines goes to another kernel.
double fr_cost(const Problem &) { return 1e30; }

const Variant kBfFr = {"bf16 few rows x 8 to 40 rows, eight waves split k, through registers, mfma16", fr_can_run<false>, fr_launch<false>, fr_cost};
const Variant kI8Fr = {"i8 few rows x 8 to 40 rows, eight waves split k, through registers, mfma16", fr_can_run<true>, fr_launch<true>, fr_cost};

}  // namespace

// Whether the call is better off here than on what else would run it.  Both sides were timed over 5400 calls (1 to 256
// problems, bf16 and int8, 16 to 130000 rows of W, 64 bytes to 34 KB of K), with the operands from memory and with the
// same ones over and over; the lines lie where the mean ratio of the times passes one.  What counts is how many 64-row
// tiles of W there are (the other kernels have about a workgroup for each), how many rows of X share a load of W, and how
// long K is.  Ratio here / there, operands from memory:
//   up to 32 tiles   0.17 .. 0.97 up to 32 rows of X whatever K, up to 64 rows from 512 bytes on (below 1.0 .. 1.14)
//   up to 64         0.25 .. 0.96 up to 16 rows, 0.4 .. 0.98 up to 32 from 256 bytes on, 0.5 .. 0.95 up to 64 from where the line is
//   up to 128        0.4 .. 1.0 up to 16 rows, 0.55 .. 0.93 up to 32 from 1 KB, 0.6 .. 0.82 up to 48 from 2 KB, 0.6 .. 0.81 up to 64 from 4 KB
//   one problem      its W are weights, which come from memory: up to 16 rows 0.57 .. 0.97 from 2 KB on; up to 48 rows 0.48 .. 0.91 where a
//                    compute unit has at most one workgroup, 0.7 .. 0.9 to 192 tiles from 8 KB on and 0.75 .. 0.9 where two full rounds
//                    stand against a second one there, else 1.0 .. 1.5
// The operands of several problems are as a rule another kernel's results and still in the caches, where a tile kernel gains
// more: 17 to 32 rows end at 128 tiles (beyond 1.1 .. 1.8), 33 to 48 at 64 (beyond 0.97 .. 1.6), 49 to 64 at 16 (32 problems 64 x 64 x
// 4096 int8 12.6 us and 8.2), 9 to 16 at 128 and 8 at 256 (192 x 16 x 256 x 2048 int8 31.9 and 20.4, 128 x 4 x 256 x 2048 18 and 13.5)
// -- unless W is more than the 256 MB last-level cache holds: up to 16 rows those have the lines of one problem (8 x 13 x 6872 x 4288
// 76 and 107, 192 x 16 x 1024 x 1024 73 and 96).
// 16 x 8192 x 8192 25 us here and 57, 16 x 4096 x 4096 7.8 and 18.7, 42 x 9266 x 11712 48 and 82; 192 problems 64 x 1024 x 64 97 and 15,
// 96 problems 49 x 6144 x 48 297 and 27.  Rows off a 16-byte boundary (there: the any-alignment kernel) have the same lines
// up to 128 tiles for at most 48 rows of X (more: 0.96 .. 1.6 beyond 32 tiles, 64 x 6976 x 3456 40 us here and 21), and 0.78 .. 1.0
// up to 16 rows and 256 tiles from 1 KB on.  A matrix-vector product with aligned rows (of
// any length) has a kernel of its own.
bool few_rows_preferred(const Problem &q)
{
    if (q.in_type == XP_F32 || !(q.in_type == XP_BF16 ? fr_can_run<false>(q) : fr_can_run<true>(q))) return false;
    const int64_t epc = 16 / elem_size(q.in_type);
    if (q.N == 1 && (((uintptr_t)q.A | (uintptr_t)q.B) & 15) == 0 && q.a_sm % epc == 0 && q.strideA % epc == 0 && q.strideB % epc == 0) return false;
    const int64_t n = fr_swapped(q) ? q.M : q.N, m = fr_swapped(q) ? q.N : q.M, kb = q.K * elem_size(q.in_type);
    const int64_t tiles = (n + 63) / 64 * q.batch;
    const bool from_memory = n * kb * q.batch > 300000000;
    if (q.batch > 1 && !(from_memory && m <= 16) && tiles > (m <= 8 ? 256 : m <= 32 ? 128 : m <= 48 ? 64 : 16)) return false;
    if (tiles <= 32) return m <= 32 || kb >= 512;
    if (m > 48 && !fr_aligned(q)) return false;
    if (tiles <= 64) return m <= 16 || kb >= (m <= 32 ? 256 : m <= 48 ? 1024 : 4096);
    if (tiles <= 128) return m <= 16 || kb >= (m <= 32 ? 1024 : m <= 48 ? 2048 : 4096);
    if (!fr_aligned(q)) return tiles <= 256 && m <= 16 && kb >= 1024;
    if (m <= 16) return kb >= (m <= 8 && tiles <= 256 ? 1024 : tiles <= 1024 || q.batch > 1 ? 2048 : 4096);
    const int64_t rows = 8 * fr_w_blocks(n, m, 1), workgroups = (n + rows - 1) / rows;
    return m <= 48 && kb >= 4096 && (workgroups <= 256 || (kb >= 8192 && tiles <= 192) || (m <= 32 && tiles > 256 && workgroups <= 512));
}

int fr_variants(xp_dtype in_type, const Variant **out)
{
    if (in_type == XP_F32) return 0;
    out[0] = in_type == XP_BF16 ? &kBfFr : &kI8Fr;
    return 1;
}

}  // namespace xp
