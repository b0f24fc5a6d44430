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

// Microseconds: W from memory at 5 TB/s (8 out of the last-level cache), the fullest compute unit's loads of W and X at 45 KB a
// microsecond (35 above 48 rows of X in several rounds: 60 x 12000 x 9000 92 us, 78 on the 64-row tile), 18 where rows start off a multiple of 4 bytes (64 x 8192 x 8192 37.7 us, 16 x 8191 x 8193 59 us)
double fr_cost(const Problem &q)
{
    const double n = (double)(fr_swapped(q) ? q.M : q.N), m = (double)(fr_swapped(q) ? q.N : q.M), kb = (double)q.K * elem_size(q.in_type);
    const int wb = fr_w_blocks((int64_t)n, (int64_t)m, q.batch);
    const double per_cu = __builtin_ceil(__builtin_ceil(n / (8.0 * wb)) * q.batch / 256.0);
    const double loads = per_cu * (8.0 * wb + fr_rows((int64_t)m)) * kb / (!fr_aligned(q) ? 18e3 : m > 48.0 && per_cu > 1.0 ? 35e3 : 45e3);
    const double w_us = n * kb * q.batch / (n * kb * q.batch >= 6.7e7 ? 5e6 : 8e6);
    return 4.0 + (loads > w_us ? loads : w_us);
}

const Variant kBfFr = {"bf16 few rows x 8 to 32 rows, eight waves split k, through registers, mfma16", fr_can_run<false>, fr_launch<false>, fr_cost};
const Variant kI8Fr = {"i8 few rows x 8 to 32 rows, eight waves split k, through registers, mfma16", fr_can_run<true>, fr_launch<true>, fr_cost};

}  // namespace

// Whether the call is better off here than on a tile of 64 rows, whose compute units take 64 + 64 rows of K at 70 KB a
// microsecond (40 where W does not fit the last-level cache, 30 where rows are not aligned) and W at 4.6 TB/s (8).
// Measured us, here and there: 16 x 8192 x 8192 25 and 57, 16 x 4096 x 4096 7.8 and 18.7, 64 x 4096 x 4096 13.1 and 19.2,
// 64 x 1024 x 16384 35 and 62; on the other side of the line 64 x 16384 x 2048 25 and 20, 32 x 16384 x 1024 10.7 and 7.8,
// 64 x 8191 x 8193 89 and 71.  A K of less than a block for every wave and a
// matrix-vector product with aligned rows (of any length) stay where they were.
bool few_rows_preferred(const Problem &q)
{
    if (q.in_type == XP_F32 || !(q.in_type == XP_BF16 ? fr_can_run<false>(q) : fr_can_run<true>(q))) return false;
    const double n = (double)(fr_swapped(q) ? q.M : q.N), kb = (double)q.K * elem_size(q.in_type);
    const bool aligned = fr_aligned(q);
    const int64_t epc = 16 / elem_size(q.in_type);
    const bool gemv = q.N == 1 && (((uintptr_t)q.A | (uintptr_t)q.B) & 15) == 0 && q.a_sm % epc == 0 && q.strideA % epc == 0 && q.strideB % epc == 0;
    if (kb < NW * BLOCKB || gemv) return false;
    const bool cold = n * kb * q.batch >= 6.7e7;
    const double loads = __builtin_ceil(__builtin_ceil(n / 64.0) * q.batch / 256.0) * 128.0 * kb / (!aligned ? 30e3 : cold ? 40e3 : 70e3);
    const double w_us = n * kb * q.batch / (cold ? 4.6e6 : 8e6);
    return fr_cost(q) <= 4.0 + (loads > w_us ? loads : w_us);
}

int fr_variants(xp_dtype in_type, const Variant **out)
{
    if (in_type == XP_F32) return 0;
    out[0] = in_type == XP_BF16 ? &kBfFr : &kI8Fr;
    return 1;
}

}  // namespace xp
