// MFMA kernel for operands of any alignment: bf16 x bf16 -> fp32 and int8 x int8 -> int32 GEMM, strided-batched GEMM and
// the NHWC convolution (Table 5 of the paper: GEMM, Batch GEMM, Conv2D NHWC) with extents, pitches and channel counts
// that are no multiple of a 16-byte chunk: odd sequence lengths and feature counts, a first layer's three channels.
//
// The direct-to-LDS kernels need 16-byte rows; here the tiles pass through registers, and a chunk may start at any
// element (a 16-byte load at an odd multiple of 2 bytes costs 10 to 20 % of the kernel: 2048 x 1024 x 1534 17.0 us, x 1535
// 17.3 to 18.5; cutting chunks out of dword-aligned loads instead was slower, 30 us against 27 at 2049 x 1021 x 1535, whether
// the fifth dword was loaded or taken from the next lane).  Care is needed where a chunk is not wholly inside its operand:
//   GEMM   rows (columns) past the edge are clamped to the last one, their results are not stored; a chunk along K past the
//          end exists in the last K step only, which takes a checked path (zeros past K).  A chunk along M or N may run
//          into the next k row, which is memory of the operand in every step but the last.
//   conv   for a filter row r the taps (s, c) of a pixel are one run of S*Cin consecutive elements of the image, and of the
//          filter: K is walked as R runs, each padded to whole chunks.  What of a chunk lies outside the image (left or
//          right) or past the run is an interval of its elements: it is loaded with the rest and masked with zeros.
// A chunk that would leave the whole operand is loaded from its last (first) 16 bytes and shifted into place.
// Structure: 4 waves, 2 x 2; two LDS buffers; one to three steps' loads fly while a step is multiplied; one barrier a step.
// Operands along K lie in LDS as 128-byte rows, operands along M or N as they lie in memory and come back through the
// transposing reads (ds_read_b64_tr_b16 / _b8).  Blocks are computed transposed (16x16x32 bf16, 16x16x64 int8): a lane
// stores four consecutive columns at once, at any 4-byte aligned address.
//
// Measured against the general kernel it takes over from: 2049 x 1021 x 1535 278 -> 26 us, 4001 x 4003 x 4005 180 us (710 TFLOP/s),
// int8 128 x 3196 x 4544 915 -> 19 us, 3x3 convolution 8 x 112 x 112 x 34 -> 44 205 -> 22 us.  Bound: a step's chain of LDS writes,
// barrier and reads (64x64 .. 128x128 tiles, 0.33 .. 0.85 us a step where MFMAs take 0.06 .. 0.25).
#include "xp_internal.hpp"
#include "xp_any_align.hpp"
#include "xp_epilogue.hpp"
#include "xp_lds_tr.hpp"

#include <climits>
#include <type_traits>

namespace xp {
namespace {

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;

constexpr int NTH = 256;
constexpr int STEPB = 128;                // bytes of K a step takes of every row (8 chunks)

struct UaParams {
    const char *A, *B;
    char *C;
    int M, N;
    long long K;                          // elements
    int run, R, run_c, steps;             // K as R runs of `run` elements = run_c chunks each; steps of 8 chunks
    unsigned run_magic;                   // ceil(2^32 / run_c); 0: one run, or one chunk a run
    int full;                             // the first `full` steps need no checks (GEMM)
    long long lda_b, ldb_b;               // bytes between rows (along K: of the outer index; along M or N: of k)
    long long a_ext, b_ext;               // bytes of one operand slice, from its first to past its last element
    long long ldc, c_plane, strideA_b, strideB_b, strideC;
    float alpha, beta;
    int tiles_m, tiles_n, group_m;
    int H, W, Cin, PQ, Q, sh, sw, ph, pw; // convolution
};

// the run that chunk number c of K belongs to
__device__ __forceinline__ unsigned run_of(unsigned c, const UaParams &p)
{
    return p.run_magic != 0u ? __umulhi(c, p.run_magic) : (p.R > 1 ? c : 0u);
}

// all of this wave's LDS reads and writes done, then the workgroup barrier; global loads stay in flight
__device__ __forceinline__ void wg_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One operand's tile: ROWS rows (or columns) x 128 bytes of K.
//   OC = false: contiguous along K (in a convolution the A operand: pixels x filter window)
//   OC = true:  contiguous along the outer index
template <int ESZ, int ROWS, bool OC, int PF>
struct Operand {
    static constexpr int EPC = 16 / ESZ;
    static constexpr int CH = ROWS * 8 / NTH;                    // chunks per thread and step
    static constexpr int CPR = OC ? ROWS * ESZ / 16 : 8;         // chunks per LDS row
    static constexpr int RSTEP = NTH / CPR;                      // rows between a thread's chunks
    static constexpr int ROWB = CPR * 16;
    static constexpr int BYTES = ROWS * STEPB;
    static constexpr unsigned ALL = (1u << EPC) - 1;

    // chunk swizzle of an LDS row (bank-conflict-free fragment reads; constant over a thread's rows)
    static __device__ __forceinline__ int swz(int row)
    {
        if constexpr (!OC) return row & 6;
        else if constexpr (ESZ == 2) return ROWB == 256 ? ((row & 3) | ((row >> 3) & 1) << 2) << 1 : (((row >> 1) & 1) | ((row >> 3) & 1) << 1) << 1;
        else return ROWB == 128 ? ((row >> 1) & 3) | ((row >> 4) & 1) << 2 : ((row >> 2) & 1) | ((row >> 4) & 1) << 1;
    }
    static __device__ __forceinline__ int row_of(int t) { return t / CPR; }
    static __device__ __forceinline__ int col_of(int t) { return t % CPR; }

    unsigned off[CH];                                            // byte offset of the thread's chunks within a step (from `base`)
    const char *base;                                            // the tile's first row (column)
    int t, outer0, outer;
    long long pitch, room;                                       // room: bytes from `base` to the operand's end
    u32x4 v[PF][CH];
    unsigned bits[PF][CH];

    __device__ __forceinline__ void init(const char *op, long long ext, long long pitch_b, int o0, int o_ext, int tid)
    {
        t = tid; pitch = pitch_b; outer0 = o0; outer = o_ext;
        const long long first = OC ? (long long)o0 * ESZ : (long long)o0 * pitch_b;
        base = op + first;
        room = ext - first;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int row = row_of(t) + i * RSTEP;
            if constexpr (OC) off[i] = (unsigned)(row * pitch) + (unsigned)(min(EPC * col_of(t), o_ext - 1 - o0) * ESZ);
            else off[i] = (unsigned)(min(row, o_ext - 1 - o0) * pitch) + 16 * col_of(t);
        }
    }
    // every chunk of the step lies inside the operand
    template <int SET> __device__ __forceinline__ void load(int step)
    {
        const char *at = base + (OC ? (long long)step * (STEPB / ESZ) * pitch : (long long)step * STEPB);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            v[SET][i] = load16(at + off[i]);
            bits[SET][i] = ALL;
        }
    }
    // K as p.R runs; zeros past a run, nothing read outside the operand
    template <int SET> __device__ __forceinline__ void load_checked(int step, const UaParams &p)
    {
        if constexpr (!OC) {
            const unsigned c = 8 * step + col_of(t), r = run_of(c, p);
            const int e0 = EPC * (int)(c - r * p.run_c);
            const int n = (int)r < p.R ? min(p.run - e0, EPC) : 0;
            const long long k_at = ((long long)r * p.run + e0) * ESZ;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const long long at = (long long)(off[i] - 16 * col_of(t)) + k_at;
                bits[SET][i] = (1u << max(n, 0)) - 1;
                v[SET][i] = load16_within(base, n > 0 ? at : 0, LLONG_MIN, room);
            }
        } else {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const unsigned kp = step * (STEPB / ESZ) + row_of(t) + i * RSTEP, r = run_of(kp / EPC, p);
                const int e = (int)(kp - r * p.run_c * EPC);
                const bool ok = (int)r < p.R && e < p.run;
                const int col = min(EPC * col_of(t), outer - 1 - outer0);
                const long long at = ((long long)r * p.run + e) * pitch + col * ESZ;
                bits[SET][i] = ok ? ALL : 0u;
                v[SET][i] = load16_within(base, ok ? at : 0, LLONG_MIN, room);
            }
        }
    }
    template <int SET, bool MASK> __device__ __forceinline__ void store(char *lds) const
    {
        char *at = lds + row_of(t) * ROWB + ((col_of(t) ^ swz(row_of(t))) << 4);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            u32x4 x = v[SET][i];
            if (MASK && __builtin_amdgcn_ballot_w64(bits[SET][i] != ALL) != 0) x = keep<ESZ>(x, bits[SET][i]);
            *(u32x4 *)(at + i * RSTEP * ROWB) = x;
        }
    }
    // MFMA fragment of rows (columns) 16*blk .. +15, k sub-step s of two
    static __device__ __forceinline__ u32x4 frag(const char *lds, int blk, int s, int lane)
    {
        const int a = lane & 15, g = lane >> 4;
        if constexpr (!OC) {
            const int row = blk * 16 + a;
            return *(const u32x4 *)(lds + row * ROWB + (((4 * s + g) ^ swz(row)) << 4));
        } else if constexpr (ESZ == 2) {
            const int row = 32 * s + 8 * g + (a >> 2);
            const char *at = lds + row * ROWB + (((2 * blk + ((a & 3) >> 1)) ^ swz(row)) << 4) + 8 * (a & 1);
            const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)at);
            const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(at + 4 * ROWB));
            return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            const int row = 64 * s + 16 * g + (a >> 1);
            const char *at = lds + row * ROWB + ((blk ^ swz(row)) << 4) + 8 * (a & 1);
            const i32x2 lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)at);
            const i32x2 hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2 *)(at + 8 * ROWB));
            return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3));
        }
    }
};

// The A operand of a convolution: output pixels x filter window (see the head of the file).
template <int ROWS, int PF>
struct Window {
    typedef Operand<2, ROWS, false, PF> Op;
    static constexpr int CH = Op::CH;
    const char *image;
    int t, at0[CH], h0[CH], lo[CH], hi[CH];                      // the window's first element (byte offset), its first image row, columns inside the image
    u32x4 v[PF][CH];
    unsigned bits[PF][CH];

    __device__ __forceinline__ void init(const UaParams &p, int m0, int tid)
    {
        t = tid;
        image = p.A;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const unsigned m = (unsigned)min(m0 + Op::row_of(t) + i * Op::RSTEP, p.M - 1);
            const unsigned n = m / (unsigned)p.PQ, pq = m - n * (unsigned)p.PQ;
            const unsigned oy = pq / (unsigned)p.Q, ox = pq - oy * (unsigned)p.Q;
            const int w0 = (int)ox * p.sw - p.pw;
            h0[i] = (int)oy * p.sh - p.ph;
            at0[i] = (int)((((long long)n * p.H + h0[i]) * p.W + w0) * p.Cin * 2);
            lo[i] = max(0, -w0 * p.Cin);
            hi[i] = min(p.run, (p.W - w0) * p.Cin);
        }
    }
    template <int SET> __device__ __forceinline__ void load_checked(int step, const UaParams &p)
    {
        const unsigned c = 8 * step + Op::col_of(t), r = run_of(c, p);
        const int e0 = 8 * (int)(c - r * p.run_c);
        const int at_k = (int)(((long long)r * p.W * p.Cin + e0) * 2);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int a = min(max(lo[i] - e0, 0), 8), b = min(max(hi[i] - e0, 0), 8);
            const bool inside = (int)r < p.R && (unsigned)(h0[i] + (int)r) < (unsigned)p.H && a < b;
            bits[SET][i] = inside ? ((1u << b) - 1) & ~((1u << a) - 1) : 0u;
            v[SET][i] = load16_within(image, inside ? at0[i] + at_k : 0, 0, p.a_ext);
        }
    }
    template <int SET, bool MASK> __device__ __forceinline__ void store(char *lds) const
    {
        char *to = lds + Op::row_of(t) * Op::ROWB + ((Op::col_of(t) ^ Op::swz(Op::row_of(t))) << 4);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            u32x4 x = v[SET][i];
            if (__builtin_amdgcn_ballot_w64(bits[SET][i] != Op::ALL) != 0) x = keep<2>(x, bits[SET][i]);
            *(u32x4 *)(to + i * Op::RSTEP * Op::ROWB) = x;
        }
    }
};

enum { A_K = 0, A_OC = 1, A_CONV = 2 };

template <bool INT8, int AF, bool B_OC, int BM, int BN, int PF>
__global__ __launch_bounds__(NTH, 2) void ua_kernel(UaParams p)
{
    using KD = Kind<INT8>;
    constexpr int ESZ = KD::ESZ;
    using OpA = Operand<ESZ, BM, AF == A_OC, PF>;
    using OpB = Operand<ESZ, BN, B_OC, PF>;
    constexpr int MI = BM / 32, NI = BN / 32;
    constexpr int STAGE = OpA::BYTES + OpB::BYTES;
    __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // workgroup -> tile: one XCD owns a run of consecutive tiles, walked in groups of group_m tile rows
    int bid = blockIdx.x;
    const int nb = p.tiles_m * p.tiles_n;
    if ((nb & 7) == 0) bid = (bid & 7) * (nb >> 3) + (bid >> 3);
    const int gsz = p.group_m * p.tiles_n;
    const int grp = bid / gsz, first_m = grp * p.group_m;
    const int gm = min(p.tiles_m - first_m, p.group_m);
    const int tm = first_m + (bid % gsz) % gm, tn = (bid % gsz) / gm;
    const int m0 = tm * BM, n0 = tn * BN;
    const long long batch = blockIdx.y;

    typename std::conditional<AF == A_CONV, Window<BM, PF>, OpA>::type a;
    OpB b;
    if constexpr (AF == A_CONV) a.init(p, m0, tid);
    else a.init(p.A + batch * p.strideA_b, p.a_ext, p.lda_b, m0, p.M, tid);
    b.init(p.B + batch * p.strideB_b, p.b_ext, p.ldb_b, n0, p.N, tid);

    auto load = [&](int step, auto set_c, auto checked_c) {
        constexpr int SET = decltype(set_c)::value;
        if constexpr (decltype(checked_c)::value) {
            a.template load_checked<SET>(step, p);
            b.template load_checked<SET>(step, p);
        } else if constexpr (AF != A_CONV) {
            a.template load<SET>(step);
            b.template load<SET>(step);
        }
    };

    typename KD::acc_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = typename KD::acc_t{0, 0, 0, 0};

    // One step of 128 bytes of K, two sub-steps of MFMAs.  Everything else is issued under them: the second sub-step's
    // fragments are read under the first one's MFMAs, then the next tile goes into the other LDS buffer, and behind the
    // barrier its first fragments are read under the second sub-step's MFMAs.  PF register sets hold the global loads: step
    // s + PF is requested during step s.  (Not so woven in a convolution: there more workgroups per compute unit do the
    // hiding, and the second fragment set's registers cost one; first layer 224 x 224 x 3, 51.7 us against 57.1.)
    constexpr bool WOVEN = AF != A_CONV;
    u32x4 af[2][MI], bf[2][NI];
    auto read = [&](int at, auto s_c) {
        constexpr int S = decltype(s_c)::value;
#pragma unroll
        for (int i = 0; i < MI; ++i) af[S][i] = OpA::frag(lds + at, wm * MI + i, S, lane);
#pragma unroll
        for (int j = 0; j < NI; ++j) bf[S][j] = OpB::frag(lds + at + OpA::BYTES, wn * NI + j, S, lane);
    };
    auto multiply = [&](auto s_c) {
        constexpr int S = decltype(s_c)::value;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = KD::mma(bf[S][j], af[S][i], acc[i][j]);
    };
    constexpr std::integral_constant<int, 0> S0{};
    constexpr std::integral_constant<int, 1> S1{};
    static_for<PF>([&](auto u) {
        if (u < p.steps) {
            if (AF != A_CONV && u < p.full) load(u, u, std::false_type{});
            else load(u, u, std::true_type{});
        }
    });
    a.template store<0, true>(lds);
    b.template store<0, true>(lds + OpA::BYTES);
    wg_barrier();
    if constexpr (WOVEN) read(0, S0);
    int cur = 0;
    // u: the register set of the step; CHECK: loads may need checks; LAST: steps may be over (a condition around a load makes
    // the waits for older ones stricter than they need be, so only the last few steps have it)
    auto one = [&](int step, auto u_c, auto check_c, auto last_c) {
        constexpr int U = decltype(u_c)::value, NX = (U + 1) % PF;
        constexpr bool CHECK = decltype(check_c)::value, LAST = decltype(last_c)::value;
        if (!LAST || step + PF < p.steps) load(step + PF, u_c, check_c);
        const bool next = !LAST || step + 1 < p.steps;
        if constexpr (WOVEN) {
            read(cur, S1);
            multiply(S0);
        } else {
            read(cur, S0);
            multiply(S0);
            read(cur, S1);
            multiply(S1);
        }
        cur = STAGE - cur;
        if (next) {
            a.template store<NX, CHECK>(lds + cur);               // the buffer every wave finished reading before the last barrier
            b.template store<NX, CHECK>(lds + cur + OpA::BYTES);
            wg_barrier();
            if constexpr (WOVEN) read(cur, S0);
        }
        if constexpr (WOVEN) multiply(S1);
    };
    int step = 0;
    constexpr std::integral_constant<bool, AF == A_CONV> checked{};
    const int plain = AF == A_CONV ? p.steps : p.full;
    for (; step + 2 * PF <= plain; step += PF)
        static_for<PF>([&](auto u) { one(step + u, u, checked, std::false_type{}); });
    for (; step < p.steps; step += PF)
        static_for<PF>([&](auto u) {
            if (step + u < p.steps) one(step + u, u, std::true_type{}, std::true_type{});
        });

    // accumulator register v of lane l: row l & 15, column 4 * (l >> 4) + v
    using OutT = typename KD::out_t;
    typedef OutT out4_any __attribute__((ext_vector_type(4), aligned(4)));
    OutT *C = (OutT *)p.C + batch * p.strideC;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row0 = m0 + (wm * MI + i) * 16, row = row0 + (lane & 15);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col0 = n0 + (wn * NI + j) * 16, col = col0 + 4 * (lane >> 4);
            if constexpr (!INT8) {
                if (p.c_plane) {
                    store_block16t_planar(acc[i][j], C, p.c_plane, row0, col0, lane, p.M, p.N, p.alpha);
                    continue;
                }
            }
            if (row >= p.M) continue;
            OutT *dst = C + (long long)row * p.ldc + col;
            if constexpr (INT8) {
                if (col + 4 <= p.N) *(out4_any *)dst = acc[i][j];
                else
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (col + v < p.N) dst[v] = acc[i][j][v];
            } else {
                if (p.beta == 0.0f && col + 4 <= p.N) {
                    *(out4_any *)dst = p.alpha * acc[i][j];
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (col + v < p.N) {
                            float x = p.alpha * acc[i][j][v];
                            if (p.beta != 0.0f) x = __builtin_fmaf(p.beta, dst[v], x);
                            dst[v] = x;
                        }
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------ host side

// contiguous along K (1), along the outer index (2) or neither (0).  An outer extent of one is both: along K if it can be.
int ua_form(int64_t s_outer, int64_t s_k)
{
    return s_k == 1 ? 1 : (s_outer == 1 ? 2 : 0);
}

template <bool INT8>
bool ua_operand_ok(int64_t s_outer, int64_t s_k, int64_t outer, int64_t K, int tile)
{
    const int64_t esz = INT8 ? 1 : 2, epc = 16 / esz, bk = STEPB / esz;
    const int64_t ext = ua_form(s_outer, s_k) == 1 ? (outer - 1) * s_outer + K : (K - 1) * s_k + outer;
    if (ext * esz < 16) return false;                            // an operand of at least one chunk
    if (ua_form(s_outer, s_k) == 1) return (tile - 1) * s_outer * esz + K * esz < 0x7fffffffLL;
    // a chunk that starts at the last column may run into the next k row, but not past it
    return ua_form(s_outer, s_k) == 2 && s_k >= epc && outer <= 0x7fffffffLL && bk * s_k * esz + tile * esz < 0x7fffffffLL;
}

template <bool INT8, int BM, int BN>
bool ua_can_run(const Problem &q)
{
    const int64_t esz = INT8 ? 1 : 2, epc = 16 / esz;
    if (q.in_type != (INT8 ? XP_I8 : XP_BF16) || q.K <= 0 || q.batch > 65535) return false;
    if (q.c_plane && (q.beta != 0.0f || INT8)) return false;
    if (q.M > 0x3fffffffLL || q.N > 0x3fffffffLL || q.K > 0x3fffffffLL) return false;
    if (((q.M + BM - 1) / BM) * ((q.N + BN - 1) / BN) > 0x7fffffffLL) return false;
    if (q.conv) {
        if (INT8) return false;
        const int64_t run = q.S * q.Cin, in_bytes = (q.M / (q.P * q.Q)) * q.H * q.W * q.Cin * esz;
        // 32-bit byte offsets, window parts outside the image included; an image of at least one chunk
        if (in_bytes < 16 || in_bytes + (q.ph + q.R + 1) * (q.W + q.S) * q.Cin * esz + q.pw * q.Cin * esz >= 0x7fffffffLL) return false;
        if ((q.W + 2 * q.pw) * q.Cin >= 0x3fffffffLL || q.H + 2 * q.ph >= 0x3fffffffLL || q.P * q.Q >= 0x7fffffffLL) return false;
        if (q.R * ((run + epc - 1) / epc) + 16 >= 65536) return false;             // the division of a chunk number by run_c is exact below 2^16
    } else {
        if (!ua_operand_ok<INT8>(q.a_sm, q.a_sk, q.M, q.K, BM)) return false;
    }
    return ua_operand_ok<INT8>(q.b_sn, q.b_sk, q.N, q.K, BN);
}

template <bool INT8, int BM, int BN, int PF>
hipError_t ua_launch(const Problem &q)
{
    const int64_t esz = INT8 ? 1 : 2, epc = 16 / esz;
    UaParams p;
    p.A = (const char *)q.A; p.B = (const char *)q.B; p.C = (char *)q.C;
    p.M = (int)q.M; p.N = (int)q.N; p.K = q.K;
    const int af = q.conv ? A_CONV : (ua_form(q.a_sm, q.a_sk) == 1 ? A_K : A_OC);
    const bool b_oc = ua_form(q.b_sn, q.b_sk) == 2;
    p.R = q.conv ? (int)q.R : 1;
    p.run = q.conv ? (int)(q.S * q.Cin) : (int)q.K;
    p.run_c = (int)((p.run + epc - 1) / epc);
    p.run_magic = p.R == 1 || p.run_c == 1 ? 0u : (unsigned)(((1ull << 32) + p.run_c - 1) / p.run_c);
    p.steps = (int)(((int64_t)p.R * p.run_c + 7) / 8);
    p.lda_b = (af == A_OC ? q.a_sk : q.a_sm) * esz;
    p.ldb_b = (b_oc ? q.b_sk : q.b_sn) * esz;
    p.a_ext = q.conv ? (q.M / (q.P * q.Q)) * q.H * q.W * q.Cin * esz
                     : ((af == A_OC ? (q.K - 1) * q.a_sk + q.M : (q.M - 1) * q.a_sm + q.K)) * esz;
    p.b_ext = (b_oc ? (q.K - 1) * q.b_sk + q.N : (q.N - 1) * q.b_sn + q.K) * esz;
    // unchecked steps: all of K inside, and for an operand along M or N a k row after the step's last one
    p.full = (int)((q.K - (af == A_OC || b_oc ? 1 : 0)) / (STEPB / esz));
    p.ldc = q.ldc; p.c_plane = q.c_plane;
    p.strideA_b = q.strideA * esz; p.strideB_b = q.strideB * esz; p.strideC = q.strideC;
    p.alpha = q.alpha; p.beta = q.beta;
    p.tiles_m = (int)((q.M + BM - 1) / BM);
    p.tiles_n = (int)((q.N + BN - 1) / BN);
    p.group_m = p.tiles_m < 8 ? p.tiles_m : 8;
    p.H = (int)q.H; p.W = (int)q.W; p.Cin = (int)q.Cin; p.PQ = (int)(q.P * q.Q); p.Q = (int)q.Q;
    p.sh = (int)q.sh; p.sw = (int)q.sw; p.ph = (int)q.ph; p.pw = (int)q.pw;
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)q.batch);
#define XP_UA(AF, BO) hipLaunchKernelGGL((ua_kernel<INT8, AF, BO, BM, BN, PF>), grid, dim3(NTH), 0, q.stream, p)
    if (af == A_K) { if (b_oc) XP_UA(A_K, true); else XP_UA(A_K, false); }
    else if (af == A_OC) { if (b_oc) XP_UA(A_OC, true); else XP_UA(A_OC, false); }
    else if constexpr (!INT8) { if (b_oc) XP_UA(A_CONV, true); else XP_UA(A_CONV, false); }
#undef XP_UA
    return hipGetLastError();
}

// Calls that the kernels for aligned operands decline: rows or channel counts that are no multiple of 16 (convolution: 64)
// bytes, bases that are not aligned, filters along their output channels.  Filters of more than 32 taps are beyond the direct-to-LDS
// kernels, but where channels fill whole 128-byte rows the register-staged ones take them (not with a planar output) at
// up to three times the speed: 6 x 7 x 7 x 256 -> 32, 11 x 11 121 us and 403 here, 11 x 112 x 112 x 320 -> 8, 7 x 7 273 and 337.
bool ua_needed(const Problem &q)
{
    const int64_t epc = 16 / elem_size(q.in_type);
    const bool base = (((uintptr_t)q.A | (uintptr_t)q.B) & 15) != 0;
    if (q.conv) return base || q.Cin % 32 != 0 || q.b_sk != 1 || (q.R * q.S > 32 && (q.Cin % 64 != 0 || q.c_plane != 0));
    auto rows = [&](int64_t s_outer, int64_t s_k, int64_t outer, int64_t stride) {
        return stride % epc != 0 || (s_k == 1 ? (s_outer % epc != 0 || q.K % epc != 0) : (s_k % epc != 0 || outer % epc != 0));
    };
    return base || rows(q.a_sm, q.a_sk, q.M, q.strideA) || rows(q.b_sn, q.b_sk, q.N, q.strideB);
}

// Measured (us per K step and tile on a compute unit, misaligned rows; 2049 x 1021 x 1535, 2048 x 1024 x 1535, 4001 x 4003 x
// 4005, 501 x 503 x 505): 128x128 0.85 alone on its compute unit and 0.71 beside another, 128x64 0.5, 64x64 0.34.  Up to a
// few tiles per compute unit it is the fullest one that counts.  Where the operands are aligned the direct-to-LDS kernels
// are up to twice as fast (2048 x 1024 x 1536: 11 us, this kernel 14), whatever their estimates say.
template <int BM, int BN>
double ua_cost(const Problem &q)
{
    const double per_cu = (double)((q.M + BM - 1) / BM) * (double)((q.N + BN - 1) / BN) * (double)q.batch / 256.0;
    const double full = per_cu <= 3.0 ? __builtin_ceil(per_cu) : per_cu;
    const double chunk = 16.0 / elem_size(q.in_type);
    const double steps = __builtin_ceil(q.conv ? (double)q.R * __builtin_ceil((double)(q.S * q.Cin) / chunk) / 8.0 : (double)q.K / (8.0 * chunk));
    const double us = BM * BN == 128 * 128 ? (full <= 1.0 ? 0.85 : 0.71) : (BM * BN == 128 * 64 ? 0.5 : 0.34);
    return (4.0 + steps * full * us) * (ua_needed(q) ? 1.0 : 8.0);
}

#define XP_UA_VARIANT(NAME, TYPE, INT8, BM, BN, PF) \
    const Variant NAME = {TYPE " " #BM "x" #BN "x128B waves 2x2 any alignment, through registers, mfma16", ua_can_run<INT8, BM, BN>, ua_launch<INT8, BM, BN, PF>, ua_cost<BM, BN>};

XP_UA_VARIANT(kBfUa128, "bf16", false, 128, 128, 2)
XP_UA_VARIANT(kBfUa128x64, "bf16", false, 128, 64, 2)
XP_UA_VARIANT(kBfUa64, "bf16", false, 64, 64, 3)
XP_UA_VARIANT(kI8Ua128, "i8", true, 128, 128, 2)
XP_UA_VARIANT(kI8Ua128x64, "i8", true, 128, 64, 2)
XP_UA_VARIANT(kI8Ua64, "i8", true, 64, 64, 3)

}  // namespace

int ua_variants(xp_dtype in_type, const Variant **out)
{
    if (in_type == XP_BF16) { out[0] = &kBfUa128; out[1] = &kBfUa128x64; out[2] = &kBfUa64; return 3; }
    if (in_type == XP_I8) { out[0] = &kI8Ua128; out[1] = &kI8Ua128x64; out[2] = &kI8Ua64; return 3; }
    return 0;
}

}  // namespace xp
