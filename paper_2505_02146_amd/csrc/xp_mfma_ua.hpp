// MFMA kernel for operands of any alignment: bf16 x bf16 -> fp32 and int8 x int8 -> int32 GEMM, strided-batched GEMM and
// the NHWC convolution (Table 5 of the paper: GEMM, Batch GEMM, Conv2D NHWC) with extents, pitches and channel counts
// that are no multiple of a 16-byte chunk: odd sequence lengths and feature counts, a first layer's three channels.
//
// The direct-to-LDS kernels need 16-byte rows; here the tiles pass through registers, and a chunk may start at any
// element (a 16-byte load at an odd multiple of 2 bytes costs 10 to 20 % of the kernel: 2048 x 1024 x 1534 17.0 us, x 1535
// 17.3 to 18.5; cutting chunks of 128 bytes a row out of dword-aligned loads was slower, 30 us against 27 at 2049 x 1021 x 1535, whether
// the fifth dword was loaded or taken from the next lane: it pays with 256 bytes a row, below).  Care is needed where a chunk is not wholly inside its operand:
//   GEMM   rows (columns) past the edge are clamped to the last one, their results are not stored; a chunk along K past the
//          end exists in the last K step only, which takes a checked path (zeros past K).  A chunk along M or N may run
//          into the next k row, which is memory of the operand in every step but the last.
//   conv   for a filter row r the taps (s, c) of a pixel are one run of S*Cin consecutive elements of the image, and of the
//          filter: K is walked as R runs, each padded to whole chunks.  What of a chunk lies outside the image (left or
//          right) or past the run is an interval of its elements: it is loaded with the rest and masked with zeros.
// A chunk that would leave the whole operand is loaded from its last (first) 16 bytes and shifted into place.  Loads from dwords
// take a dword whole: up to three bytes that share it with the first element of an operand, and lie before that, come along unused.
// Structure: two LDS buffers; one or two steps' loads fly while a step is multiplied; one barrier a step.  Operands along K lie in
// LDS as rows of a step's bytes, operands along M or N as they lie in memory and come back through the transposing reads
// (ds_read_b64_tr_b16 / _b8).  Blocks are computed transposed (16x16x32 bf16, 16x16x64 int8): a lane stores four consecutive
// columns at once, at any 4-byte aligned address.
//
// What bounds it, by time stamps (2049 x 1021 x 1535, 18.6 us, 96x96 tiles on 242 of 256 compute units, 12 steps of 128 k): 3.1 us to the first
// step in LDS, 8 steps in the loop at 0.73 us (67 KB/us of loads), the last four, on the path for any step, at 1.25, 0.8 for the groups'
// sums, 1.2 for the stores, 2.7 outside the workgroups.  By themselves a unit's loads run at 65 KB/us of rows that start on any element, 98 of rows
// on 16 bytes.  So tiles are chosen to fill the card once, and:
//   K groups   tiles of 32x64, 64x32 and 64x64 by eight waves, a quarter or half of a step's K each (their sums meet in LDS): few
//              tiles and a long K.  75 x 3719 x 6108 31.9 -> 19.7 us, 896 x 104 x 5196 26.8 -> 17.3, int8 216 x 923 x 6985 26 -> 17
//   eight waves over 192x128: half the bytes a flop of 64x64, for large products.  2624 x 4450 x 5376 157 -> 139
//   from dwords  96x96: rows that start inside a dword are loaded from dword boundaries, 256 bytes a row and step, and put in place
//              between the lanes (a DPP move and four byte alignments a chunk, against 66 -> 96 KB/us for the load alone)
//   dealt out  loads between the MFMAs and LDS writes instead of in one run: a wave stands still at a load that the memory unit has
//              no room for.  Pays where one workgroup is alone on its unit: 2049 x 1021 x 1535 128x128 27.9 -> 24.4; two on a unit hide
//              it from each other already (4001 x 4003 x 4005 197 without, 213 with)
// Measured against the general kernel they took over from: 2049 x 1021 x 1535 278 -> 19.4 us, 4001 x 4003 x 4005 170 us (750 TFLOP/s),
// int8 128 x 3196 x 4544 915 -> 16 us, 3x3 convolution 8 x 112 x 112 x 34 -> 44 205 -> 22 us.
#pragma once

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

constexpr int SUBB = 128;                 // bytes of K that one group of waves takes of every row and step (8 chunks)

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
    int tiles_m, tiles_n, group_m, batch;
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

constexpr int pow2_from(int n) { int p = 1; while (p < n) p *= 2; return p; }

// One operand's tile: ROWS rows (or columns) x STEPB bytes of K, loaded by NT threads.
//   OC = false: contiguous along K (in a convolution the A operand: pixels x filter window)
//   OC = true:  contiguous along the outer index (LDS rows are whole powers of two: the last chunks of a 96-column row
//               repeat the one before them)
template <int ESZ, int ROWS, bool OC, bool SH, bool RUNS, int PF, int NT, int STEPB>
struct Operand {
    static constexpr int EPC = 16 / ESZ;
    static constexpr int CPR = OC ? pow2_from(ROWS * ESZ / 16 + (SH ? 1 : 0)) : STEPB / 16;     // lanes that load a row
    static constexpr int ROWB = OC ? pow2_from(ROWS * ESZ / 16) * 16 : STEPB;
    static constexpr int RSTEP = NT / CPR;                       // rows between a thread's chunks
    static constexpr int NROW = OC ? STEPB / ESZ : ROWS;         // LDS rows
    static constexpr int CH = (NROW + RSTEP - 1) / RSTEP;        // chunks per thread and step
    static constexpr int BYTES = CH * RSTEP * ROWB;
    static constexpr unsigned ALL = (1u << EPC) - 1;
    static_assert(NT % CPR == 0 && (RSTEP % 16 == 0 || CH == 1), "whole rounds of the workgroup; the swizzle is a thread's");
    static_assert(!SH || (OC ? CPR <= 16 : CPR == 16), "a row's chunks in the sixteen lanes that exchange their dwords");

    // chunk swizzle of an LDS row (bank-conflict-free fragment reads; constant over a thread's rows)
    static __device__ __forceinline__ int swz(int row)
    {
        if constexpr (!OC) return ROWB == 128 ? row & 6 : row & 15;
        else if constexpr (ESZ == 2) return ROWB == 64 ? 0 : ROWB >= 256 ? ((row & 3) | ((row >> 3) & 1) << 2) << 1 : (((row >> 1) & 1) | ((row >> 3) & 1) << 1) << 1;
        else return ROWB >= 256 ? (row & 7) | ((row >> 4) & 1) << 3 : ROWB == 128 ? ((row >> 1) & 3) | ((row >> 4) & 1) << 2 : ROWB == 64 ? ((row >> 2) & 1) | ((row >> 4) & 1) << 1 : 0;
    }
    static __device__ __forceinline__ int row_of(int t) { return t / CPR; }
    static __device__ __forceinline__ int col_of(int t) { return t % CPR; }

    unsigned off[CH];                                            // byte offset of the thread's chunks within a step (from `from`)
    const char *base, *from;                                     // the tile's first row (column); the same, SH: its dword
    unsigned sh[SH ? CH : 1], carry[SH && !OC ? CH : 1];         // bytes of a chunk's first dword in front of it; the dword in front of a row's step
    bool exact[PF];                                              // SH: the set's chunks are in place already (load_checked)
    bool tail_inside;                                            // what the last, partly filled step reads past K lies in the operand
    int t, outer0, outer;
    long long pitch, room;                                       // room: bytes from `base` to the operand's end
    u32x4 v[PF][CH];
    unsigned bits[RUNS ? PF : 1][RUNS ? CH : 1];

    __device__ __forceinline__ void init(const char *op, long long ext, long long pitch_b, int o0, int o_ext, int tid, int steps)
    {
        t = tid; pitch = pitch_b; outer0 = o0; outer = o_ext;
        const long long first = OC ? (long long)o0 * ESZ : (long long)o0 * pitch_b;
        base = op + first;
        room = ext - first;
        tail_inside = OC ? o0 + ROWS + (SH ? EPC : 0) <= o_ext : (long long)min(ROWS - 1, o_ext - 1 - o0) * pitch_b + (long long)steps * STEPB + 8 <= room;
        const unsigned lead = SH ? (unsigned)(unsigned long long)base & 3u : 0u;
        from = base - lead;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int row = row_of(t) + i * RSTEP;
            if constexpr (OC) {
                off[i] = (unsigned)(row * pitch) + (unsigned)(min(min(EPC * col_of(t), ROWS - (SH ? 0 : EPC)), o_ext - 1 - o0) * ESZ) + lead;
                if constexpr (SH) { sh[i] = off[i] & 3u; off[i] &= ~3u; }
            } else {
                const unsigned start = (unsigned)(min(row, min(ROWS - 1, o_ext - 1 - o0)) * pitch) + lead;
                if constexpr (SH) {
                    sh[i] = start & 3u;
                    carry[i] = *(const unsigned *)(from + (start & ~3u));        // the dword of the row's first element
                    off[i] = (start & ~3u) + 4 + 16 * col_of(t);
                } else off[i] = start + 16 * col_of(t);
            }
        }
    }
    // chunk i of a step that lies inside the operand
    template <int SET> __device__ __forceinline__ void load(int step, int i)
    {
        const char *at = from + (OC ? (long long)step * (STEPB / ESZ) * pitch : (long long)step * STEPB);
        if constexpr (SH) v[SET][i] = *(const u32x4_dw *)(at + off[i]);
        else v[SET][i] = load16(at + off[i]);
    }
    // any step of a product: what lies past K is read, if it is memory of the operand, and masked when it is stored
    template <int SET> __device__ __forceinline__ void load_any(int step, const UaParams &p)
    {
        if (!tail_inside && step >= p.full) { load_checked<SET>(step, p); return; }
        exact[SET] = false;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if constexpr (OC) {
                const int krow = step * (STEPB / ESZ) + row_of(t) + i * RSTEP, past = max(krow - (p.run - 1), 0);      // (k rows past the last one: that one)
                const char *at = from + (long long)step * (STEPB / ESZ) * pitch - (long long)past * pitch + off[i];
                if constexpr (SH) v[SET][i] = *(const u32x4_dw *)((unsigned long long)at & ~3ull);
                else v[SET][i] = load16(at);
            } else load<SET>(step, i);
        }
    }
    // K as p.R runs; zeros past a run, nothing read outside the operand
    template <int SET> __device__ __forceinline__ void load_checked(int step, const UaParams &p)
    {
        exact[SET] = true;
        if constexpr (!OC) {
            const unsigned c = CPR * step + col_of(t), r = run_of(c, p);
            const int e0 = EPC * (int)(c - r * p.run_c);
            const int n = (int)r < p.R ? min(p.run - e0, EPC) : 0;
            const long long k_at = ((long long)r * p.run + e0) * ESZ;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const long long at = (long long)min(row_of(t) + i * RSTEP, min(ROWS - 1, outer - 1 - outer0)) * pitch + k_at;
                if constexpr (RUNS) bits[SET][i] = (1u << max(n, 0)) - 1;
                v[SET][i] = load16_within(base, n > 0 ? at : 0, LLONG_MIN, room);
            }
        } else {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const unsigned kp = step * (STEPB / ESZ) + row_of(t) + i * RSTEP, r = run_of(kp / EPC, p);
                const int e = (int)(kp - r * p.run_c * EPC);
                const bool ok = (int)r < p.R && e < p.run;
                const int col = min(min(EPC * col_of(t), ROWS - (SH ? 0 : EPC)), outer - 1 - outer0);
                const long long at = ((long long)r * p.run + e) * pitch + col * ESZ;
                if constexpr (RUNS) bits[SET][i] = ok ? ALL : 0u;
                v[SET][i] = load16_within(base, ok ? at : 0, LLONG_MIN, room);
            }
        }
    }
    // chunk i of the step into LDS; MASK: parts of it may lie past K
    template <int SET, bool MASK> __device__ __forceinline__ void store(char *lds, int i, int step, const UaParams &p)
    {
        u32x4 x = v[SET][i];
        if constexpr (SH) {
            if (!MASK || !exact[SET]) {
                if constexpr (!OC) {
                    // the loads run one dword ahead of the row: dword j of the chunk ends in dword j of the load and begins in the
                    // dword before it, the lane to the left's last (the row's first lane: of the step before)
                    const unsigned before = __builtin_amdgcn_update_dpp(carry[i], x[3], 0x111, 0xf, 0xf, false);      // row_shr:1
                    carry[i] = __builtin_amdgcn_update_dpp(0u, x[3], 0x121, 0xf, 0xf, false);                         // row_ror:1
                    x = u32x4{__builtin_amdgcn_alignbyte(x[0], before, sh[i]), __builtin_amdgcn_alignbyte(x[1], x[0], sh[i]),
                              __builtin_amdgcn_alignbyte(x[2], x[1], sh[i]), __builtin_amdgcn_alignbyte(x[3], x[2], sh[i])};
                } else {
                    // the loads begin in the dword of the chunk's first element: its last elements are in the lane to the right's first dword
                    const unsigned behind = __builtin_amdgcn_update_dpp(0u, x[0], 0x101, 0xf, 0xf, false);   // row_shl:1
                    x = u32x4{__builtin_amdgcn_alignbyte(x[1], x[0], sh[i]), __builtin_amdgcn_alignbyte(x[2], x[1], sh[i]),
                              __builtin_amdgcn_alignbyte(x[3], x[2], sh[i]), __builtin_amdgcn_alignbyte(behind, x[3], sh[i])};
                }
            }
        }
        if constexpr (MASK) {
            unsigned b;
            if constexpr (RUNS) b = bits[SET][i];
            else if constexpr (OC) b = step * (STEPB / ESZ) + row_of(t) + i * RSTEP < p.run ? ALL : 0u;
            else b = (1u << min(max(p.run - EPC * (CPR * step + col_of(t)), 0), EPC)) - 1;
            if (__builtin_amdgcn_ballot_w64(b != ALL) != 0) x = keep<ESZ>(x, b);
        }
        char *at = lds + row_of(t) * ROWB + ((col_of(t) ^ swz(row_of(t))) << 4);
        if (CPR * 16 == ROWB || col_of(t) < ROWB / 16) *(u32x4 *)(at + i * RSTEP * ROWB) = x;
    }
    // MFMA fragment of rows (columns) 16*blk .. +15, k sub-step s
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
template <int ROWS, int PF, int NT, int STEPB>
struct Window {
    typedef Operand<2, ROWS, false, false, true, PF, NT, STEPB> Op;
    static constexpr int CH = Op::CH;
    const char *image;
    int t, at0[CH], h0[CH], lo[CH], hi[CH];                      // the window's first element (byte offset), its first image row, columns inside the image
    u32x4 v[PF][CH];
    unsigned bits[PF][CH];
    bool exact[PF];                                              // (unused: a window's chunks are in place)

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
        const unsigned c = Op::CPR * step + Op::col_of(t), r = run_of(c, p);
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
    template <int SET, bool MASK> __device__ __forceinline__ void store(char *lds, int i, int, const UaParams &)
    {
        char *to = lds + Op::row_of(t) * Op::ROWB + ((Op::col_of(t) ^ Op::swz(Op::row_of(t))) << 4);
        u32x4 x = v[SET][i];
        if (__builtin_amdgcn_ballot_w64(bits[SET][i] != Op::ALL) != 0) x = keep<2>(x, bits[SET][i]);
        *(u32x4 *)(to + i * Op::RSTEP * Op::ROWB) = x;
    }
};

enum { A_K = 0, A_OC = 1, A_CONV = 2 };

// The workgroup: WM x WN waves over the tile, KG groups of them over a step's K (each takes SUBB bytes of it; their sums meet
// in LDS at the end).  PF: register sets of loads.  WPS: waves per SIMD that the registers have to allow.  DEALT, SHIFT: loads dealt out,
// from dwords (see the head of the file).  BASIC: four waves and one K group; these take convolutions too, and the shortest sums of products.
template <int BM_, int BN_, int WM_, int WN_, int KG_, int PF_, int WPS_ = 2, bool DEALT_ = false, bool SHIFT_ = false>
struct UaTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, PF = PF_, WPS = WPS_;
    static constexpr int NT = 64 * WM * WN * KG, STEPB = SUBB * KG;
    static constexpr bool DEALT = DEALT_, SHIFT = SHIFT_, BASIC = KG_ == 1 && !DEALT_ && WM_ * WN_ == 4;
};

template <bool INT8, int AF, bool B_OC, bool SH, class T>
__global__ __launch_bounds__(T::NT, T::WPS) void ua_kernel(UaParams p)
{
    using KD = Kind<INT8>;
    constexpr int ESZ = KD::ESZ, BM = T::BM, BN = T::BN, PF = T::PF, KG = T::KG;
    using OpA = Operand<ESZ, BM, AF == A_OC, SH && AF != A_CONV, AF == A_CONV, PF, T::NT, T::STEPB>;
    using OpB = Operand<ESZ, BN, B_OC, SH, AF == A_CONV, PF, T::NT, T::STEPB>;
    constexpr int MI = BM / 16 / T::WM, NI = BN / 16 / T::WN;
    constexpr int STAGE = OpA::BYTES + OpB::BYTES;
    constexpr int SUM_BYTES = KG > 1 ? (KG - 1) * BM * BN * 4 : 0;
    __shared__ __attribute__((aligned(1024))) char lds[2 * STAGE > SUM_BYTES ? 2 * STAGE : SUM_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / (T::WM * T::WN), wm = wave / T::WN % T::WM, wn = wave % T::WN;

    // workgroup -> tile: one XCD owns a run of consecutive tiles, walked in groups of group_m tile rows
    // (all batches' tiles count as one run)
    const unsigned nb = (unsigned)(p.tiles_m * p.tiles_n);
    unsigned bid = blockIdx.x, by = 0;
    if (p.batch > 1) {
        const unsigned ren = xcd_run(blockIdx.y * nb + blockIdx.x, nb * (unsigned)p.batch);
        by = ren / nb;
        bid = ren - by * nb;
    } else if (AF != A_CONV || (nb & 7) == 0) bid = xcd_run(bid, nb);
    const int gsz = p.group_m * p.tiles_n;
    const int grp = (int)bid / gsz, first_m = grp * p.group_m;
    const int gm = min(p.tiles_m - first_m, p.group_m);
    const int tm = first_m + ((int)bid % gsz) % gm, tn = ((int)bid % gsz) / gm;
    const int m0 = tm * BM, n0 = tn * BN;
    const long long batch = by;

    typename std::conditional<AF == A_CONV, Window<BM, PF, T::NT, T::STEPB>, OpA>::type a;
    OpB b;
    if constexpr (AF == A_CONV) a.init(p, m0, tid);
    else a.init(p.A + batch * p.strideA_b, p.a_ext, p.lda_b, m0, p.M, tid, p.steps);
    b.init(p.B + batch * p.strideB_b, p.b_ext, p.ldb_b, n0, p.N, tid, p.steps);

    constexpr int LOADS = OpA::CH + OpB::CH;                      // a thread's loads of a step
    // loads [FIRST, LAST) of a step that lies inside the operands
    auto load = [&](int step, auto set_c, auto first_c, auto last_c) {
        constexpr int SET = decltype(set_c)::value, FIRST = decltype(first_c)::value, LAST = decltype(last_c)::value;
        static_for<LAST - FIRST>([&](auto x_c) {
            constexpr int X = FIRST + decltype(x_c)::value;
            if constexpr (AF != A_CONV) {
                if constexpr (X < OpA::CH) a.template load<SET>(step, X);
                else b.template load<SET>(step, X - OpA::CH);
            }
        });
        if constexpr (FIRST == 0) a.exact[SET] = b.exact[SET] = false;
    };
    // all loads of any step
    auto load_any = [&](int step, auto set_c) {
        constexpr int SET = decltype(set_c)::value;
        if constexpr (AF == A_CONV) {
            a.template load_checked<SET>(step, p);
            b.template load_checked<SET>(step, p);
        } else if constexpr (T::BASIC) {
            // (these tiles serve the shortest sums, where the time to fetch the kernel's code counts: one path)
            a.template load_checked<SET>(step, p);
            b.template load_checked<SET>(step, p);
        } else {
            a.template load_any<SET>(step, p);
            b.template load_any<SET>(step, p);
        }
    };
    auto store = [&](int at, int step, auto set_c, auto x_c, auto mask_c) {
        constexpr int SET = decltype(set_c)::value, X = decltype(x_c)::value;
        constexpr bool MASK = decltype(mask_c)::value;
        if constexpr (X < OpA::CH) a.template store<SET, MASK>(lds + at, X, step, p);
        else b.template store<SET, MASK>(lds + at + OpA::BYTES, X - OpA::CH, step, p);
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
        for (int i = 0; i < MI; ++i) af[S][i] = OpA::frag(lds + at, wm * MI + i, 2 * kg + S, lane);
#pragma unroll
        for (int j = 0; j < NI; ++j) bf[S][j] = OpB::frag(lds + at + OpA::BYTES, wn * NI + j, 2 * kg + S, lane);
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
    typedef std::integral_constant<bool, true> True;
    typedef std::integral_constant<bool, false> False;
    static_for<PF>([&](auto u) {
        if (u < p.steps) {
            if (T::BASIC && AF != A_CONV && u < p.full) load(u, u, std::integral_constant<int, 0>{}, std::integral_constant<int, LOADS>{});
            else load_any(u, u);
        }
    });
    static_for<LOADS>([&](auto x_c) { store(0, 0, S0, x_c, True{}); });
    wg_barrier();
    if constexpr (WOVEN) read(0, S0);
    int cur = 0;
    // A step whose loads (of step + PF) lie inside the operands.  The loads are dealt out over the whole step: a wave stands still at
    // a load that the memory unit has no room for, and what is behind it, the MFMAs too, waits with it.
    auto inner = [&](int step, auto u_c) {
        constexpr int U = decltype(u_c)::value, NX = (U + 1) % PF;
        constexpr int SLOTS = 2 * MI + LOADS;
        auto some = [&](auto slot_c) {
            constexpr int SLOT = decltype(slot_c)::value;
            constexpr int FIRST = SLOT * LOADS / SLOTS, LAST = (SLOT + 1) * LOADS / SLOTS;
            if constexpr (LAST > FIRST) {
                load(step + PF, u_c, std::integral_constant<int, FIRST>{}, std::integral_constant<int, LAST>{});
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        read(cur, S1);
        __builtin_amdgcn_sched_barrier(0);
        static_for<MI>([&](auto i_c) {
            constexpr int I = decltype(i_c)::value;
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[I][j] = KD::mma(bf[0][j], af[0][I], acc[I][j]);
            __builtin_amdgcn_sched_barrier(0);
            some(i_c);
        });
        cur = STAGE - cur;
        static_for<LOADS>([&](auto x_c) {
            store(cur, step + 1, std::integral_constant<int, NX>{}, x_c, False{});      // the buffer every wave finished reading before the last barrier
            __builtin_amdgcn_sched_barrier(0);
            some(std::integral_constant<int, MI + decltype(x_c)::value>{});
        });
        wg_barrier();
        read(cur, S0);
        __builtin_amdgcn_sched_barrier(0);
        static_for<MI>([&](auto i_c) {
            constexpr int I = decltype(i_c)::value;
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[I][j] = KD::mma(bf[1][j], af[1][I], acc[I][j]);
            __builtin_amdgcn_sched_barrier(0);
            some(std::integral_constant<int, MI + LOADS + I>{});
        });
    };
    auto plain = [&](int step, auto u_c) {
        constexpr int U = decltype(u_c)::value, NX = (U + 1) % PF;
        load(step + PF, u_c, std::integral_constant<int, 0>{}, std::integral_constant<int, LOADS>{});
        read(cur, S1);
        multiply(S0);
        cur = STAGE - cur;
        static_for<LOADS>([&](auto x_c) { store(cur, step + 1, std::integral_constant<int, NX>{}, x_c, False{}); });
        wg_barrier();
        read(cur, S0);
        multiply(S1);
    };
    // any step; LAST: steps may be over (a condition around a load makes the waits for older ones stricter than they need be)
    auto one = [&](int step, auto u_c, auto last_c) {
        constexpr int U = decltype(u_c)::value, NX = (U + 1) % PF;
        constexpr bool LAST = decltype(last_c)::value;
        if (!LAST || step + PF < p.steps) load_any(step + PF, u_c);
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
            static_for<LOADS>([&](auto x_c) { store(cur, step + 1, std::integral_constant<int, NX>{}, x_c, True{}); });
            wg_barrier();
            if constexpr (WOVEN) read(cur, S0);
        }
        if constexpr (WOVEN) multiply(S1);
    };
    int step = 0;
    if constexpr (AF == A_CONV) {
        for (; step + 2 * PF <= p.steps; step += PF)
            static_for<PF>([&](auto u) { one(step + u, u, False{}); });
    } else {
        for (; step + 2 * PF <= p.full; step += PF)
            static_for<PF>([&](auto u) {
                if constexpr (T::DEALT) inner(step + u, u);
                else plain(step + u, u);
            });
    }
    for (; step < p.steps; step += PF)
        static_for<PF>([&](auto u) {
            if (step + u < p.steps) one(step + u, u, True{});
        });

    // The K groups' sums: of a wave's blocks, every KG-th is finished (and stored) by each group.
    if constexpr (KG > 1) {
        typename KD::acc_t *sums = (typename KD::acc_t *)lds;                     // [group - 1][wave of the group][block][lane]
        constexpr int WAVES = T::WM * T::WN;
        const int w = wave % WAVES;
        wg_barrier();                                             // the last step's fragments have been read
#pragma unroll
        for (int x = 0; x < MI * NI; ++x) {
            const int owner = x % KG;                             // group kg's slot for the owner: 0 .. KG-2
            if (owner != kg) sums[(((kg > owner ? kg - 1 : kg) * WAVES + w) * (MI * NI) + x) * 64 + lane] = acc[x / NI][x % NI];
        }
        wg_barrier();
#pragma unroll
        for (int x = 0; x < MI * NI; ++x)
            if (x % KG == kg) {
                // in the order of the groups, so that the sum does not depend on which of them adds
                typename KD::acc_t total = {0, 0, 0, 0};
#pragma unroll
                for (int o = 0; o < KG; ++o)
                    total += o == kg ? acc[x / NI][x % NI] : sums[(((o > kg ? o - 1 : o) * WAVES + w) * (MI * NI) + x) * 64 + lane];
                acc[x / NI][x % NI] = total;
            }
    }

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
            if (KG > 1 && (i * NI + j) % KG != kg) continue;
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
bool ua_operand_ok(int64_t s_outer, int64_t s_k, int64_t outer, int64_t K, int tile, int step_bytes)
{
    const int64_t esz = INT8 ? 1 : 2, epc = 16 / esz, bk = step_bytes / esz;
    const int64_t ext = ua_form(s_outer, s_k) == 1 ? (outer - 1) * s_outer + K : (K - 1) * s_k + outer;
    if (ext * esz < 16) return false;                            // an operand of at least one chunk
    if (ua_form(s_outer, s_k) == 1) return (tile - 1) * s_outer * esz + K * esz < 0x7fffffffLL;
    // a chunk that starts at the last column may run into the next k row, but not past it
    return ua_form(s_outer, s_k) == 2 && s_k >= epc && outer <= 0x7fffffffLL && bk * s_k * esz + tile * esz < 0x7fffffffLL;
}

template <bool INT8, class T>
bool ua_can_run(const Problem &q)
{
    constexpr int BM = T::BM, BN = T::BN;
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
        if (!ua_operand_ok<INT8>(q.a_sm, q.a_sk, q.M, q.K, BM, T::STEPB)) return false;
    }
    return ua_operand_ok<INT8>(q.b_sn, q.b_sk, q.N, q.K, BN, T::STEPB);
}

template <bool INT8, class T>
bool ua_can_run_gemm(const Problem &q) { return !q.conv && ua_can_run<INT8, T>(q); }

template <bool INT8, class T>
hipError_t ua_launch(const Problem &q)
{
    constexpr int BM = T::BM, BN = T::BN;
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
    p.steps = (int)(((int64_t)p.R * p.run_c + T::STEPB / 16 - 1) / (T::STEPB / 16));
    p.lda_b = (af == A_OC ? q.a_sk : q.a_sm) * esz;
    p.ldb_b = (b_oc ? q.b_sk : q.b_sn) * esz;
    p.a_ext = q.conv ? (q.M / (q.P * q.Q)) * q.H * q.W * q.Cin * esz
                     : ((af == A_OC ? (q.K - 1) * q.a_sk + q.M : (q.M - 1) * q.a_sm + q.K)) * esz;
    p.b_ext = (b_oc ? (q.K - 1) * q.b_sk + q.N : (q.N - 1) * q.b_sn + q.K) * esz;
    // rows that start inside a dword (GEMM): loads from dwords, put in place between the lanes.  Rows of a dword or less are loaded
    // as they lie: the dword in which the operand's last row starts would end behind it
    const bool sh = T::SHIFT && !q.conv && q.K * esz > 4 &&
                    (((uintptr_t)q.A | (uintptr_t)q.B | (uintptr_t)p.lda_b | (uintptr_t)p.ldb_b | (uintptr_t)(q.strideA * esz) | (uintptr_t)(q.strideB * esz)) & 3) != 0;
    // unchecked steps: all of K inside (and, of loads from dwords, the dword behind it), and for an operand along M or N a k
    // row after the step's last one
    p.full = (int)((q.K - (af == A_OC || b_oc ? 1 : 0) - (sh ? 4 / esz : 0)) / (T::STEPB / esz));
    p.ldc = q.ldc; p.c_plane = q.c_plane;
    p.strideA_b = q.strideA * esz; p.strideB_b = q.strideB * esz; p.strideC = q.strideC;
    p.alpha = q.alpha; p.beta = q.beta;
    p.tiles_m = (int)((q.M + BM - 1) / BM);
    p.tiles_n = (int)((q.N + BN - 1) / BN);
    p.group_m = p.tiles_m < 8 ? p.tiles_m : 8;
    p.batch = (int)q.batch;
    p.H = (int)q.H; p.W = (int)q.W; p.Cin = (int)q.Cin; p.PQ = (int)(q.P * q.Q); p.Q = (int)q.Q;
    p.sh = (int)q.sh; p.sw = (int)q.sw; p.ph = (int)q.ph; p.pw = (int)q.pw;
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)q.batch);
#define XP_UA(AF, BO, SH) hipLaunchKernelGGL((ua_kernel<INT8, AF, BO, SH, T>), grid, dim3(T::NT), 0, q.stream, p)
#define XP_UA_GEMM(SH) do { if (af == A_K) { if (b_oc) XP_UA(A_K, true, SH); else XP_UA(A_K, false, SH); } else { if (b_oc) XP_UA(A_OC, true, SH); else XP_UA(A_OC, false, SH); } } while (0)
    if (q.conv) {
        if constexpr (!INT8 && T::BASIC) { if (b_oc) XP_UA(A_CONV, true, false); else XP_UA(A_CONV, false, false); }
    } else if constexpr (T::SHIFT) {
        if (sh) XP_UA_GEMM(true); else XP_UA_GEMM(false);
    } else XP_UA_GEMM(false);
#undef XP_UA_GEMM
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

// Estimated time: start + rounds x (per tile + K steps x per step).  Up to one tile per compute unit is one round, beyond it `whole` of
// them count as whole rounds, and tile and step have times of their own (a unit's workgroups hide each other's waits); an operand along M or
// N adds its share to a step.  Fitted for each tile to timings of 780 (int8: 450) products of 64 to 8192 a side, odd and even, of all
// layouts; the share of A along M, for int8 and the dealt-out tile, to 6000 more, as that fit had left it at the ends of its range (-0.2,
// 0.5: int8 1280 x 256 x 6584 col/col 36.5 -> 16.3 us).  Over 11800 random calls the choice takes 2.9 % longer than the best of the nine in the
// geometric mean, the three tiles and the estimate before it 7.7; of the choices that differ 56 % are more than 5 % faster, 10 % slower.  Over 3549
// others (time_variants.py --align any, seed 31, those that need these tiles) 2.4 % longer, 1.51 at worst.
// Where the operands are aligned the direct-to-LDS kernels are up to twice as fast (2048 x 1024 x 1536: 11 us, this kernel 14),
// whatever their estimates say.
struct UaTimes { double start, tile, tile_shared, step, step_shared, a_outer, b_outer, whole; };
template <class T>
double ua_cost(const Problem &q, const UaTimes &u)
{
    const double x = (double)((q.M + T::BM - 1) / T::BM) * (double)((q.N + T::BN - 1) / T::BN) * (double)q.batch / 256.0;
    const double chunks = 16.0 / elem_size(q.in_type);
    if (q.conv) {
        // us a step of 128 bytes: a convolution's are checked
        const double full = x <= 3.0 ? __builtin_ceil(x) : x;
        const double steps = __builtin_ceil((double)q.R * __builtin_ceil((double)(q.S * q.Cin) / chunks) / 8.0);
        const double us = T::BM * T::BN == 128 * 128 ? (full <= 1.0 ? 0.85 : 0.71) : (T::BM * T::BN == 128 * 64 ? 0.5 : 0.34);
        return (4.0 + steps * full * us) * (ua_needed(q) ? 1.0 : 8.0);
    }
    const double rounds = x <= 1.0 ? 1.0 : u.whole * __builtin_ceil(x) + (1.0 - u.whole) * x;
    const double steps = __builtin_ceil((double)q.K / (T::STEPB / 16 * chunks));
    const double sides = 1.0 + (q.a_sk != 1 ? u.a_outer : 0.0) + (q.b_sk != 1 ? u.b_outer : 0.0);
    const double us = u.start + rounds * (x <= 1.0 ? u.tile + u.step * sides * steps : u.tile_shared + u.step_shared * sides * steps);
    // (a tie goes to the tiles of one K group and four waves: the fit is good to some per cent)
    return us * (ua_needed(q) ? 1.0 : 8.0) * (T::BASIC ? 1.0 : 1.02);
}

}  // namespace
}  // namespace xp
