// Convolution of few input channels (Table 5 of the paper: Conv2D NHWC): the first layer of a network, 7x7x3 with stride 2 or
// 3x3x3, whose whole filter window is a few chunks of 16 bytes.
//
// Bound: the output.  224 x 224 x 3 -> 112 x 112 x 64, 32 images, fp32: 103 MB written, 10 MB read, 7.6 GFLOP.  As an implicit
// GEMM every pixel's window is gathered from memory anew (seven times what the image holds) and masked chunk by chunk.
// Here a workgroup (4 waves) keeps the filter's MFMA fragments in registers and walks over tiles of a few output rows: the
// image rows a tile needs lie in LDS as they lie in memory, zeros where they leave the image, and a window is read from there:
// for a filter row the taps (s, c) of a pixel are one run of S*Cin consecutive elements, so a fragment's 8 k values are 16
// bytes at some even address.  K is R runs, each padded to whole chunks; what lies past a run is masked (it is the next pixels'
// data, which may be infinite).  The next tile's rows are requested before a tile is multiplied and go into the other LDS buffer
// after it.  Blocks are computed transposed: a lane stores four consecutive channels of a pixel.
//
// Measured (32 images): the general kernel 335 us, the any-alignment kernel 57, this one 29 (3.9 TB/s); without its stores 20,
// without its MFMAs 26.  No unit is the bound: of the time the matrix units are busy 13 %, the vector units 21 %, LDS 17 % (half of
// it conflicts of the window reads); a workgroup's staging, products and stores follow one another, and 448 workgroups of
// this call leave a fourth of the compute units with one instead of two.
#include "xp_internal.hpp"
#include "xp_any_align.hpp"
#include "xp_lds_tr.hpp"

namespace xp {
namespace {

constexpr int NT = 256;
constexpr int NB = 4;                     // blocks of 16 output channels per workgroup
constexpr int CH = 5;                     // chunks of a tile's image rows per thread
constexpr int LDS_CHUNKS = CH * NT;       // 20 KB a buffer

typedef unsigned int u32x4_dw __attribute__((ext_vector_type(4), aligned(4)));

struct FlParams {
    const char *image, *filter;
    float *out;
    long long image_b;                    // bytes of all images
    int filter_b, one_b;                  // bytes of the filter, of one image
    int H, W, Cin, Cout, P, Q, R, sh, sw, ph, pw;
    int run, run_c;                       // elements and chunks of a filter row's run
    unsigned run_magic, rc_magic;         // ceil(2^32 / run_c), ceil(2^32 / RC); 0 for a divisor of one
    int f_sk, f_sn;                       // filter strides (elements) along k and along the output channel
    int TP, GQ, RC;                       // tile: output rows, 16-pixel groups per row; chunks per image row in LDS
    int rows;                             // image rows per tile
    int tiles_p, tiles_q, tiles, per_wg;
};

__device__ __forceinline__ int divide(int n, unsigned magic) { return magic != 0u ? (int)__umulhi((unsigned)n, magic) : n; }

// load16_within with 32-bit offsets
__device__ __forceinline__ u32x4 load16_near(const char *base, int at, int first, int last)
{
    const int from = min(max(at, first), last - 16);
    if (__builtin_amdgcn_ballot_w64(from != at) != 0) return load16_within(base, at, first, last);
    return load16(base + from);
}

// KS: MFMA steps of four chunks; ODD: pixels lie an odd number of elements apart
template <int KS, bool ODD>
__global__ __launch_bounds__(NT, 2) void fl_kernel(FlParams p)
{
    __shared__ __attribute__((aligned(16))) char lds[2 * (LDS_CHUNKS + 2) * 16];      // (a window at the end may read a little past the rows)
    const int tid = threadIdx.x, lane = tid & 63, a = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = blockIdx.y * 16 * NB;
    const int pitch = p.RC * 16;
    const int px_shift = ODD ? 2 * ((a * p.sw * p.Cin) & 1) : 0; // bytes of the pixel's first element past a dword

    // the thread's chunks of a tile's image rows
    int c_row[CH], c_el[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int id = tid + NT * i;
        c_row[i] = divide(id, p.rc_magic);
        c_el[i] = 8 * (id - c_row[i] * p.RC);
    }
    u32x4 v[CH];
    unsigned bits[CH];
    struct Place { int n, p0, q0; };
    auto place = [&](int t) {
        Place x;
        x.n = t / (p.tiles_p * p.tiles_q);
        const int rest = t - x.n * p.tiles_p * p.tiles_q, tp = rest / p.tiles_q;
        x.p0 = tp * p.TP;
        x.q0 = (rest - tp * p.tiles_q) * p.GQ * 16;
        return x;
    };
    auto load = [&](const Place &x) {
        const int first = (x.q0 * p.sw - p.pw) * p.Cin, h0 = x.p0 * p.sh - p.ph;         // element in the image row, image row
        const long long before = (long long)x.n * p.one_b;
        const char *image = p.image + before;
        const int lowest = x.n > 0 ? -16 : 0, end = (int)min(p.image_b - before, (long long)p.one_b + 16);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int el = first + c_el[i], h = h0 + c_row[i];
            const int lo = min(max(-el, 0), 8), hi = min(max(p.W * p.Cin - el, 0), 8);
            const bool inside = c_row[i] < p.rows && (unsigned)h < (unsigned)p.H && lo < hi;
            bits[i] = inside ? ((1u << hi) - 1) & ~((1u << lo) - 1) : 0u;
            v[i] = load16_near(image, inside ? (h * p.W * p.Cin + el) * 2 : lowest, lowest, end);
        }
    };
    auto store = [&](char *to) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            u32x4 w = v[i];
            if (__builtin_amdgcn_ballot_w64(bits[i] != 0xffu) != 0) w = keep<2>(w, bits[i]);
            *(u32x4 *)(to + (tid + NT * i) * 16) = w;
        }
    };

    const int t0 = blockIdx.x * p.per_wg, t1 = min(t0 + p.per_wg, p.tiles);
    if (t0 >= t1) return;                                        // the whole workgroup
    constexpr int BUF = (LDS_CHUNKS + 2) * 16;
    Place x = place(t0);
    load(x);

    // The filter's fragments by way of LDS: 64 channels x 4 KS chunks, each loaded once by the workgroup.  (Every lane loading
    // its fragments itself is four times the loads, and their edge cases four times the code: 5 us before the first tile.)
    constexpr int FC = 4 * KS, FCH = FC * 16 * NB / NT;
    static_assert(FC * 16 * NB * 16 <= 2 * BUF, "the filter fits the tile buffers");
    u32x4 fv[FCH];
#pragma unroll
    for (int i = 0; i < FCH; ++i) {
        const int id = tid + NT * i, c = id % FC, co = min(c0 + id / FC, p.Cout - 1);
        const int r = divide(c, p.run_magic), e0 = 8 * (c - r * p.run_c), n = r < p.R ? min(p.run - e0, 8) : 0, k_at = r * p.run + e0;
        if (p.f_sk == 1) {
            fv[i] = load16_near(p.filter, n > 0 ? (co * p.f_sn + k_at) * 2 : 0, 0, p.filter_b);
        } else {
            fv[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < n) fv[i][e >> 1] |= (unsigned)((const unsigned short *)p.filter)[(k_at + e) * p.f_sk + co * p.f_sn] << (16 * (e & 1));
        }
    }
    // (a chunk's 64 channels one after the other; fragments are read 16 channels at a time)
#pragma unroll
    for (int i = 0; i < FCH; ++i) {
        const int id = tid + NT * i;
        *(u32x4 *)(lds + (id % FC * 16 * NB + id / FC) * 16) = fv[i];
    }
    // this lane's chunk of every step: where in the window, which of its elements count
    int at[KS];
    u32x4 mask[KS], ff[KS][NB];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int c = 4 * s + g, r = divide(c, p.run_magic), e0 = 8 * (c - r * p.run_c);
        const int n = r < p.R ? min(p.run - e0, 8) : 0;
        at[s] = n > 0 ? r * pitch + e0 * 2 + a * p.sw * p.Cin * 2 : px_shift;
        mask[s] = keep<2>(u32x4{~0u, ~0u, ~0u, ~0u}, (1u << n) - 1);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < NB; ++j) ff[s][j] = *(const u32x4 *)(lds + ((4 * s + g) * 16 * NB + 16 * j + a) * 16) & mask[s];
    __syncthreads();
    store(lds);
    __syncthreads();
    int cur = 0;
    for (int t = t0; t < t1; ++t) {
        const Place nx = place(t + 1);
        if (t + 1 < t1) load(nx);
        for (int gi = wave; gi < p.TP * p.GQ; gi += NT / 64) {
            const int pr = gi / p.GQ, gq = gi - pr * p.GQ;
            const int oy = x.p0 + pr;
            if (oy >= p.P || x.q0 + 16 * gq >= p.Q) continue;    // (uniform)
            const char *from = lds + cur + pr * p.sh * pitch + gq * 16 * p.sw * p.Cin * 2;
            f32x4 acc[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                u32x4 px;
                if constexpr (ODD) {
                    const char *src = from + at[s] - px_shift;
                    const u32x4 w = *(const u32x4_dw *)src;
                    const unsigned fifth = *(const unsigned *)(src + 16);
                    px = u32x4{__builtin_amdgcn_alignbyte(w[1], w[0], px_shift), __builtin_amdgcn_alignbyte(w[2], w[1], px_shift),
                               __builtin_amdgcn_alignbyte(w[3], w[2], px_shift), __builtin_amdgcn_alignbyte(fifth, w[3], px_shift)};
                } else {
                    px = *(const u32x4_dw *)(from + at[s]);
                }
                px &= mask[s];
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = Kind<false>::mma(ff[s][j], px, acc[j]);
            }
            // (plain stores: as non-temporal ones, whose 64 bytes a pixel are not joined to lines in the L2, the first layer took
            // 44.6 us instead of 36.2; whole lines gathered through LDS were no faster, 38.4)
            const int ox = x.q0 + 16 * gq + a;
            if (ox < p.Q) {
                float *dst = p.out + (((long long)x.n * p.P + oy) * p.Q + ox) * p.Cout + c0 + 4 * g;
                typedef float out4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int co = c0 + 16 * j + 4 * g;
                    if (co + 4 <= p.Cout) *(out4_any *)(dst + 16 * j) = acc[j];
                    else
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (co + e < p.Cout) dst[16 * j + e] = acc[j][e];
                }
            }
        }
        cur = BUF - cur;
        if (t + 1 < t1) store(lds + cur);                        // the buffer every wave finished reading before the last barrier
        __syncthreads();
        x = nx;
    }
}

// ------------------------------------------------------------------------------------ host side

struct FlTile { int TP, GQ, RC, rows, steps; };

// The tile: whole output rows (or equal parts of them) whose image rows fit the LDS buffer; four rows, so that every wave has
// the same work, unless that leaves compute units without a tile.
bool fl_tile(const Problem &q, FlTile *t)
{
    const int64_t run = q.S * q.Cin, run_c = (run + 7) / 8;
    t->steps = (int)((q.R * run_c + 3) / 4);
    if (t->steps > 8) return false;
    const int64_t groups = (q.Q + 15) / 16;
    for (int64_t parts = 1; parts <= groups; ++parts) {
        const int64_t gq = (groups + parts - 1) / parts;
        const int64_t rc = ((16 * gq - 1) * q.sw * q.Cin + 8 * run_c + 7) / 8;
        for (int tp = 4; tp >= 1; tp /= 2) {
            const int64_t rows = (tp - 1) * q.sh + q.R;
            if (rows * rc > LDS_CHUNKS) continue;
            const int64_t tiles = (q.M / (q.P * q.Q)) * ((q.P + tp - 1) / tp) * parts;
            if (tp > 1 && tiles * ((q.N + 63) / 64) < 512) continue;
            t->TP = tp; t->GQ = (int)gq; t->RC = (int)rc; t->rows = (int)rows;
            return true;
        }
    }
    return false;
}

bool fl_can_run(const Problem &q)
{
    if (q.in_type != XP_BF16 || !q.conv || q.c_plane || q.K <= 0 || q.beta != 0.0f || q.alpha != 1.0f) return false;
    if (q.M > 0x3fffffffLL || q.N > 0xfffffLL || q.S * q.Cin > 0xffff || q.R > 0xffff || q.sh > 0xfff || q.sw > 0xfff) return false;
    const int64_t images = q.M / (q.P * q.Q);
    if (images * q.H * q.W * q.Cin * 2 < 16 || q.N * q.K * 2 < 16) return false;       // tensors of at least one chunk
    if ((q.W + 2 * q.pw + q.S) * q.Cin >= 0x3fffffffLL || q.H + 2 * q.ph >= 0x3fffffffLL || q.N * q.K >= 0x3fffffffLL) return false;
    if (q.H * q.W * q.Cin >= 0x3ffffff0LL || q.H * q.W * q.Cin * 2 < 32) return false;       // 32-bit offsets inside an image, neighbours' chunks included
    FlTile t;
    return fl_tile(q, &t);
}

hipError_t fl_launch(const Problem &q)
{
    FlTile t;
    if (!fl_tile(q, &t)) return hipErrorInvalidValue;
    FlParams p;
    const int64_t images = q.M / (q.P * q.Q);
    p.image = (const char *)q.A; p.filter = (const char *)q.B; p.out = (float *)q.C;
    p.image_b = images * q.H * q.W * q.Cin * 2; p.filter_b = (int)(q.N * q.K * 2); p.one_b = (int)(q.H * q.W * q.Cin * 2);
    p.H = (int)q.H; p.W = (int)q.W; p.Cin = (int)q.Cin; p.Cout = (int)q.N; p.P = (int)q.P; p.Q = (int)q.Q; p.R = (int)q.R;
    p.sh = (int)q.sh; p.sw = (int)q.sw; p.ph = (int)q.ph; p.pw = (int)q.pw;
    p.run = (int)(q.S * q.Cin); p.run_c = (p.run + 7) / 8;
    p.run_magic = p.run_c == 1 ? 0u : (unsigned)(((1ull << 32) + p.run_c - 1) / p.run_c);
    p.rc_magic = t.RC == 1 ? 0u : (unsigned)(((1ull << 32) + t.RC - 1) / t.RC);
    p.f_sk = (int)q.b_sk; p.f_sn = (int)q.b_sn;
    p.TP = t.TP; p.GQ = t.GQ; p.RC = t.RC; p.rows = t.rows;
    p.tiles_p = (int)((q.P + t.TP - 1) / t.TP);
    p.tiles_q = (int)((q.Q + 16 * t.GQ - 1) / (16 * t.GQ));
    p.tiles = (int)(images * p.tiles_p * p.tiles_q);
    const int blocks_n = (int)((q.N + 16 * NB - 1) / (16 * NB));
    // two workgroups per compute unit, each walking over neighbouring tiles
    const int wgs = blocks_n >= 512 ? 1 : 512 / blocks_n;
    p.per_wg = (p.tiles + wgs - 1) / wgs;
    const dim3 grid((unsigned)((p.tiles + p.per_wg - 1) / p.per_wg), (unsigned)blocks_n);
    const bool odd = ((q.sw * q.Cin) & 1) != 0;
#define XP_FL(KS)                                                                                      \
    do {                                                                                               \
        if (odd) hipLaunchKernelGGL((fl_kernel<KS, true>), grid, dim3(NT), 0, q.stream, p);            \
        else hipLaunchKernelGGL((fl_kernel<KS, false>), grid, dim3(NT), 0, q.stream, p);               \
    } while (0)
    if (t.steps <= 2) XP_FL(2);
    else if (t.steps <= 4) XP_FL(4);
    else if (t.steps <= 6) XP_FL(6);
    else XP_FL(8);
#undef XP_FL
    return hipGetLastError();
}

// Below 8 channels it is the choice from about 90000 output pixels on: up to there its start, some 5 us for the filter and the
// first tile, costs more than the reuse saves (both sides timed over 1800 calls; pixels, time here over that of the any-alignment
// kernel: 8000 1.2 .. 1.3, 50000 1.3, 80000 .. 100000 0.93 .. 1.04, 130000 0.64 .. 1.0; 247000 22 us and 39, the first layer's
// 401408 29 and 56, 516128 17 and 40), above 128 output channels from 50000 on (75264 x 448 30 us and 43, 20000 1.3).  A filter
// along its output channels is gathered element by element at the start and takes twice as many.  Four output rows or fewer
// leave waves of a tile without work, and long rows of few elements leave few tiles: there it takes 250000 pixels and a
// tile for every compute unit (47 x 1 x 27594 x 6 -> 8, 5 taps 24 us and 48, but
// 2 x 1 x 7427 x 1 -> 128, 15 taps, a tile per image, 56 and 6.3, 14 x 1 x 33664 x 1 -> 16, one tap, 67 and 36).  Where the any-alignment
// kernel declines (fewer than 8 channels, filter along them) the other side is the general kernel: 0.2 .. 0.85 of its time
// but for few rows and short filters.  The estimate is the output at a rate above any that others are priced at.
double fl_cost(const Problem &q)
{
    if (q.Cin >= 8) return 1e30;
    bool chosen;
    if (q.b_sk != 1 && q.N < 8) {
        chosen = q.P > 4 || q.K >= 24;
    } else if (q.P > 4) {
        chosen = q.M >= (q.N > 128 ? 50000 : 90000) * (q.b_sk == 1 ? 1 : 2);
    } else {
        FlTile t;
        chosen = q.M >= 250000 && fl_tile(q, &t) && q.M / (q.P * q.Q) * ((q.P + t.TP - 1) / t.TP) * ((q.Q + 16 * t.GQ - 1) / (16 * t.GQ)) *
                 ((q.N + 16 * NB - 1) / (16 * NB)) >= 256;
    }
    return chosen ? 3.0 + (double)q.M * (double)q.N * 4.0 / 16.0e6 : 1e30;
}

const Variant kFl = {"bf16 few input channels, image rows in LDS, filter in registers, mfma16", fl_can_run, fl_launch, fl_cost};

}  // namespace

int fl_variants(xp_dtype in_type, const Variant **out)
{
    if (in_type != XP_BF16) return 0;
    out[0] = &kFl;
    return 1;
}

}  // namespace xp
