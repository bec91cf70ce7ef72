// UNet convolutions as implicit GEMM on the CDNA4 matrix cores (FP32).
//
// The UNet of Section 2 (arXiv:2602.19959) is a stack of 1D convolutions.
// Each is a GEMM  D[m][n] = sum_k A[m][k] B[k][n]  with
//   m = (event, position)  rows of the channels-last activation,
//   n = output channel     (transposed conv: (tap, output channel)),
//   k = (tap, input channel).
//
// FP32 operands on the BF16 matrix instructions: an FP32 value is the exact
// sum of three BF16 values (8 + 8 + 8 significant bits, each piece the nearest
// BF16 of what the pieces before it leave), so a product of two FP32 values
// is nine BF16 products.  Six of them are accumulated in FP32,
//   hi*hi, hi*mid, mid*hi, mid*mid, hi*lo, lo*hi;
// the three left out add up to at most 2^-24 of the product, half an ulp of it.
// The five small ones of a step (32 channels of one tap) are summed apart and
// added to the accumulator once, so that it is rounded by one of the six
// instructions and one addition instead of by all six.  Measured error against
// FP64, relative 2-norm of p over 48 drawn calls (both widths and layouts, 1 to
// 20 events), root mean square and largest: 2.6e-7 and 5.4e-7, against 6.2e-7 and
// 1.2e-6 with the FP32 instruction and 5.3e-7 and 1.2e-6 with all six in one
// chain; call by call 0.42 of the FP32 instruction's error on average and at most
// 0.54 (one chain: 0.84 and 1.1).  The additions cost 4% to 5% of the time: 1000
// events 9.08 -> 9.55 ms.
// v_mfma_f32_16x16x4_f32 runs at 157 TFLOP/s dense, the BF16 form at 2.5
// PFLOP/s, so six of those are 2.65 times as fast as one FP32 instruction.
// Activations stay FP32 in HBM and are split while they are staged; the weights
// are split once, at set-up.  Bound by the matrix rate at the card's sustained
// clock: at 1000 events enc3.c2 takes 1.38 ms, 237 TFLOP/s of FP32 work or 1.42
// PFLOP/s of BF16 (2.37 ms and 138 TFLOP/s with the FP32 instruction, 86% of its
// peak), the whole network 9.6 ms (15.0 ms).
//
// A is never materialised: a block stages the (BM + 4) x 32 halo tile of input
// rows once per 32-channel chunk in LDS, as three BF16 planes, and all five
// taps read it with a row shift.
//
// MFMA: v_mfma_f32_16x16x32_bf16.  Lane group g = lane/16 supplies channels
// 8 g .. 8 g + 7 of the chunk, for the weights and the rows alike.  The k
// order of every output (chunk, tap, product, MFMA) is fixed by the kernel
// alone, never by the tile's position or shape, so results are bitwise
// independent of the batch size, of where an event sits in it and of the
// tile-shape variant.
//
// Epilogues (fused, nothing re-read from HBM):
//   EPI_STORE  bias + LeakyReLU
//   EPI_POOL   bias + LeakyReLU, plus the width-2 max-pool of row pairs into
//              the next level's input
//   EPI_CONVT  stride-2 2-tap transposed conv: row t of the coarse level goes
//              to rows 2t and 2t+1 of the fine level, bias, no activation
//   EPI_HEAD   bias + LeakyReLU, then the 1x1 head over all channels and the
//              sigmoid, writing the per-bin probability
// Guard rows (the two zero rows before and after each event) are never written.
//
// conv_mfma_f32_first runs enc0.c2 with the first convolution (one input
// channel, five taps) computed in its halo staging from the histogram rows,
// so that 32-channel tensor never goes through HBM.
#include <cmath>

#include "pvf_internal.h"

namespace pvf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int KC = 32;         // input channels per stage
constexpr int FRAG = 1024;     // bytes of one packed weight fragment: 16 columns x 32 channels of one piece

__device__ __forceinline__ float lrelu(float x, float s) { return x >= 0.f ? x : s * x; }

// the products that are accumulated, smallest first: (weight piece, row piece), 0 = hi
constexpr int kF32Products = 6;
constexpr int kProd[kF32Products][2] = {{0, 2}, {1, 1}, {2, 0}, {0, 1}, {1, 0}, {0, 0}};

// The top of FP32's range.  Values from kBf16Cut on round to infinity in BF16;
// and where hi*hi overflows, as FP32 does there, a smaller product of a rounded
// piece may overflow to the other sign, a sum of NaN.  Pieces that are cut off
// instead of rounded have the value's own sign.  Row values are cut off where
// their products may reach 2^127, w_sum being the layer's largest sum of
// |weight| over an output channel (f32_split_cut).  Weights are rounded where
// that sum is at most kRoundSum: their smaller pieces' products are below 2^-8
// of theirs, so they stay below 2^127 over finite rows; else they are cut off
// too.  (Sums within 2^-7 of FP32's largest value may round up to infinity.
// Products left out reach 2^-22 with one operand cut off, 2^-21 with both; the
// measured error of p with every weight cut off is that of rounded ones, 0.42.)
constexpr float kBf16Cut = 0x1.ffp127f;
constexpr float kRoundSum = 0x1p7f;

// Epilogue shared by the FP32 kernels, straight from the accumulators.  The
// kernels issue the MFMA as D^T = W X^T (weight fragment in the A slot), so
// lane (li, lg) of a 16 x 16 tile holds channels 4 lg + v (v = 0..3) of tile
// row li: four consecutive outputs of one position, one 16-byte store.
template <int WM, int TMW, int TNW, int EPI>
__device__ __forceinline__ void f32_epilogue(const f32x4 (&acc)[TMW][TNW], const ConvArgs& a, int64_t m0, int n0,
                                             int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lg = lane >> 4;
    const int rw = (wave % WM) * TMW * 16;
    const int cbase = n0 + (wave / WM) * TNW * 16 + 4 * lg;   // this lane's first channel of tile j = 0
    const RowMap rows(m0, a.r_in);
    float* out = static_cast<float*>(a.out);
    float* pout = static_cast<float*>(a.pool_out);

    if constexpr (EPI == EPI_HEAD) {
        // the block holds every channel of its rows (BN == n, one wave in N)
#pragma unroll
        for (int i = 0; i < TMW; ++i) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < TNW; ++j) {
                const int c = cbase + j * 16;
#pragma unroll
                for (int v = 0; v < 4; ++v) s += lrelu(acc[i][j][v] + a.bias[c + v], a.slope) * a.head_w[c + v];
            }
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            const int t = rw + i * 16 + li;
            if (lg == 0 && m0 + t < a.m_rows) {
                int64_t e;
                int loc;
                rows.at(t, e, loc);
                if (loc >= kGuard && loc < a.r_in - kGuard)
                    a.prob[e * a.l_out + (loc - kGuard)] = 1.f / (1.f + expf(-(s + a.head_b)));
            }
        }
        return;
    }

#pragma unroll
    for (int i = 0; i < TMW; ++i) {
        const int t = rw + i * 16 + li;
        int64_t e;
        int loc;
        rows.at(t, e, loc);
        const bool ok = m0 + t < a.m_rows && loc >= kGuard && loc < a.r_in - kGuard;
#pragma unroll
        for (int j = 0; j < TNW; ++j) {
            const int c = cbase + j * 16;
            const bool col_ok = c < a.n;            // n % 4 == 0: a lane's four channels are all in or all out
            const int cc = col_ok ? c : 0;
            if constexpr (EPI == EPI_CONVT) {
                const int tj = cc / a.cout;          // which of the two output rows
                const int o = cc - tj * a.cout;
                f32x4 y;
#pragma unroll
                for (int v = 0; v < 4; ++v) y[v] = acc[i][j][v] + a.bias[o + v];
                if (ok && col_ok) {
                    const int64_t ro = e * a.r_out + kGuard + 2 * (loc - kGuard) + tj;
                    *reinterpret_cast<f32x4*>(out + ro * a.ld_out + o) = y;
                }
            } else {
                f32x4 y;
#pragma unroll
                for (int v = 0; v < 4; ++v) y[v] = lrelu(acc[i][j][v] + a.bias[cc + v], a.slope);
                if (ok && col_ok) *reinterpret_cast<f32x4*>(out + (m0 + t) * a.ld_out + c) = y;
                if constexpr (EPI == EPI_POOL) {
                    // rows per event and the guard are even, so an even row is
                    // the first of a pooling pair; its partner is lane li ^ 1
                    f32x4 p;
#pragma unroll
                    for (int v = 0; v < 4; ++v) p[v] = fmaxf(y[v], __shfl_xor(y[v], 1));
                    if (ok && col_ok && (li & 1) == 0) {
                        const int64_t rp = e * a.r_pool + kGuard + (loc - kGuard) / 2;
                        *reinterpret_cast<f32x4*>(pout + rp * a.ld_pool + c) = p;
                    }
                }
            }
        }
    }
}

// Eight FP32 values as three planes of eight BF16 values; the pieces add up
// to the value exactly (24 significant bits; below 2^-103 the last piece
// loses bits to BF16's subnormals).  From `cut` on they are cut off instead of
// rounded.  An infinity is (0, 0, infinity): its last piece meets only the
// weight's first, so its product has the right sign.
__device__ __forceinline__ void split8(const f32x4& x0, const f32x4& x1, float cut, u32x4 (&p)[kF32Pieces])
{
    float most = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)    // fmaxf would first quiet every operand, twice the instructions
        asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(x0[k]), "v"(x1[k]));
    if (__builtin_expect(most >= cut, 0)) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float x = k < 4 ? x0[k & 3] : x1[k & 3];
            const bool large = fabsf(x) >= cut, inf = isinf(x);
            float r = x;
#pragma unroll
            for (int q = 0; q < kF32Pieces; ++q) {
                float y = large ? __builtin_bit_cast(float, __builtin_bit_cast(unsigned, r) & 0xffff0000u) : (float)(__bf16)r;
                if (inf) y = q + 1 < kF32Pieces ? 0.f : x;
                r -= y;
                const unsigned u = __builtin_bit_cast(unsigned, y);
                p[q][k >> 1] = k & 1 ? p[q][k >> 1] | (u & 0xffff0000u) : u >> 16;
            }
        }
        return;
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        f32x2 r = h < 2 ? f32x2{x0[2 * h], x0[2 * h + 1]} : f32x2{x1[2 * h - 4], x1[2 * h - 3]};
#pragma unroll
        for (int q = 0; q < kF32Pieces; ++q) {
            const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
            p[q][h] = u;
            if (q + 1 < kF32Pieces) {
                r[0] -= __builtin_bit_cast(float, u << 16);
                r[1] -= __builtin_bit_cast(float, u & 0xffff0000u);
            }
        }
    }
}

// Set-up: weights [n][taps][cin] -> per 32-channel chunk, tap, group of 16
// columns and piece one 1 KB fragment, in which lane l holds channels
// 8 (l / 16) .. + 7 of column l % 16.  One thread per lane of a fragment group.
__global__ __launch_bounds__(256) void split_weights(const float* w, int n, int taps, int cin, float cut, uint16_t* pieces)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int lane = t & 63, group = t >> 6;           // group = (chunk * taps + tap) * (n / 16) + column group
    if (group >= n / 16 * taps * (cin / KC)) return;
    const int cg = group % (n / 16), step = group / (n / 16);
    const int tap = step % taps, chunk = step / taps;
    const f32x4* src = reinterpret_cast<const f32x4*>(w + ((int64_t)(16 * cg + lane % 16) * taps + tap) * cin +
                                                      KC * chunk + 8 * (lane / 16));
    u32x4 p[kF32Pieces];
    split8(src[0], src[1], cut, p);
#pragma unroll
    for (int q = 0; q < kF32Pieces; ++q)
        *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(pieces) + ((int64_t)group * kF32Pieces + q) * FRAG + lane * 16) = p[q];
}

// LDS rows of a halo plane: at least `rows`, and 2 modulo 8, so that the four
// planes of a piece start 32 bytes apart modulo 128 and the staging stores of
// two rows x four planes fall on different banks.
constexpr int plane_rows(int rows) { return (rows + 5) / 8 * 8 + 2; }

// LDS of a block: XB halo buffers of three pieces x four 8-channel planes
// (16 bytes per row and plane: the fragment reads of 16 rows are contiguous),
// and a ring of D weight buffers of one (chunk, tap) step each.
template <int BM, int BN, int XB, int D, int TAPS> struct F32Lds {
    static constexpr int rows = plane_rows(BM + TAPS - 1);
    static constexpr int x = kF32Pieces * 4 * rows * 16;
    static constexpr int w = BN / 16 * kF32Pieces * FRAG;
    static constexpr int v = XB * x + D * w;
};
// Waves per SIMD handed to the register allocator: what the LDS allows on one
// CU (160 KB), at most 2 for the 4 x 4-tile waves (64 accumulator and 80
// fragment and partial-sum registers), 4 for the others.
template <int WM, int WN, int TMW, int TNW, int XB, int D, int TAPS> struct F32Occ {
    static constexpr int w = (163840 / F32Lds<WM * TMW * 16, WN * TNW * 16, XB, D, TAPS>::v * WM * WN + 3) / 4;
    static constexpr int most = TMW * TNW >= 16 ? 2 : 4;
    static constexpr int v = w < 1 ? 1 : w > most ? most : w;
};

// FC: enc0.c2 with the first convolution fused into the staging: each halo
// chunk is computed from five histogram rows (first_conv_at, the operation
// order of the standalone kernel, so the bits match) instead of read back;
// guard rows are zero, as in the stored tensor.
template <int WM, int WN, int TMW, int TNW, int XB, int D, int TAPS, int EPI, bool FC>
__device__ __forceinline__ void conv_f32_tile(const ConvArgs& a)
{
    static_assert(!FC || (TAPS == kTaps && XB == 1), "the fused first convolution feeds a 5-tap, single-buffered tile");
    constexpr int NW = WM * WN;
    constexpr int NT = NW * 64;
    constexpr int BM = WM * TMW * 16;
    constexpr int BN = WN * TNW * 16;
    constexpr int RAD = (TAPS - 1) / 2;
    constexpr int XROWS = BM + TAPS - 1;
    using Lds = F32Lds<BM, BN, XB, D, TAPS>;
    constexpr int PLANE = Lds::rows * 16;         // bytes
    constexpr int WI = Lds::w / FRAG;             // 1 KB loads per weight step

    __shared__ __attribute__((aligned(16))) char smem[Lds::v];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM;
    const int wn = wave / WM;
    const int li = lane & 15;
    const int lg = lane >> 4;

    // XCD-aware tile order: block b runs on XCD b % 8; every N tile of one M
    // tile goes to the same XCD back to back, so the halo rows (and the
    // weights) are served from that XCD's L2 instead of HBM.
    const int n_tiles = a.n / BN;
    const int m_tiles = (a.m_rows + BM - 1) / BM;
    const int xcd = (int)(blockIdx.x % kXcds), slot = (int)(blockIdx.x / kXcds);
    const int m_tile = (slot / n_tiles) * kXcds + xcd;
    if (m_tile >= m_tiles) return;
    const int64_t m0 = (int64_t)m_tile * BM;
    const int n0 = (slot % n_tiles) * BN;
    const float* in = static_cast<const float*>(a.in);
    const char* wt = static_cast<const char*>(a.w) + (int64_t)n0 / 16 * kF32Pieces * FRAG;
    const int64_t wstep = (int64_t)a.n / 16 * kF32Pieces * FRAG;    // bytes of one (chunk, tap) step, all columns

    // column tiles at a time: 2 x 4-tile waves have registers for one at four
    // waves a SIMD (12 spilled with two, 130 MB of HBM writes a launch at 1000 events)
    constexpr int JG = TMW * TNW == 8 && TNW == 4 ? 1 : 2;
    f32x4 acc[TMW][TNW];
#pragma unroll
    for (int i = 0; i < TMW; ++i)
#pragma unroll
        for (int j = 0; j < TNW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Halo staging: a thread owns 8 channels (octet tid % 4) of rows tid / 4 +
    // u * NT / 4.  Rows outside the batch are clamped to valid ones: they only
    // feed outputs that the epilogue discards.
    constexpr int RS = NT / 4;
    constexpr int XPT = (XROWS + RS - 1) / RS;
    const int oct = tid & 3, row0 = tid >> 2;
    auto x_has = [&](int u) __attribute__((always_inline)) { return (u + 1) * RS <= XROWS || row0 + u * RS < XROWS; };
    auto x_row = [&](int u) __attribute__((always_inline)) {
        const int64_t g = m0 - RAD + min(row0 + u * RS, XROWS - 1);
        return g < 0 ? (int64_t)0 : (g >= a.m_rows ? (int64_t)a.m_rows - 1 : g);
    };
    f32x4 xr[FC ? 1 : XPT][2];
    auto x_fetch = [&](int c0) __attribute__((always_inline)) {
        if constexpr (!FC) {
#pragma unroll
            for (int u = 0; u < XPT; ++u)
                if (D > 2 || x_has(u)) {               // without a branch where the waits are counted
                    const f32x4* p = reinterpret_cast<const f32x4*>(in + x_row(u) * a.ld_in + c0 + 8 * oct);
                    xr[u][0] = p[0];
                    xr[u][1] = p[1];
                }
        }
    };
    auto x_put = [&](char* xs, int u, const f32x4& y0, const f32x4& y1) __attribute__((always_inline)) {
        u32x4 p[kF32Pieces];
        split8(y0, y1, a.split_cut, p);
#pragma unroll
        for (int q = 0; q < kF32Pieces; ++q)
            *reinterpret_cast<u32x4*>(xs + (q * 4 + oct) * PLANE + (row0 + u * RS) * 16) = p[q];
    };
    auto x_store = [&](int buf, int c0) __attribute__((always_inline)) {
        char* xs = smem + buf * Lds::x;
        if constexpr (FC) {
            const int c = c0 + 8 * oct;               // this thread's 8 channels
            const RowMap rmap(m0, a.r_in);
            float fw[8][kTaps], fb[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                fb[v] = a.first_b[c + v];
#pragma unroll
                for (int j = 0; j < kTaps; ++j) fw[v][j] = a.first_w[(c + v) * kTaps + j];
            }
#pragma unroll
            for (int u = 0; u < XPT; ++u) {
                if (!x_has(u)) continue;
                const int64_t g = x_row(u);
                int64_t e;
                int loc;
                rmap.at((int)(g - m0), e, loc);
                f32x4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                if (loc >= kGuard && loc < a.r_in - kGuard) {
                    float x[kTaps];
#pragma unroll
                    for (int j = 0; j < kTaps; ++j) x[j] = a.first_x0[g + j - kGuard];
#pragma unroll
                    for (int v = 0; v < 8; ++v) y[v / 4][v % 4] = first_conv_at(fw[v], fb[v], x, a.slope);
                }
                x_put(xs, u, y[0], y[1]);
            }
        } else {
            (void)c0;
#pragma unroll
            for (int u = 0; u < XPT; ++u)
                if (x_has(u)) x_put(xs, u, xr[u][0], xr[u][1]);
        }
    };
    // Weights of step g: WI fragments of 1 KB, contiguous, straight into LDS
    // in the order the waves read them.
    auto w_issue = [&](int g, int slot) __attribute__((always_inline)) {
        const char* src = wt + g * wstep;
        char* dst = smem + XB * Lds::x + slot * Lds::w;
#pragma unroll
        for (int t = 0; t < (WI + NW - 1) / NW; ++t) {
            const int j = wave + t * NW;
            if ((t + 1) * NW <= WI || j < WI)
                __builtin_amdgcn_global_load_lds((const void*)(src + j * FRAG + lane * 16),
                                                 (__attribute__((address_space(3))) void*)(dst + j * FRAG), 16, 0, 0);
        }
    };

    const int nc = a.cin / KC, nk = nc * TAPS;
    // The barrier that opens step g: this wave's share of step g has arrived
    // and its halo stores are done; the loads of steps g + 1 .. g + D - 2, at
    // least WI / NW each, may still be in flight (halo loads among them, and
    // the waves that issue one more a step, only make the wait longer).
    // With D > 2, steps past the last one are issued too, as copies of the
    // last, so that the count always holds; nothing reads them.
    auto open = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((D - 2) * (WI / NW)) : "memory");
    };
#pragma unroll
    for (int g = 0; g < D - 1; ++g) w_issue(min(g, nk - 1), g);
    x_fetch(0);
    x_store(0, 0);
    int ring = 0;                                  // ring slot of step g
    for (int c = 0; c < nc; ++c) {
        const char* xs = smem + (XB == 2 ? (c & 1) * Lds::x : 0) + lg * PLANE + (wm * TMW * 16 + li) * 16;
#pragma unroll
        for (int tap = 0; tap < TAPS; ++tap) {
            const int g = c * TAPS + tap;
            open();
            if (tap == 0 && c + 1 < nc) x_fetch((c + 1) * KC);
            if (D > 2 || g + 1 < nk) w_issue(min(g + D - 1, nk - 1), ring == 0 ? D - 1 : ring - 1);
            const char* ws = smem + XB * Lds::x + ring * Lds::w + wn * TNW * kF32Pieces * FRAG + lane * 16;
            bf16x8 xf[TMW][kF32Pieces];
#pragma unroll
            for (int q = 0; q < kF32Pieces; ++q)
#pragma unroll
                for (int i = 0; i < TMW; ++i)
                    xf[i][q] = *reinterpret_cast<const bf16x8*>(xs + q * 4 * PLANE + (i * 16 + tap) * 16);
#pragma unroll
            for (int j0 = 0; j0 < TNW; j0 += JG) {
                bf16x8 wf[JG][kF32Pieces];
#pragma unroll
                for (int q = 0; q < kF32Pieces; ++q)
#pragma unroll
                    for (int j = 0; j < JG; ++j)
                        wf[j][q] = *reinterpret_cast<const bf16x8*>(ws + ((j0 + j) * kF32Pieces + q) * FRAG);
                f32x4 low[TMW][JG];                 // the step's five smaller products
#pragma unroll
                for (int t = 0; t < kF32Products; ++t)
#pragma unroll
                    for (int i = 0; i < TMW; ++i)
#pragma unroll
                        for (int j = 0; j < JG; ++j) {
                            f32x4& d = t + 1 < kF32Products ? low[i][j] : acc[i][j0 + j];
                            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][kProd[t][0]], xf[i][kProd[t][1]],
                                                                        t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : d, 0, 0, 0);
                        }
#pragma unroll
                for (int i = 0; i < TMW; ++i)
#pragma unroll
                    for (int j = 0; j < JG; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j0 + j][v] += low[i][j][v];
            }
            if (XB == 2 && tap == TAPS - 1 && c + 1 < nc) x_store((c + 1) & 1, (c + 1) * KC);
            ring = ring + 1 == D ? 0 : ring + 1;
        }
        if (XB == 1 && c + 1 < nc) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // every wave has read the chunk
            x_store(0, (c + 1) * KC);
        }
    }

    // no load may reach this block's LDS after the block has ended
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    f32_epilogue<WM, TMW, TNW, EPI>(acc, a, m0, n0, tid);
}

template <int WM, int WN, int TMW, int TNW, int D, int TAPS, int EPI>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(F32Occ<WM, WN, TMW, TNW, 1, D, TAPS>::v)))
void conv_mfma_f32(ConvArgs a)
{
    conv_f32_tile<WM, WN, TMW, TNW, 1, D, TAPS, EPI, false>(a);
}

// Double-buffered halo: the next chunk is split into the second buffer behind
// the current chunk's last step, one barrier less per chunk for twice the LDS.
template <int WM, int WN, int TMW, int TNW, int TAPS, int EPI>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(F32Occ<WM, WN, TMW, TNW, 2, 2, TAPS>::v)))
void conv_mfma_f32_db(ConvArgs a)
{
    conv_f32_tile<WM, WN, TMW, TNW, 2, 2, TAPS, EPI, false>(a);
}

// enc0.c2 with the first convolution in its staging (max-pool epilogue)
template <int WM, int WN, int TMW, int TNW, int D>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(F32Occ<WM, WN, TMW, TNW, 1, D, kTaps>::v)))
void conv_mfma_f32_first(ConvArgs a)
{
    conv_f32_tile<WM, WN, TMW, TNW, 1, D, kTaps, EPI_POOL, true>(a);
}

template <int WM, int WN, int TMW, int TNW>
dim3 tile_grid(const ConvArgs& a)
{
    constexpr int BM = WM * TMW * 16;
    constexpr int BN = WN * TNW * 16;
    const unsigned m_tiles = (unsigned)((a.m_rows + BM - 1) / BM);
    return dim3((m_tiles + kXcds - 1) / kXcds * kXcds * (unsigned)(a.n / BN));
}

template <int WM, int WN, int TMW, int TNW, int XB, int D, int TAPS, int EPI>
hipError_t run(const ConvArgs& a, hipStream_t s)
{
    const dim3 grid = tile_grid<WM, WN, TMW, TNW>(a);
    if constexpr (XB == 2)
        hipLaunchKernelGGL((conv_mfma_f32_db<WM, WN, TMW, TNW, TAPS, EPI>), grid, dim3(WM * WN * 64), 0, s, a);
    else
        hipLaunchKernelGGL((conv_mfma_f32<WM, WN, TMW, TNW, D, TAPS, EPI>), grid, dim3(WM * WN * 64), 0, s, a);
    return hipGetLastError();
}

template <int WM, int WN, int TMW, int TNW, int D>
hipError_t run_first(const ConvArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL((conv_mfma_f32_first<WM, WN, TMW, TNW, D>), (tile_grid<WM, WN, TMW, TNW>(a)), dim3(WM * WN * 64), 0,
                       s, a);
    return hipGetLastError();
}

// Tile-shape variants.  Every variant accumulates each output's k terms in
// the same order (32-channel chunk, tap, product), so all of them give
// bitwise-identical results; they differ only in speed.
struct Variant { int wm, wn, tmw, tnw, xb, d; };
constexpr Variant kVariants[] = {
    {4, 1, 4, 2, 1, 2}, {4, 1, 2, 2, 1, 2}, {2, 1, 4, 2, 1, 2},                         // 0-2: 32 columns
    {4, 1, 4, 4, 1, 2}, {4, 1, 2, 4, 1, 2}, {2, 1, 4, 4, 1, 2},                         // 3-5: 64 columns
    {2, 2, 4, 4, 1, 2}, {4, 2, 2, 4, 1, 2}, {4, 2, 4, 4, 1, 2}, {2, 2, 2, 4, 1, 2},     // 6-9: 128 columns
    {2, 4, 4, 4, 1, 2},                                                                 // 10: 256 columns
    {4, 1, 4, 2, 2, 2}, {4, 1, 4, 4, 2, 2}, {4, 2, 4, 4, 2, 2}, {2, 1, 4, 2, 2, 2},     // 11-14: double-buffered halo
    {4, 1, 1, 2, 1, 6}, {2, 1, 1, 2, 1, 6}, {4, 1, 2, 2, 1, 4},                         // 15-17: 64, 32, 128 x 32, deep weight ring
    {4, 1, 1, 4, 1, 4},                                                                 // 18: 64 x 64, the same
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

#define PVF_VARIANT_CASE(V, TAPS, EPI)                                                                  \
    case V:                                                                                             \
        return run<kVariants[V].wm, kVariants[V].wn, kVariants[V].tmw, kVariants[V].tnw, kVariants[V].xb, \
                   kVariants[V].d, TAPS, EPI>(a, s);

template <int TAPS, int EPI>
hipError_t dispatch(int v, const ConvArgs& a, hipStream_t s)
{
    if constexpr (EPI == EPI_HEAD) {
        switch (v) {
            PVF_VARIANT_CASE(0, TAPS, EPI)
            PVF_VARIANT_CASE(1, TAPS, EPI)
            PVF_VARIANT_CASE(2, TAPS, EPI)
            PVF_VARIANT_CASE(3, TAPS, EPI)
            PVF_VARIANT_CASE(5, TAPS, EPI)
            PVF_VARIANT_CASE(11, TAPS, EPI)
            PVF_VARIANT_CASE(12, TAPS, EPI)
            PVF_VARIANT_CASE(14, TAPS, EPI)
            PVF_VARIANT_CASE(15, TAPS, EPI)
            PVF_VARIANT_CASE(16, TAPS, EPI)
            PVF_VARIANT_CASE(17, TAPS, EPI)
            PVF_VARIANT_CASE(18, TAPS, EPI)
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (v) {
            PVF_VARIANT_CASE(0, TAPS, EPI)
            PVF_VARIANT_CASE(1, TAPS, EPI)
            PVF_VARIANT_CASE(2, TAPS, EPI)
            PVF_VARIANT_CASE(3, TAPS, EPI)
            PVF_VARIANT_CASE(4, TAPS, EPI)
            PVF_VARIANT_CASE(5, TAPS, EPI)
            PVF_VARIANT_CASE(6, TAPS, EPI)
            PVF_VARIANT_CASE(7, TAPS, EPI)
            PVF_VARIANT_CASE(8, TAPS, EPI)
            PVF_VARIANT_CASE(9, TAPS, EPI)
            PVF_VARIANT_CASE(10, TAPS, EPI)
            PVF_VARIANT_CASE(11, TAPS, EPI)
            PVF_VARIANT_CASE(12, TAPS, EPI)
            PVF_VARIANT_CASE(13, TAPS, EPI)
            PVF_VARIANT_CASE(14, TAPS, EPI)
            PVF_VARIANT_CASE(15, TAPS, EPI)
            PVF_VARIANT_CASE(16, TAPS, EPI)
            PVF_VARIANT_CASE(17, TAPS, EPI)
            PVF_VARIANT_CASE(18, TAPS, EPI)
        default: return hipErrorInvalidValue;
        }
    }
}

}  // namespace

hipError_t launch_split_weights(const float* w, int n, int taps, int cin, float w_sum, uint16_t* pieces, hipStream_t s)
{
    if (n % 16 != 0 || cin % KC != 0) return hipErrorInvalidValue;
    const unsigned threads = (unsigned)(n / 16 * taps * (cin / KC)) * 64;
    hipLaunchKernelGGL(split_weights, dim3((threads + 255) / 256), dim3(256), 0, s, w, n, taps, cin,
                       w_sum > kRoundSum ? 0.f : kBf16Cut, pieces);
    return hipGetLastError();
}

float f32_split_cut(float w_sum) { return std::fmin(kBf16Cut, 0x1p127f / w_sum); }

int f32_variant_count() { return kNumVariants; }

bool f32_variant_ok(int v, int n, int taps, Epi epi)
{
    if (v < 0 || v >= kNumVariants) return false;
    const Variant& x = kVariants[v];
    const int bn = x.wn * x.tnw * 16;
    // the head reduces over all channels inside one wave's columns
    if (epi == EPI_HEAD) return (v <= 3 || v == 5 || v == 11 || v == 12 || (v >= 14 && v <= 18)) && bn == n && x.wn == 1;
    (void)taps;
    return bn <= (n < 32 ? 32 : n);
}

// Defaults from a sweep on MI355X (1000 events of the 32-channel network, 123
// of the 64-channel one): the waves of 32 positions win, as their blocks take
// half the registers and a third more waves share a CU; 128 columns where
// there are as many, since a halo tile is then split for twice the columns
// (enc3.c2 1393 us, against 1468 with 64 x 64 waves and 1437 with 64 columns).
int f32_default_variant(int n, int cin, int taps, Epi epi)
{
    (void)cin;
    (void)taps;
    if (n == 32) return 1;
    if (n == 64) return epi == EPI_HEAD ? 3 : 4;
    return 7;
}

// Tiles of small batches, from sweeps of 1 to 200 events of the 32-channel
// network.  A launch then waits on one block's serial chain of steps, not on
// throughput, so the smallest tile wins that still keeps every block on the
// device at once: three blocks a CU of the deep-ring tiles (enc3.c2, launch and
// its event, one event: 32 x 32 tiles 17 us, 64 x 32 20 us, 128 x 32 26 us, 128 x
// 128 50 us; eight events, 1008 32 x 32 blocks: 33 us against 24 us with 64 x 32;
// 16 events, 1008 64 x 32 blocks: 41 us against 35 us with 128 x 32).
int f32_batch_variant(int full, int n, Epi epi, int m_rows, int cus)
{
    const int at_once = 3 * cus;
    if (epi == EPI_HEAD && n == 64) return tile_blocks(m_rows, n, 64, 64) <= at_once ? 18 : full;
    if (tile_blocks(m_rows, n, 32, 32) <= at_once) return 16;
    if (tile_blocks(m_rows, n, 64, 32) <= at_once) return 15;
    if (tile_blocks(m_rows, n, 128, 32) <= at_once) return 17;
    if (n >= 64 && tile_blocks(m_rows, n, 128, 64) <= at_once) return 4;
    return full;
}

std::string f32_kernel_name(int v, int taps, Epi epi)
{
    const Variant& x = kVariants[v];
    return std::string(x.xb == 2 ? "conv_mfma_f32_db<" : "conv_mfma_f32<") + std::to_string(x.wm) + ", " +
           std::to_string(x.wn) + ", " + std::to_string(x.tmw) + ", " + std::to_string(x.tnw) + ", " +
           (x.xb == 2 ? "" : std::to_string(x.d) + ", ") + std::to_string(taps) + ", " + std::to_string((int)epi) + ">";
}

// Variants that can take the fused first convolution: the single-buffered
// tiles of up to 64 columns (enc0.c2 has 32 or 64).
bool f32_first_ok(int v)
{
    return (v >= 0 && v <= 5) || (v >= 15 && v <= 17);
}

std::string f32_first_kernel_name(int v)
{
    const Variant& x = kVariants[v];
    return "conv_mfma_f32_first<" + std::to_string(x.wm) + ", " + std::to_string(x.wn) + ", " +
           std::to_string(x.tmw) + ", " + std::to_string(x.tnw) + ", " + std::to_string(x.d) + ">";
}

hipError_t launch_conv_f32_first(const ConvArgs& a, int v, hipStream_t s)
{
    if (a.cin % KC != 0 || a.m_rows <= 0 || a.n % 32 != 0 || !f32_first_ok(v) || !f32_variant_ok(v, a.n, kTaps, EPI_POOL))
        return hipErrorInvalidValue;
    switch (v) {
    case 0: return run_first<kVariants[0].wm, kVariants[0].wn, kVariants[0].tmw, kVariants[0].tnw, kVariants[0].d>(a, s);
    case 1: return run_first<kVariants[1].wm, kVariants[1].wn, kVariants[1].tmw, kVariants[1].tnw, kVariants[1].d>(a, s);
    case 2: return run_first<kVariants[2].wm, kVariants[2].wn, kVariants[2].tmw, kVariants[2].tnw, kVariants[2].d>(a, s);
    case 3: return run_first<kVariants[3].wm, kVariants[3].wn, kVariants[3].tmw, kVariants[3].tnw, kVariants[3].d>(a, s);
    case 4: return run_first<kVariants[4].wm, kVariants[4].wn, kVariants[4].tmw, kVariants[4].tnw, kVariants[4].d>(a, s);
    case 5: return run_first<kVariants[5].wm, kVariants[5].wn, kVariants[5].tmw, kVariants[5].tnw, kVariants[5].d>(a, s);
    case 15: return run_first<kVariants[15].wm, kVariants[15].wn, kVariants[15].tmw, kVariants[15].tnw, kVariants[15].d>(a, s);
    case 16: return run_first<kVariants[16].wm, kVariants[16].wn, kVariants[16].tmw, kVariants[16].tnw, kVariants[16].d>(a, s);
    case 17: return run_first<kVariants[17].wm, kVariants[17].wn, kVariants[17].tmw, kVariants[17].tnw, kVariants[17].d>(a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_f32(const ConvArgs& a, int taps, Epi epi, int variant, hipStream_t s)
{
    if (a.cin % KC != 0 || a.m_rows <= 0 || a.n % 32 != 0 || !f32_variant_ok(variant, a.n, taps, epi)) return hipErrorInvalidValue;
    if (taps == 5) {
        switch (epi) {
        case EPI_STORE: return dispatch<5, EPI_STORE>(variant, a, s);
        case EPI_POOL: return dispatch<5, EPI_POOL>(variant, a, s);
        case EPI_HEAD: return dispatch<5, EPI_HEAD>(variant, a, s);
        default: return hipErrorInvalidValue;
        }
    }
    if (taps == 1 && epi == EPI_CONVT) return dispatch<1, EPI_CONVT>(variant, a, s);
    return hipErrorInvalidValue;
}

}  // namespace pvf
