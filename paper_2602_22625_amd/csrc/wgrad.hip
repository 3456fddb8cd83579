// Weight and bias gradient of the learned initialiser's convolutions (3x3, stride 2, padding 1;
// NHWC bfloat16, float32 accumulation): dw[oc][tap][ic] += sum over output pixels p of
// dz[p][oc] x[patch(p)][tap][ic], db[oc] += sum dz[p][oc].
//
// The product's K runs over pixels, which no operand has contiguous: a matrix operand needs 8
// pixels of one channel per lane, memory holds the channels of one pixel. So a lane loads a few
// neighbouring channels of 8 consecutive output pixels (16 lanes together a contiguous run of one
// pixel's channels) and packs them by channel with v_perm: one instruction per operand register,
// no LDS, no two-byte stores. With w channels per lane, fragment c of a run of 16 w channels has
// channel w r + c in row r.
//   dz   8 loads of WM channels per lane: WM fragments;
//   x    one tap row ky of 32 channels: the 17 input columns under 8 output pixels serve all three
//        kx (2 channels per lane): 6 fragments.
// A wave accumulates 16 WM x (3 x 32) weights over its share of the pixels, 24 products per 32
// pixels (WM = 4) from 25 loads, the next 32 pixels' loads in flight during them. The four waves
// of a workgroup take different pixels of the same weights; their sums meet in LDS and go out as
// one float32 atomic per weight and workgroup. The bias gradient is one more product, with ones,
// in the workgroups of the first tap row and channels.
//
// Workgroups of one run of pixels (all weights) are dealt to one XCD: its L2 then serves the run's
// dz and x to all of them. The gather product it replaces read both operands through transposing
// two-byte LDS stores, with four integer divisions per load: at batch 64 it took 151, 98, 90, 89,
// 51 and 20 us for the six layers, and a column-sum launch of 11 to 36 us each for the biases; now
// 39, 30, 24, 25, 17 and 11 us, biases included. The first two read 134 and 101 MB, 26 and 20 us at
// the rate of a large copy; the deeper ones have few steps per wave (4 to 16), so a large part of
// theirs is the first loads' latency and the sums' way out.
// The dense layers' gradients (dw[n][k] += sum over rows of dz[row][n] x[row][k]) are the same with
// rows for pixels and one tap: at 1,024 rows, 256 -> 512 and 512 -> 512, 5.4 (15.2) and 6.5 us (17.6).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "cnn_kernels.h"

namespace dbmp_cnn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

struct WgradArgs {
    const u16 *x, *dz;  // [B][H][W][Cin], [B][OH][OW][Cout]
    float *dw, *db;     // [Cout][9][Cin], [Cout] or null
    int H, W, OH, OW, Cin, Cout;
    unsigned x_bytes, dz_bytes;
    int groups;             // runs of 8 output pixels
    int tiles_m, tiles_n;   // channel tiles of dz and x
    int splits, per_wave;   // pixel splits; 32-pixel steps per wave
};

// An offset past every buffer: reads zeros.
constexpr unsigned OOB = 0x80000000u;

template <int N>
struct Words {
    uint32_t w[N];
};

// N words at byte voff + soff of the buffer
template <int N>
__device__ __forceinline__ Words<N> load_words(__amdgpu_buffer_rsrc_t b, unsigned voff, int soff)
{
    Words<N> o;
    if constexpr (N == 1) {
        o.w[0] = __builtin_amdgcn_raw_buffer_load_b32(b, voff, soff, 0);
    } else if constexpr (N == 2) {
        const uintx2 v = __builtin_amdgcn_raw_buffer_load_b64(b, voff, soff, 0);
        o.w[0] = v.x;
        o.w[1] = v.y;
    } else {
        const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(b, voff, soff, 0);
        o.w[0] = v.x;
        o.w[1] = v.y;
        o.w[2] = v.z;
        o.w[3] = v.w;
    }
    return o;
}

// (channel c of a, channel c of b) as one operand register
__device__ __forceinline__ uint32_t pair(uint32_t a, uint32_t b, int c)
{
    return __builtin_amdgcn_perm(b, a, c & 1 ? 0x07060302u : 0x05040100u);
}

// The pixel split and weight tile of a workgroup: splits in multiples of 8 (or 1, 2, 4) so that
// the workgroups of one split, dealt round-robin over the XCDs, share an XCD (or 8 / splits).
__device__ __forceinline__ void place(int bid, int tiles, int splits, int &split, int &tile)
{
    const int xcd = bid & 7, k = bid >> 3;
    if (splits >= 8) {
        split = xcd + 8 * (k / tiles);
        tile = k % tiles;
    } else {
        split = xcd % splits;
        tile = k * (8 / splits) + xcd / splits;
    }
}

// Sum of the four waves' N accumulators, left in LDS: s[0][i] + s[1][i] is accumulator word i of
// the layout [fragment][lane][4]. (Two halves, so that 2 N KB suffice.)
template <int N>
__device__ __forceinline__ void meet(floatx4 (&acc)[N], float (&s)[2][N * 256], int lane, int wave)
{
    if (wave >= 2) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            *reinterpret_cast<floatx4 *>(&s[wave - 2][i * 256 + lane * 4]) = acc[i];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            floatx4 *p = reinterpret_cast<floatx4 *>(&s[wave][i * 256 + lane * 4]);
            *p = acc[i] + *p;
        }
    }
    __syncthreads();
}

// The bias sums of the four waves (every column of accb is the sum over pixels).
template <int WM>
__device__ __forceinline__ void add_bias(const floatx4 (&accb)[WM], float *s, float *db, int lane,
                                         int wave)
{
    if ((lane & 15) == 0) {
#pragma unroll
        for (int c = 0; c < WM; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s[wave * 64 + (4 * (lane >> 4) + e) * WM + c] = accb[c][e];
    }
    __syncthreads();
    if (threadIdx.x < 16 * WM)
        unsafeAtomicAdd(db + threadIdx.x, (s[threadIdx.x] + s[64 + threadIdx.x]) +
                                              (s[128 + threadIdx.x] + s[192 + threadIdx.x]));
}

constexpr uint32_t ONES = 0x3f803f80u;  // a pair of bf16 ones

// WM channels of dz per lane (16 WM per workgroup), 32 channels of x. ROWS: the 8 output pixels of
// a group lie in ROWS image rows (OW % (8 / ROWS) == 0); ROWS = 0: a dense layer, whose 8 rows are
// the pixels of a 1 x 1 filter.
template <int WM, int ROWS>
__global__ void __launch_bounds__(256, 2) k_wgrad(WgradArgs a)
{
    constexpr int NR = ROWS ? ROWS : 1, SUB = 8 / NR, COLS = ROWS ? 2 * SUB + 1 : 8;
    constexpr int KX = ROWS ? 3 : 1, NF = WM * 2 * KX, TAPS = KX * KX;
    __shared__ __attribute__((aligned(16))) float s_red[2][NF * 256];
    __shared__ float s_b[256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    int split, tile;
    place(blockIdx.x, a.tiles_m * a.tiles_n * KX, a.splits, split, tile);
    if (split >= a.splits || tile >= a.tiles_m * a.tiles_n * KX) return;
    const int tm = tile % a.tiles_m, ky = tile / a.tiles_m % KX, tn = tile / a.tiles_m / KX;
    const int m0 = tm * 16 * WM, n0 = tn * 32;
    const bool bias = a.db && ky == 0 && tn == 0;
    const auto bz = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16 *>(a.dz), (short)0,
                                                      (int)a.dz_bytes, 0x00020000);
    const auto bx = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16 *>(a.x), (short)0,
                                                      (int)a.x_bytes, 0x00020000);
    struct Step {
        Words<WM / 2> z[8];
        uint32_t x[NR][COLS];
    };
    auto load = [&](int step, Step &s) {
        const int gr = step * 4 + g;
        const bool in = gr < a.groups;
        const unsigned p = (unsigned)gr * 8;
        const unsigned zo = in ? (p * (unsigned)a.Cout + m0 + WM * r) * 2 : OOB;
#pragma unroll
        for (int j = 0; j < 8; ++j) s.z[j] = load_words<WM / 2>(bz, zo, j * a.Cout * 2);
        if constexpr (ROWS == 0) {
            const unsigned xo = in ? (p * (unsigned)a.Cin + n0 + 2 * r) * 2 : OOB;
#pragma unroll
            for (int j = 0; j < 8; ++j) s.x[0][j] = load_words<1>(bx, xo, j * a.Cin * 2).w[0];
            return;
        }
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            const unsigned ps = in ? p + q * SUB : 0, row = ps / (unsigned)a.OW;
            const unsigned ox = ps - row * (unsigned)a.OW, b = row / (unsigned)a.OH;
            const int iy = 2 * (int)(row - b * (unsigned)a.OH) + ky - 1;
            const unsigned at =
                (((b * a.H + (unsigned)iy) * a.W + 2 * ox) * a.Cin + n0 + 2 * r) * 2;
            const unsigned xo = in && iy >= 0 ? at : OOB;
            s.x[q][0] = load_words<1>(bx, xo == OOB || ox == 0 ? OOB : at - 2 * a.Cin, 0).w[0];
#pragma unroll
            for (int i = 1; i < COLS; ++i)
                s.x[q][i] = load_words<1>(bx, xo, (i - 1) * a.Cin * 2).w[0];
        }
    };
    floatx4 acc[NF], accb[WM];
#pragma unroll
    for (int i = 0; i < NF; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < WM; ++c) accb[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int steps = (a.groups + 3) / 4, s0 = (split * 4 + wave) * a.per_wave;
    const int s1 = min(steps, s0 + a.per_wave);
    Step cur, nxt;
    if (s0 < s1) load(s0, cur);
    for (int s = s0; s < s1; ++s) {
        if (s + 1 < s1) load(s + 1, nxt);
        bf16x8 fa[WM];
#pragma unroll
        for (int c = 0; c < WM; ++c) {
            uintx4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = pair(cur.z[2 * q].w[c / 2], cur.z[2 * q + 1].w[c / 2], c);
            fa[c] = __builtin_bit_cast(bf16x8, v);
        }
        if (bias) {
            const uintx4 one = {ONES, ONES, ONES, ONES};
#pragma unroll
            for (int c = 0; c < WM; ++c)
                accb[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    fa[c], __builtin_bit_cast(bf16x8, one), accb[c], 0, 0, 0);
        }
#pragma unroll
        for (int kx = 0; kx < KX; ++kx)
#pragma unroll
            for (int cn = 0; cn < 2; ++cn) {
                uintx4 v;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] = ROWS == 0
                               ? pair(cur.x[0][2 * q % COLS], cur.x[0][(2 * q + 1) % COLS], cn)
                               : pair(cur.x[2 * q / SUB][2 * (2 * q % SUB) + kx],
                                      cur.x[(2 * q + 1) / SUB][2 * ((2 * q + 1) % SUB) + kx], cn);
                const bf16x8 fb = __builtin_bit_cast(bf16x8, v);
#pragma unroll
                for (int c = 0; c < WM; ++c)
                    acc[(c * KX + kx) * 2 + cn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        fa[c], fb, acc[(c * KX + kx) * 2 + cn], 0, 0, 0);
            }
        cur = nxt;
    }
    meet<NF>(acc, s_red, lane, wave);
    // thread t adds the weights of input channel t % 32 (neighbouring lanes: 128 contiguous bytes)
    const int cn = threadIdx.x & 1, col = (threadIdx.x >> 1) & 15;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (threadIdx.x >> 5) + 8 * i;
        const int at = ((row >> 2) * 16 + col) * 4 + (row & 3);
#pragma unroll
        for (int c = 0; c < WM; ++c)
#pragma unroll
            for (int kx = 0; kx < KX; ++kx) {
                const int k = ((c * KX + kx) * 2 + cn) * 256 + at;
                unsafeAtomicAdd(a.dw + ((size_t)(m0 + WM * row + c) * TAPS + ky * KX + kx) * a.Cin +
                                    n0 + 2 * col + cn,
                                s_red[0][k] + s_red[1][k]);
            }
    }
    if (bias) add_bias<WM>(accb, s_b, a.db + m0, lane, wave);
}

// The first layer (Cin = 8): column r of the x operand is tap r (9 of 16), a lane's 16 bytes the 8
// channels of its tap: 8 fragments.
template <int WM, int ROWS>
__global__ void __launch_bounds__(256, 2) k_wgrad8(WgradArgs a)
{
    constexpr int SUB = 8 / ROWS, NF = WM * 8;
    __shared__ __attribute__((aligned(16))) float s_red[2][NF * 256];
    __shared__ float s_b[256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    int split, tile;
    place(blockIdx.x, a.tiles_m, a.splits, split, tile);
    if (split >= a.splits || tile >= a.tiles_m) return;
    const int m0 = tile * 16 * WM;
    const auto bz = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16 *>(a.dz), (short)0,
                                                      (int)a.dz_bytes, 0x00020000);
    const auto bx = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16 *>(a.x), (short)0,
                                                      (int)a.x_bytes, 0x00020000);
    const int ky = r / 3, kx = r - 3 * ky;
    struct Step {
        Words<WM / 2> z[8];
        Words<4> x[8];
    };
    auto load = [&](int step, Step &s) {
        const int gr = step * 4 + g;
        const bool in = gr < a.groups;
        const unsigned p = (unsigned)gr * 8;
        const unsigned zo = in ? (p * (unsigned)a.Cout + m0 + WM * r) * 2 : OOB;
#pragma unroll
        for (int j = 0; j < 8; ++j) s.z[j] = load_words<WM / 2>(bz, zo, j * a.Cout * 2);
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
            const unsigned ps = in ? p + q * SUB : 0, row = ps / (unsigned)a.OW;
            const unsigned ox = ps - row * (unsigned)a.OW, b = row / (unsigned)a.OH;
            const int iy = 2 * (int)(row - b * (unsigned)a.OH) + ky - 1;
            // the second pixel's column, 2 (ox + 1) + kx - 1: inside the image for every tap
            const unsigned at = ((b * a.H + (unsigned)iy) * a.W + 2 * ox + (unsigned)kx + 1) * 16;
            const unsigned xo = in && r < 9 && iy >= 0 ? at : OOB;
            s.x[q * SUB] =
                load_words<4>(bx, xo == OOB || (kx == 0 && ox == 0) ? OOB : at - 32, 0);
#pragma unroll
            for (int j = 1; j < SUB; ++j) s.x[q * SUB + j] = load_words<4>(bx, xo, (j - 1) * 32);
        }
    };
    floatx4 acc[NF], accb[WM];
#pragma unroll
    for (int i = 0; i < NF; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < WM; ++c) accb[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int steps = (a.groups + 3) / 4, s0 = (split * 4 + wave) * a.per_wave;
    const int s1 = min(steps, s0 + a.per_wave);
    Step cur, nxt;
    if (s0 < s1) load(s0, cur);
    for (int s = s0; s < s1; ++s) {
        if (s + 1 < s1) load(s + 1, nxt);
        bf16x8 fa[WM];
#pragma unroll
        for (int c = 0; c < WM; ++c) {
            uintx4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = pair(cur.z[2 * q].w[c / 2], cur.z[2 * q + 1].w[c / 2], c);
            fa[c] = __builtin_bit_cast(bf16x8, v);
        }
        const uintx4 one = {ONES, ONES, ONES, ONES};
#pragma unroll
        for (int c = 0; c < WM; ++c)
            accb[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                fa[c], __builtin_bit_cast(bf16x8, one), accb[c], 0, 0, 0);
#pragma unroll
        for (int ch = 0; ch < 8; ++ch) {
            uintx4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = pair(cur.x[2 * q].w[ch / 2], cur.x[2 * q + 1].w[ch / 2], ch);
            const bf16x8 fb = __builtin_bit_cast(bf16x8, v);
#pragma unroll
            for (int c = 0; c < WM; ++c)
                acc[c * 8 + ch] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[c], fb,
                                                                          acc[c * 8 + ch], 0, 0, 0);
        }
        cur = nxt;
    }
    meet<NF>(acc, s_red, lane, wave);
    for (int i = threadIdx.x; i < 16 * WM * 72; i += 256) {  // dw[m0 ..][tap][ch], contiguous
        const int oc = i / 72, q = i - oc * 72, tap = q >> 3, ch = q & 7;
        const int row = oc / WM, c = oc - row * WM;
        const int k = (c * 8 + ch) * 256 + ((row >> 2) * 16 + tap) * 4 + (row & 3);
        unsafeAtomicAdd(a.dw + (size_t)m0 * 72 + i, s_red[0][k] + s_red[1][k]);
    }
    if (a.db) add_bias<WM>(accb, s_b, a.db + m0, lane, wave);
}

constexpr long long MAX_BYTES = (1LL << 31) - (1LL << 24);  // what OOB stays beyond

template <int WM, int ROWS>
void launch(WgradArgs a, hipStream_t st)
{
    constexpr int KX = ROWS ? 3 : 1;
    // 512 workgroups (two per compute unit) at most, at least four steps per wave; splits a
    // multiple of 8, or 1, 2 or 4 (place)
    const int tiles = a.tiles_m * (ROWS && a.Cin == 8 ? 1 : a.tiles_n * KX), steps = (a.groups + 3) / 4;
    int s = std::min(std::max(1, 512 / tiles), std::max(1, steps / 16));
    s = s >= 8 ? s / 8 * 8 : s >= 4 ? 4 : s >= 2 ? 2 : 1;
    a.splits = s;
    a.per_wave = (steps + 4 * s - 1) / (4 * s);
    const int blocks = s >= 8 ? s * tiles : 8 * ((tiles + 8 / s - 1) / (8 / s));
    if constexpr (WM == 2 && ROWS != 0)
        if (a.Cin == 8) return k_wgrad8<WM, ROWS><<<blocks, 256, 0, st>>>(a);
    k_wgrad<WM, ROWS><<<blocks, 256, 0, st>>>(a);
}

}  // namespace

bool conv_backward_weight_direct(hipStream_t st, const uint16_t *x, const uint16_t *dz, int B,
                                 int H, int W, int Cin, int Cout, float *dw, float *db,
                                 hipError_t *err)
{
    const long long P = (long long)B * (H / 2) * (W / 2);
    const long long xb = 8 * P * Cin, zb = 2 * P * Cout;
    if (xb > MAX_BYTES || zb > MAX_BYTES || Cout % 32 != 0 || (Cin != 8 && Cin % 32 != 0))
        return false;
    if ((W / 2) % 4 != 0 || P % 8 != 0 || (((uintptr_t)x | (uintptr_t)dz) & 15) != 0) return false;
    const bool wide = Cout % 64 == 0 && Cin != 8, rows2 = (W / 2) % 8 != 0;
    const WgradArgs a{x, dz, dw, db, H, W, H / 2, W / 2, Cin, Cout, (unsigned)xb, (unsigned)zb,
                      (int)(P / 8), Cout / (wide ? 64 : 32), Cin / 32, 0, 0};
    if (wide) rows2 ? launch<4, 2>(a, st) : launch<4, 1>(a, st);
    else rows2 ? launch<2, 2>(a, st) : launch<2, 1>(a, st);
    *err = hipGetLastError();
    return true;
}

bool linear_backward_weight_direct(hipStream_t st, const uint16_t *x, const uint16_t *dz, int B,
                                   int K, int N, float *dw, float *db, hipError_t *err)
{
    const long long xb = 2LL * B * K, zb = 2LL * B * N;
    if (xb > MAX_BYTES || zb > MAX_BYTES || N % 32 != 0 || K % 32 != 0 || B % 8 != 0) return false;
    if ((((uintptr_t)x | (uintptr_t)dz) & 15) != 0) return false;
    const bool wide = N % 64 == 0;
    const WgradArgs a{x, dz, dw, db, 1, 1, 1, 1, K, N, (unsigned)xb, (unsigned)zb, B / 8,
                      N / (wide ? 64 : 32), K / 32, 0, 0};
    wide ? launch<4, 0>(a, st) : launch<2, 0>(a, st);
    *err = hipGetLastError();
    return true;
}

}  // namespace dbmp_cnn
