// Direct convolution kernels of the learned initialiser (3x3, stride 2, padding 1; NHWC bfloat16,
// float32 accumulation): forward and input gradient. Its dense layers run on the same kernel, a row
// in the place of a pixel and a run of C inputs in that of a tap.
//
// One wave computes MT x 16 pixels by NT x 16 channels with v_mfma_f32_16x16x32_bf16, the weights
// as the A operand (rows = channels) and the pixels as B (columns = pixels), a workgroup four
// such pixel tiles of the same channels. Both operands go through LDS, copied there by LDS-direct
// loads, RING stages (a tap's products over GC chunks of 32 channels) at a time:
//   - no address arithmetic but one addition per copy: a pixel's position is found once, a tap
//     adds a constant; a tap outside the image reads a page of zeros;
//   - four neighbouring lanes copy 64 contiguous bytes of one pixel (or weight row). Loading the
//     operand registers straight from memory instead, where 16 neighbouring lanes are 16 pixels,
//     costs a cache lookup per lane: 13 bytes per clock and compute unit, whatever was in flight;
//   - a fragment is 16 rows of 64 bytes; row r's four 16-byte groups are stored in the order
//     g ^ (r / 4), which makes the operand reads free of bank conflicts;
//   - a stage waits with a count for its own copies only (the later stages' stay in flight: a
//     kernel starts with cold L2s on this chip, and a load takes a large part of a microsecond).
// The rows of a channel fragment pair are interleaved so that a lane ends with 8 consecutive
// channels of one pixel: bias, ReLU or mask, and one 16-byte store.
// The K order (tap, then channels by 32) is that of the general gather product, so both give the
// same bits.
//
// The input gradient of a stride-2 convolution falls apart into four parity classes of input
// pixels, reached by 1, 2, 2 and 4 taps: one wave takes the four pixels (2 hy + py, 2 hx + px) of
// its 16 MT positions (hy, hx), class by class, so it runs the same nine taps as the forward and
// stores after the class's last.
//
// Measured at batch 64 (forward, then input gradient; us, against the gather product before):
//   256^2 x 8 -> 32    30 (78)             128^2 x 32 -> 64   28 (44), 44 (160)
//   64^2 x 64 -> 128   21 (38), 23 (76)    32^2 x 128 -> 256  15 (33), 21 (60)
//   16^2 x 256 -> 256  12 (34), 15 (37)    8^2 x 256 -> 256    7 (34),  8 (25)
// The first two move 134 and 100 MB (167 MB for the gradient): 26, 20 and 33 us at the rate of a
// large copy, which bounds them; the others are bound by the latency of their stages.
// Dense layers at 1,024 rows (64 images; 256 -> 512 and 512 -> 512, latency): forward 4.0 (7.4) and
// 4.6 (9.5), input gradient 3.9 (9.3) and 4.7 (9.4).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "cnn_kernels.h"

namespace dbmp_cnn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

// Convolutions, and the dense layers' y = act(x w^T + bias) and dx = [mask > 0] dz wt^T.
enum { FWD = 0, DGRAD = 1, LFWD = 2, LDGRAD = 3 };
constexpr bool is_lin(int mode) { return mode >= LFWD; }
constexpr bool is_fwd(int mode) { return mode == FWD || mode == LFWD; }

struct ConvArgs {
    const u16 *src;    // FWD: x [B][H][W][C]; DGRAD: dz [B][OH][OW][C]
    const u16 *w;      // [N][3][3][C]
    const float *bias; // FWD
    const u16 *mask;   // DGRAD
    u16 *out;          // FWD: y [B][OH][OW][N]; DGRAD: dx [B][H][W][N]
    float *out32;      // FWD
    int relu;
    int H, W, OH, OW;  // H = 2 OH, W = 2 OW
    int P, N;          // P = B OH OW pixels (FWD) or 2 x 2 quads (DGRAD)
    unsigned src_bytes;
    int taps;          // dense layers: runs of C inputs (H = W = OH = OW = 1)
};

// An offset past every buffer (sizes stay below 2^31 bytes); the instruction's immediate is added
// to it without reaching 2^32.
constexpr unsigned OOB = 0x80000000u;

// The t-th tap in the order of the products (two bits each). DGRAD: the classes (even, even),
// (even, odd), (odd, even), (odd, odd) of (y, x) in turn, each class's taps in row-major order.
template <int MODE>
__device__ __forceinline__ int tap_ky(int t)
{
    return ((MODE == FWD ? 0b10'10'10'01'01'01'00'00'00 : 0b10'10'00'00'10'00'01'01'01) >> (2 * t)) &
           3;
}
template <int MODE>
__device__ __forceinline__ int tap_kx(int t)
{
    return ((MODE == FWD ? 0b10'01'00'10'01'00'10'01'00 : 0b10'00'10'00'01'01'10'00'01) >> (2 * t)) &
           3;
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const floatx2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// Channel (within the block's NT * 16) of row r of fragment nt: fragment pairs interleave rows so
// that the accumulators of a lane hold 8 consecutive channels.
template <int NT>
__device__ __forceinline__ int frag_chan(int nt, int r)
{
    return NT == 1 ? r : 32 * (nt >> 1) + 8 * (r >> 2) + 4 * (nt & 1) + (r & 3);
}

// Blocks are dealt round-robin over the 8 XCDs: give each XCD a contiguous run of pixel tiles, so
// that the rows neighbouring tiles share meet in one L2.
__device__ __forceinline__ int xcd_run(int bid, int n)
{
    const int q = n >> 3, r = n & 7, x = bid & 7, l = bid >> 3;
    return x * q + (x < r ? x : r) + l;
}

// Bias, ReLU (forward) or mask (input gradient) and the store of one wave's accumulators.
// pix[mt] + shift: the output pixel of this lane (pix < 0: none).
template <int MODE, int MT, int NT>
__device__ __forceinline__ void store_tile(const ConvArgs &a, const floatx4 (&acc)[MT][NT],
                                           const int (&pix)[MT], int shift, int n0, int g)
{
    constexpr int NP = (NT + 1) / 2, NV = NT == 1 ? 4 : 8;
    uintx4 msk[MT][NP];
    if (!is_fwd(MODE) && a.mask) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if (pix[mt] < 0) continue;
                const u16 *mp = a.mask + (size_t)(pix[mt] + shift) * a.N + n0 + 32 * q + NV * g;
                if constexpr (NT == 1) {
                    const uint2 m2 = *reinterpret_cast<const uint2 *>(mp);
                    msk[mt][q] = uintx4{m2.x, m2.y, 0, 0};
                } else {
                    msk[mt][q] = *reinterpret_cast<const uintx4 *>(mp);
                }
            }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const int n = n0 + 32 * q + (NT == 1 ? 4 : 8) * g;
        float b[NV];
        if (is_fwd(MODE)) {
#pragma unroll
            for (int j = 0; j < NV; ++j) b[j] = a.bias ? a.bias[n + j] : 0.f;
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (pix[mt] < 0) continue;
            float v[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                v[j] = acc[mt][NT == 1 ? 0 : 2 * q + (j >> 2)][j & 3];
                if (is_fwd(MODE)) {
                    if (a.bias) v[j] += b[j];
                    if (a.relu) v[j] = fmaxf(v[j], 0.f);
                } else if (a.mask) {
                    const uint32_t w = msk[mt][q][j >> 1];
                    const float m = __uint_as_float(j & 1 ? w & 0xffff0000u : w << 16);
                    if (!(m > 0.f)) v[j] = 0.f;
                }
            }
            const size_t i = (size_t)(pix[mt] + shift) * a.N + n;
            if (!is_fwd(MODE) || a.out) {
                if constexpr (NT == 1)
                    *reinterpret_cast<uint2 *>(a.out + i) =
                        make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
                else
                    *reinterpret_cast<uint4 *>(a.out + i) =
                        make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]),
                                   pack_bf16(v[4 % NV], v[5 % NV]), pack_bf16(v[6 % NV], v[7 % NV]));
            }
            if (is_fwd(MODE) && a.out32) {
#pragma unroll
                for (int j = 0; j < NV; j += 4)
                    *reinterpret_cast<float4 *>(a.out32 + i + j) =
                        make_float4(v[j], v[j + 1], v[j + 2], v[j + 3]);
            }
        }
    }
}

// A stage's chunks: about 16 products per wave, so that the barrier and the copies' issue are a
// small part of it.
constexpr int stage_chunks(int nch, int mt, int nt)
{
    return std::min(nch, std::min(4, std::max(4 / nt, 16 / (mt * nt))));
}
constexpr int stage_kb(int nch, int mt, int nt)
{
    return stage_chunks(nch, mt, nt) * (nt + 4 * mt);
}
// Stages in LDS: as many as leave room for two workgroups per compute unit, three to five. (Three of
// the 32 KB stages of 1 x 4 tiles with 128 channels or more take 96 KB: one workgroup there.)
constexpr int ring(int nch, int mt, int nt)
{
    return std::max(3, std::min(5, 80 / stage_kb(nch, mt, nt)));
}

// Waits until at most N vector-memory operations of this wave are outstanding (and its LDS reads
// are done), then for the workgroup. A __syncthreads() would wait for all of them.
template <int N>
__device__ __forceinline__ void stage_barrier()
{
    static_assert(N < 64, "six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__device__ const uint4 g_zeros[1] = {};  // what a tap outside the image reads

using GChar = const __attribute__((address_space(1))) char;

// 16 bytes per lane from p into LDS at dst + 16 lane
__device__ __forceinline__ void copy_to_lds(GChar *p, u16 *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// C = 32 NCH channels of K per tap; dense layers: a.taps runs of C inputs per row.
// (Four waves per SIMD bound the registers of the smallest tiles alone; where the stages' LDS allows
// fewer, the compiler says so and takes what that allows. A bound of what it allows gave other code
// and the same times.)
template <int MODE, int NCH, int MT, int NT>
__global__ void __launch_bounds__(256, 4) k_conv(ConvArgs a)
{
    constexpr int C = 32 * NCH, GC = stage_chunks(NCH, MT, NT), SPT = NCH / GC;
    constexpr int FR = GC * NT, FP = GC * MT;  // weight and (per wave) pixel fragments of a stage
    constexpr int RING = ring(NCH, MT, NT), D = RING - 1;  // stages in flight
    constexpr int SLOT = (FR + 4 * FP) * 512;
    const int taps = is_lin(MODE) ? a.taps : 9, stages = taps * SPT;
    __shared__ __attribute__((aligned(1024))) u16 s_st[RING * SLOT];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.y * NT * 16;
    const int p0 = (xcd_run(blockIdx.x, gridDim.x) * 4 + wave) * (MT * 16);
    // as a copier the lane takes row cr and its 16-byte group cg
    const int cr = lane >> 2, cg = (lane & 3) ^ (cr >> 2);
    // (a wave's weight fragments all have nt = wave % NT: NT divides 4)
    GChar *wp = (GChar *)(a.w + (size_t)(n0 + frag_chan<NT>(wave % NT, cr)) * (taps * C) + cg * 8);
    GChar *zp = (GChar *)g_zeros;
    GChar *pp[MT];     // the copied pixel's channels at the centre tap
    bool ey[MT], ex[MT];  // the taps with ky = 0 / kx = 0 lie outside the image
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const unsigned i = (unsigned)min(p0 + mt * 16 + cr, a.P - 1);
        if constexpr (is_lin(MODE)) {
            pp[mt] = (GChar *)(a.src + (size_t)i * (unsigned)(taps * C) + cg * 8);
            ey[mt] = ex[mt] = false;
            continue;
        }
        const unsigned row = i / (unsigned)a.OW;
        const int x = (int)(i - row * (unsigned)a.OW), b = (int)(row / (unsigned)a.OH);
        const int y = (int)(row - (unsigned)b * (unsigned)a.OH);
        const size_t at = MODE == FWD ? ((size_t)b * a.H + 2 * y) * a.W + 2 * x : i;
        pp[mt] = (GChar *)(a.src + at * C + cg * 8);
        ey[mt] = MODE == FWD ? y == 0 : y == a.OH - 1;
        ex[mt] = MODE == FWD ? x == 0 : x == a.OW - 1;
    }
    // stage s's copies into its slot: the weights dealt over the waves, each wave's own pixels
    auto copy_stage = [&](int t, int c0, int slot) {
        const int ky = is_lin(MODE) ? 0 : tap_ky<MODE>(t), kx = is_lin(MODE) ? t : tap_kx<MODE>(t);
        u16 *dst = s_st + slot * SLOT;
#pragma unroll
        for (int i = 0; i < (FR + 3) / 4; ++i) {
            const int f = wave + 4 * i;
            if (FR % 4 != 0 && f >= FR) break;
            copy_to_lds(wp + ((ky * 3 + kx) * C + (c0 + f / NT) * 32) * 2, dst + f * 512);
        }
        const int delta = is_lin(MODE) ? t * (2 * C)
                          : MODE == FWD ? ((ky - 1) * a.W + kx - 1) * (2 * C)
                                        : ((ky == 0) * a.OW + (kx == 0)) * (2 * C);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const bool out = !is_lin(MODE) && ((ky == 0 && ey[mt]) || (kx == 0 && ex[mt]));
#pragma unroll
            for (int c = 0; c < GC; ++c)
                copy_to_lds(out ? zp : pp[mt] + delta + (c0 + c) * 64,
                            dst + (FR + wave * FP + c * MT + mt) * 512);
        }
    };
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (!is_lin(MODE) || s < stages) copy_stage(s / SPT, s % SPT * GC, s);
    // this lane's output pixels (DGRAD: pixel (2 hy, 2 hx) of the quad), or -1
    int opix[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int p = p0 + mt * 16 + r;
        opix[mt] = p < a.P ? p : -1;
        if (MODE == DGRAD && p < a.P) {
            const unsigned row = (unsigned)p / (unsigned)a.OW;  // b OH + hy: rows 2 (b OH + hy)
            opix[mt] = (int)(2 * row * (unsigned)a.W + 2 * ((unsigned)p - row * (unsigned)a.OW));
        }
    }
    const int roff = r * 32 + ((g ^ (r >> 2)) & 3) * 8;  // the operand's place in a fragment
    int slot = 0, slot_in = D;
    floatx4 acc[MT][NT];
    auto clear = [&] {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto add_tap = [&](int t) {
#pragma unroll
        for (int c = 0; c < SPT; ++c) {
            // the wave's copies of this stage have arrived (OPS: the least a later stage issues),
            // then everyone's; and everyone has read the slot that the next copies overwrite
            constexpr int OPS = FR / 4 + FP;
            if (t * SPT + c + D - 1 < stages) stage_barrier<(D - 1) * OPS>();
            else stage_barrier<0>();
            const u16 *sw = s_st + slot * SLOT + roff, *sp = sw + (FR + wave * FP) * 512;
            bf16x8 wf[NT], pf[MT];
            auto read_chunk = [&](int k) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    wf[nt] = *reinterpret_cast<const bf16x8 *>(sw + (k * NT + nt) * 512);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    pf[mt] = *reinterpret_cast<const bf16x8 *>(sp + (k * MT + mt) * 512);
            };
            read_chunk(0);  // in flight while the copies are issued
            if (t * SPT + c + D < stages)
                copy_stage(t + (c + D) / SPT, (c + D) % SPT * GC, slot_in);
#pragma unroll
            for (int k = 0; k < GC; ++k) {
                if (k > 0) read_chunk(k);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            wf[nt], pf[mt], acc[mt][nt], 0, 0, 0);
            }
            if (++slot == RING) slot = 0;
            if (++slot_in == RING) slot_in = 0;
        }
    };
    if constexpr (MODE == DGRAD) {
        // Unrolled over the classes and their taps (END: one past a class's last). A loop over the
        // taps that cleared the sums after a class's last was compiled to copies of one word into all
        // of them (1 x 2 tiles of 128 and 256 channels); a loop around one took 126 us instead of
        // 117 for the second layer's three passes.
        constexpr int END[5] = {0, 1, 3, 5, 9};
#pragma unroll
        for (int cls = 0; cls < 4; ++cls) {
            clear();
#pragma unroll
            for (int t = 0; t < 9; ++t)
                if (t >= END[cls] && t < END[cls + 1]) add_tap(t);
            store_tile<MODE, MT, NT>(a, acc, opix, (cls >> 1) * a.W + (cls & 1), n0, g);
        }
    } else {
        clear();
        for (int t = 0; t < taps; ++t) add_tap(t);
        store_tile<MODE, MT, NT>(a, acc, opix, 0, n0, g);
    }
}

// The first layer (C = 8, three of them used): K = 72 is three chunks of four taps, lane group g
// reading tap 4 c + g, the weights (3 NT fragments) in registers.
template <int MT, int NT>
__global__ void __launch_bounds__(256) k_conv8(ConvArgs a, int block_tiles, int per)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.y * NT * 16;
    const auto src = __builtin_amdgcn_make_buffer_rsrc(const_cast<u16 *>(a.src), (short)0,
                                                       (int)a.src_bytes, 0x00020000);
    bf16x8 wf[3][NT];
    int delta[3];
    bool ty[3], tx[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int tap = 4 * c + g, ky = tap / 3, kx = tap - 3 * ky;
        ty[c] = ky == 0;
        tx[c] = kx == 0;
        delta[c] = tap < 9 ? ((ky - 1) * a.W + kx - 1) * 16 : 0;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            uintx4 z = {0, 0, 0, 0};
            if (tap < 9)
                z = *reinterpret_cast<const uintx4 *>(
                    a.w + ((size_t)(n0 + frag_chan<NT>(nt, r)) * 9 + tap) * 8);
            wf[c][nt] = __builtin_bit_cast(bf16x8, z);
        }
    }
    const bool last = g > 0;  // chunk 2 holds tap 8 alone (lane group 0)
    const int rb = xcd_run(blockIdx.x, gridDim.x);
    uintx4 buf[3][MT];
    int pix[MT];
    auto load_tile = [&](int bt) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int p = (bt * 4 + wave) * (MT * 16) + mt * 16 + r;
            const unsigned q = (unsigned)min(p, a.P - 1);
            const unsigned row = q / (unsigned)a.OW, px = q - row * (unsigned)a.OW;
            const unsigned b = row / (unsigned)a.OH, py = row - b * (unsigned)a.OH;
            const unsigned base = ((b * a.H + 2 * py) * a.W + 2 * px) * 16;
            pix[mt] = p < a.P ? p : -1;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool out = (ty[c] && py == 0) || (tx[c] && px == 0) || p >= a.P ||
                                 (c == 2 && last);
                buf[c][mt] = __builtin_amdgcn_raw_buffer_load_b128(
                    src, out ? OOB : base + (unsigned)delta[c], 0, 0);
            }
        }
    };
    const int end = min(block_tiles, rb * per + per);
    if (rb * per < end) load_tile(rb * per);
    for (int bt = rb * per; bt < end; ++bt) {
        floatx4 acc[MT][NT];
        int opix[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            opix[mt] = pix[mt];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                acc[mt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        wf[c][nt], __builtin_bit_cast(bf16x8, buf[c][mt]), acc[mt][nt], 0, 0, 0);
            }
        }
        if (bt + 1 < end) load_tile(bt + 1);  // in flight during the stores
        store_tile<FWD, MT, NT>(a, acc, opix, 0, n0, g);
    }
}

constexpr int N_CU = 256;

// Workgroups of the first layer walk runs of pixel tiles (cap: about what is resident at once).
void run_of(int P, int mt, int cap, int *tiles, int *grid, int *per)
{
    *tiles = (P + 64 * mt - 1) / (64 * mt);
    *grid = std::max(1, std::min(*tiles, cap));
    *per = (*tiles + *grid - 1) / *grid;
    *grid = (*tiles + *per - 1) / *per;
}

template <int MODE, int NCH, int MT, int NT>
void launch(const ConvArgs &a, hipStream_t st)
{
    const dim3 grid((a.P + 64 * MT - 1) / (64 * MT), a.N / (16 * NT));
    k_conv<MODE, NCH, MT, NT><<<grid, 256, 0, st>>>(a);
}

// The wave tile. Large tiles copy less per product (a weight fragment serves MT pixel fragments, a
// pixel fragment NT channel fragments), but a layer must give every SIMD a wave: 2 x 4 fragments
// where that leaves 1,024 waves (64 x 32 x 32 x 128 -> 256: forward 16.0 us with 2 x 4, 25.3 with
// 1 x 4; input gradient 26.6 against 30.8), else 1 x 4 (64 x 16 x 16 x 256 -> 256: 11.4 against 18.0
// with 2 x 4, 15.8 with 1 x 1), else the smallest (64 x 8 x 8 x 256 -> 256: 5.9 against 10.9 with
// 1 x 4). 4 x 4 was no faster anywhere, nor 2 x 2 for 32 channels (64 x 128 x 128 x 32 <- 64, input
// gradient: 53 us, 46 with 1 x 2).
template <int MODE, int NCH>
void launch_mn(const ConvArgs &a, hipStream_t st)
{
    auto waves = [&](int mt, int nt) {
        return (long long)((a.P + 16 * mt - 1) / (16 * mt)) * (a.N / (16 * nt));
    };
    if (a.N % 64 == 0 && waves(2, 4) >= 4 * N_CU) return launch<MODE, NCH, 2, 4>(a, st);
    if (a.N % 64 == 0 && waves(1, 4) >= 4 * N_CU) return launch<MODE, NCH, 1, 4>(a, st);
    if (a.N % 64 != 0 && a.N % 32 == 0 && waves(1, 2) >= 4 * N_CU)
        return launch<MODE, NCH, 1, 2>(a, st);
    launch<MODE, NCH, 1, 1>(a, st);
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

template <int MODE>
bool launch_c(const ConvArgs &a, int C, hipStream_t st)
{
    switch (C) {
    case 32: launch_mn<MODE, 1>(a, st); return true;
    case 64: launch_mn<MODE, 2>(a, st); return true;
    case 128: launch_mn<MODE, 4>(a, st); return true;
    case 256: launch_mn<MODE, 8>(a, st); return true;
    }
    return false;
}

// A dense layer of K inputs, as runs of the widest C that divides K: a run's stages are unrolled, its
// end costs a branch.
template <int MODE>
bool launch_lin(const uint16_t *x, long long B, int K, const uint16_t *w, const float *bias,
                const uint16_t *mask, int N, int relu, uint16_t *y, float *y32, hipStream_t st)
{
    if (B > (1 << 30) || K % 32 != 0 || N % 16 != 0) return false;
    if (!aligned16(x) || !aligned16(w) || !aligned16(mask) || !aligned16(y) || !aligned16(y32))
        return false;
    const int C = std::min(K & -K, 256);
    const ConvArgs a{x, w, bias, mask, y, y32, relu, 1, 1, 1, 1, (int)B, N, 0, K / C};
    return launch_c<MODE>(a, C, st);
}

// Buffers a 31-bit byte offset addresses (with room for a tap and an immediate past the end).
constexpr long long MAX_BYTES = (1LL << 31) - (1LL << 24);

}  // namespace

bool conv_forward_direct(hipStream_t st, const uint16_t *x, int B, int H, int W, int Cin,
                         const uint16_t *w, const float *bias, int Cout, int relu, uint16_t *y,
                         float *y32, hipError_t *err)
{
    const long long P = (long long)B * (H / 2) * (W / 2), bytes = 2LL * B * H * W * Cin;
    if (bytes > MAX_BYTES || P > (1 << 30) || Cout % 16 != 0) return false;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y) || !aligned16(y32)) return false;
    ConvArgs a{x, w, bias, nullptr, y, y32, relu, H, W, H / 2, W / 2, (int)P, Cout,
               (unsigned)bytes, 0};
    if (Cin == 8) {
        int tiles, grid, per;
        run_of(a.P, 4, 8 * N_CU, &tiles, &grid, &per);
        if (Cout % 32 == 0)
            k_conv8<4, 2><<<dim3(grid, Cout / 32), 256, 0, st>>>(a, tiles, per);
        else
            k_conv8<4, 1><<<dim3(grid, Cout / 16), 256, 0, st>>>(a, tiles, per);
    } else if (!launch_c<FWD>(a, Cin, st)) {
        return false;
    }
    *err = hipGetLastError();
    return true;
}

bool conv_backward_data_direct(hipStream_t st, const uint16_t *dz, int B, int H, int W, int Cin,
                               const uint16_t *wt, int Cout, const uint16_t *mask, uint16_t *dx,
                               hipError_t *err)
{
    const long long P = (long long)B * (H / 2) * (W / 2), bytes = 2 * P * Cout;
    if (bytes > MAX_BYTES || 4 * P > (1LL << 30) || Cin % 16 != 0) return false;
    if (!aligned16(dz) || !aligned16(wt) || !aligned16(mask) || !aligned16(dx)) return false;
    ConvArgs a{dz, wt, nullptr, mask, dx, nullptr, 0, H, W, H / 2, W / 2, (int)P, Cin,
               (unsigned)bytes, 0};
    if (!launch_c<DGRAD>(a, Cout, st)) return false;
    *err = hipGetLastError();
    return true;
}

bool linear_forward_direct(hipStream_t st, const uint16_t *x, int B, int K, const uint16_t *w,
                           const float *bias, int N, int relu, uint16_t *y, float *y32,
                           hipError_t *err)
{
    if (!launch_lin<LFWD>(x, B, K, w, bias, nullptr, N, relu, y, y32, st)) return false;
    *err = hipGetLastError();
    return true;
}

bool linear_backward_data_direct(hipStream_t st, const uint16_t *dz, int B, int N,
                                 const uint16_t *wt, int K, const uint16_t *mask, uint16_t *dx,
                                 hipError_t *err)
{
    if (!launch_lin<LDGRAD>(dz, B, N, wt, nullptr, mask, K, 0, dx, nullptr, st)) return false;
    *err = hipGetLastError();
    return true;
}

}  // namespace dbmp_cnn
