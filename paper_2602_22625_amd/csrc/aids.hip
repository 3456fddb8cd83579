// Optimisation aids around the rasteriser (Sec. 3.2, Eqs. 8-9; Supp. Table S1, Sec. S1.4.2):
// Gaussian blur of the bitmaps, structure-aware initialisation, the noise canvas, the
// spatial-constraint loss and the re-initialisation of transparent primitives. Declared in
// include/dbmp_aids.h. All of it is elementwise, stencil or scan work: bound by memory, laid out
// for coalesced rows, with LDS staging where a value is read by many neighbours.
#include "dbmp_aids.h"
#include "dbmp_internal.h"
#include "diffbmp.h"
#include "sa_layout.h"

#include <limits.h>
#include <math.h>

#include <algorithm>

namespace dbmp {
namespace {

// ------------------------------------------------------------------------------------------
// Gaussian blur (Sec. 3.2.1): a band of output rows per workgroup. The band's input rows plus
// r rows above and below are staged in LDS (as float32, between r columns of zeros), blurred along
// x into a second LDS buffer, then along y into the output. Waves take rows, lanes columns: no
// division. Bands are short where that fills the chip (a 64 x 128 x 128 atlas, 16 rows: 512
// workgroups): bands as tall as LDS holds left one workgroup per compute unit, and each of its
// threads 24 pixels of dependent LDS reads: 33 us for a 64 x 128 x 128 bfloat16 atlas, 10 us now. They
// are cut evenly and never taller than the bitmap (1,024 x 128 x 128 float32: 97 us cut into
// 42, 42, 42 and 2 rows, 62 into four of 32; 4,096 x 32 x 32 at radius 15: 197 us as bands of 64 rows,
// 72 as 32).
// Bitmaps of up to 32 columns give a wave several rows (60,000 of 8 x 8: 224 us with one, 32 now).
// ------------------------------------------------------------------------------------------
constexpr int BLUR_RMAX = 16;
constexpr int BLUR_LDS_BYTES = 48 * 1024;

struct BlurTaps {
    float w[2 * BLUR_RMAX + 1];
    int r;
};

template <typename TexT> __device__ __forceinline__ TexT from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ uint16_t from_f32<uint16_t>(float v)
{
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)0x7fc0;  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                // round to nearest even
    return (uint16_t)(u >> 16);
}
template <> __device__ __forceinline__ _Float16 from_f32<_Float16>(float v)
{
    return (_Float16)v;  // round to nearest even
}

// RAD > 0: the radius at compile time (3 is sigma = 1, the method's), so that a pixel's LDS reads
// are all in flight; 0: t.r.
template <typename TexT, int RAD, bool NARROW>
__global__ void __launch_bounds__(256)
k_blur(const TexT *__restrict__ in, TexT *__restrict__ out, int Hb, int Wb, int band, int lg_,
       BlurTaps t)
{
    extern __shared__ float sh[];
    const int r = RAD ? RAD : t.r;
    const int b = blockIdx.y, y0 = blockIdx.x * band, rows = band + 2 * r;
    const int pitch = Wb + 2 * r;
    // a wave takes 1 << (6 - lg) rows of 1 << lg columns: of bitmaps of up to 32 columns (NARROW),
    // several rows
    const int lg = NARROW ? lg_ : 6;
    const int row0 = (int)threadIdx.x >> lg, col0 = (int)threadIdx.x & ((1 << lg) - 1);
    const int nrow = 256 >> lg, ncol = 1 << lg;
    float *raw = sh;                  // rows y0 - r .. y0 + band + r - 1 (zero outside the bitmap)
    float *hor = sh + rows * pitch;   // the same rows blurred along x
    const TexT *src = in + (size_t)b * Hb * Wb;
    for (int y = row0; y < rows; y += nrow) {
        const int yy = y0 - r + y;
        const bool in_y = yy >= 0 && yy < Hb;
        for (int x = col0; x < pitch; x += ncol) {
            const int xx = x - r;
            raw[y * pitch + x] =
                in_y && xx >= 0 && xx < Wb ? texel<TexT>(src[(size_t)yy * Wb + xx]) : 0.f;
        }
    }
    __syncthreads();
    for (int y = row0; y < rows; y += nrow)
        for (int x = col0; x < Wb; x += ncol) {
            const float *p = raw + y * pitch + x;
            float acc = 0.f;
            for (int d = 0; d <= 2 * r; ++d) acc = fmaf(t.w[d], p[d], acc);
            hor[y * Wb + x] = acc;
        }
    __syncthreads();
    TexT *dst = out + (size_t)b * Hb * Wb;
    for (int y = row0; y < min(band, Hb - y0); y += nrow)
        for (int x = col0; x < Wb; x += ncol) {
            const float *p = hor + y * Wb + x;
            float acc = 0.f;
            for (int d = 0; d <= 2 * r; ++d) acc = fmaf(t.w[d], p[d * Wb], acc);
            dst[(size_t)(y0 + y) * Wb + x] = from_f32<TexT>(acc);
        }
}

// ------------------------------------------------------------------------------------------
// Structure-aware initialisation (Sec. 3.2.2)
// ------------------------------------------------------------------------------------------
constexpr int LV_HMAX = 7;      // largest window half-width (15 x 15)
constexpr int BSUM_LDS = 2048;  // block totals the sampler scans in LDS

// Ordering of non-negative doubles = ordering of their bit patterns as unsigned integers.
__device__ __forceinline__ unsigned long long dbits(double x)
{
    return (unsigned long long)__double_as_longlong(x);
}

// a / n for an integer n, given inv = 1 / n rounded to nearest: one Newton step on the quotient,
// which is then a / n rounded to nearest (so that a flat region's variance is exactly 0, which a
// product with inv would miss).
__device__ __forceinline__ double div_n(double a, double n, double inv)
{
    const double q = a * inv;
    return fma(fma(-q, n, a), inv, q);
}

// Sum of N values, pairwise.
template <int N, typename At>
__device__ __forceinline__ double tree_sum(At at, int i0 = 0)
{
    if constexpr (N == 0) return 0.0;
    else if constexpr (N == 1) return at(i0);
    else {
        constexpr int K = N > 4 ? 4 : N > 2 ? 2 : 1;
        return tree_sum<K>(at, i0) + tree_sum<N - K>(at, i0 + K);
    }
}

// The local variance (float64) over the (2 h + 1)^2 window clipped to the image, 64 columns by NW R
// rows per workgroup of NW waves. Per channel: each row's window sums of values and squares along x into LDS
// (values straight from memory: a window's loads hit the same lines), then each wave adds up
// 2 h + 1 rows of them for its R rows of outputs: about 45 float64 operations per pixel and channel
// for a 7 x 7 window, where summing the window afresh took 98 and as many conversions: 58 us at
// 2048 x 2048, 176 before. Bound by latency (the operations alone would take about 27 us), so waves
// in flight count: 8 waves of 4 rows at 5 per SIMD, where 4 waves of 8 rows (3 per SIMD) took 67 and
// 16 of 2 rows 87; the three channels' loop is kept rolled, which the compiler would undo for the
// small windows at twice the registers (3 x 3: 86 us for the whole start against 54). Keeping the
// row sums in registers instead took 62 us with strips of 4 rows, 79 with 8, and spilled for the
// larger windows.
template <int HW, int R, int NW>
__global__ void __launch_bounds__(64 * NW)
k_local_var(const float *__restrict__ img, int H, int W, double *__restrict__ lv,
            unsigned long long *__restrict__ bmm)
{
    constexpr int WIN = 2 * HW + 1, ROWS = NW * R + 2 * HW;
    __shared__ double s1[ROWS][LV_W], s2[ROWS][LV_W];
    __shared__ double s_inv[WIN * WIN + 1];  // reciprocals of the window's pixel counts
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i <= WIN * WIN; i += 64 * NW) s_inv[i] = 1.0 / max(i, 1);
    const int bx = blockIdx.x * LV_W, by = blockIdx.y * NW * R, x = bx + lane;
    const size_t plane = (size_t)H * W;
    const bool inside = bx >= HW && bx + LV_W + HW <= W;  // no lane's window leaves the image in x
    const int nx = max(min(x + HW, W - 1) - max(x - HW, 0) + 1, 1);
    double v[R];
#pragma unroll
    for (int o = 0; o < R; ++o) v[o] = 0.0;
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
        if (c) __syncthreads();  // the previous channel's sums are read
#pragma unroll 2
        for (int q = wave; q < ROWS; q += NW) {
            const int y = by - HW + q;
            float f[WIN];
#pragma unroll
            for (int k = 0; k < WIN; ++k) f[k] = 0.f;
            if (y >= 0 && y < H) {
                const float *row = img + c * plane + (size_t)y * W;
#pragma unroll
                for (int k = 0; k < WIN; ++k) {
                    const int xx = x + k - HW;
                    if (inside) f[k] = row[xx];
                    else if (xx >= 0 && xx < W) f[k] = row[xx];
                }
            }
            s1[q][lane] = tree_sum<WIN>([&](int k) { return (double)f[k]; });
            double sq = (double)f[0] * (double)f[0];  // squares of float32 values are exact
#pragma unroll
            for (int k = 1; k < WIN; ++k) sq = fma((double)f[k], (double)f[k], sq);
            s2[q][lane] = sq;
        }
        __syncthreads();
        double a1[R + 2 * HW], a2[R + 2 * HW];
#pragma unroll
        for (int k = 0; k < R + 2 * HW; ++k) {
            a1[k] = s1[wave * R + k][lane];
            a2[k] = s2[wave * R + k][lane];
        }
#pragma unroll
        for (int o = 0; o < R; ++o) {
            const int y = by + wave * R + o;
            const int ni = nx * max(min(y + HW, H - 1) - max(y - HW, 0) + 1, 1);
            const double n = ni, inv = s_inv[ni];
            const double m = div_n(tree_sum<WIN>([&](int k) { return a1[o + k]; }), n, inv);
            v[o] += div_n(tree_sum<WIN>([&](int k) { return a2[o + k]; }), n, inv) - m * m;
        }
    }
    unsigned long long lo = 0x7ff0000000000000ull, hi = 0ull;
#pragma unroll
    for (int o = 0; o < R; ++o) {
        const int y = by + wave * R + o;
        if (x >= W || y >= H) continue;
        // the one-pass form can round a zero variance below zero
        const double d = fmax(div_n(v[o], 3.0, 1.0 / 3.0), 0.0);
        lv[(size_t)y * W + x] = d;
        const unsigned long long u = dbits(d);
        lo = u < lo ? u : lo;
        hi = u > hi ? u : hi;
    }
    // the block's min / max of the map (bit patterns of non-negative doubles), written to its
    // own slot (no same-address atomics across the grid)
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    __shared__ unsigned long long s_lo[NW], s_hi[NW];
    if (lane == 0) {
        s_lo[wave] = lo;
        s_hi[wave] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NW; ++w) {
            lo = s_lo[w] < lo ? s_lo[w] : lo;
            hi = s_hi[w] > hi ? s_hi[w] : hi;
        }
        const size_t b = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
        bmm[2 * b] = lo;
        bmm[2 * b + 1] = hi;
    }
}

// The map's min / max from the blocks' slots: one workgroup.
__global__ void __launch_bounds__(1024)
k_lv_minmax(const unsigned long long *__restrict__ bmm, int nblocks,
            unsigned long long *__restrict__ minmax)
{
    unsigned long long lo = 0x7ff0000000000000ull, hi = 0ull;
    for (int b = threadIdx.x; b < nblocks; b += 1024) {
        lo = bmm[2 * b] < lo ? bmm[2 * b] : lo;
        hi = bmm[2 * b + 1] > hi ? bmm[2 * b + 1] : hi;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    __shared__ unsigned long long s_lo[16], s_hi[16];
    if ((threadIdx.x & 63) == 0) {
        s_lo[threadIdx.x >> 6] = lo;
        s_hi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            lo = s_lo[w] < lo ? s_lo[w] : lo;
            hi = s_hi[w] > hi ? s_hi[w] : hi;
        }
        minmax[0] = lo;
        minmax[1] = hi;
    }
}

// The integer sampling weight of a pixel from its NLV (below 2^24 + 1).
__device__ __forceinline__ uint32_t sample_weight(float nf, double base)
{
    const double wd = base + (1.0 - base) * (double)nf;  // built without contraction
    return (uint32_t)floor(wd * 16777216.0);
}

// NLV (float32, the caller's map) and the sums of the sampling weights computed from it, in two
// levels: inclusive sums over the workgroup's groups of 64 pixels, and its total. The sampler
// recomputes a group's weights from the map: writing and scanning one int64 per pixel instead
// moved 136 MB more at 2048 x 2048 (59 us for this kernel and the scan's three, 15 us now). Every
// workgroup reduces the map's min / max from the nslots of k_local_var (or of k_lv_minmax) itself.
__global__ void __launch_bounds__(256)
k_nlv(const double *__restrict__ lv, long long n, const unsigned long long *__restrict__ bmm,
      int nslots, double base, float *__restrict__ nlv_out, long long *__restrict__ gsum,
      long long *__restrict__ bsum)
{
    __shared__ unsigned long long s_lo[4], s_hi[4];
    __shared__ uint32_t s_g[NLV_BLOCK / NLV_GROUP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long p0 = (long long)blockIdx.x * NLV_BLOCK;
    double d[4][4];  // this thread's pixels, requested before the reduction below
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const long long p = p0 + k * 1024 + threadIdx.x * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) d[k][j] = p + j < n ? lv[p + j] : 0.0;
    }
    unsigned long long lo = 0x7ff0000000000000ull, hi = 0ull;
    for (int b = threadIdx.x; b < nslots; b += 256) {
        lo = bmm[2 * b] < lo ? bmm[2 * b] : lo;
        hi = bmm[2 * b + 1] > hi ? bmm[2 * b + 1] : hi;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long a = __shfl_xor(lo, o), b = __shfl_xor(hi, o);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if (lane == 0) {
        s_lo[wave] = lo;
        s_hi[wave] = hi;
    }
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        lo = s_lo[w] < lo ? s_lo[w] : lo;
        hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    const double dlo = __longlong_as_double((long long)lo);
    const double dhi = __longlong_as_double((long long)hi);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const long long p = p0 + k * 1024 + threadIdx.x * 4;
        float f[4];
        uint32_t w = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double q = dhi > dlo ? (d[k][j] - dlo) / (dhi - dlo) : 0.0;
            f[j] = (float)q;
            if (p + j < n) w += sample_weight(f[j], base);
        }
        if (p + 3 < n && ((uintptr_t)nlv_out & 15) == 0) {
            *reinterpret_cast<float4 *>(nlv_out + p) = make_float4(f[0], f[1], f[2], f[3]);
        } else {
            for (int j = 0; j < 4; ++j)
                if (p + j < n) nlv_out[p + j] = f[j];
        }
        for (int o = 8; o > 0; o >>= 1) w += __shfl_xor(w, o);  // 16 lanes: 64 pixels, below 2^31
        if ((lane & 15) == 0) s_g[k * 16 + (threadIdx.x >> 4)] = w;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        long long x = s_g[threadIdx.x];
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        gsum[(size_t)blockIdx.x * 64 + threadIdx.x] = x;
        if (threadIdx.x == 63) bsum[blockIdx.x] = x;
    }
}

__device__ __forceinline__ long long wave_incl_scan(long long x, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        const long long y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

// Inclusive scan of the block totals in place, one workgroup (more totals than the sampler scans
// itself).
__global__ void __launch_bounds__(1024) k_scan_sums(long long *__restrict__ bsum, int nb)
{
    __shared__ long long wsum[16];
    __shared__ long long carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int i = b0 + threadIdx.x;
        const long long x = i < nb ? bsum[i] : 0;
        const long long incl = wave_incl_scan(x, lane);
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        long long off = carry;
        for (int q = 0; q < wave; ++q) off += wsum[q];
        if (i < nb) bsum[i] = incl + off;
        __syncthreads();
        if (threadIdx.x == 1023) carry = incl + off;
        __syncthreads();
    }
}

// One primitive per lane: inverse-CDF draw of its pixel, then its parameter row. The pixel is found
// from the block totals (scanned in LDS, or already scanned in memory: SCANNED), the block's sums
// over groups of 64 pixels, and the group's weights (65,536 draws from 2048 x 2048: 13 us, 17 with
// 22 dependent steps through the whole cumulative sum).
template <bool SCANNED>
__global__ void __launch_bounds__(256)
k_sa_sample(const long long *__restrict__ gsum, const long long *__restrict__ bsum, int nb,
            long long n, double base, const float *__restrict__ nlv, const float *__restrict__ img,
            int H, int W, const float *__restrict__ u_pos, const float *__restrict__ u_theta,
            const float *__restrict__ z, int N, double s_min, double s_max, double nu_init,
            double sigma_c, float *__restrict__ params)
{
    __shared__ long long s_b[SCANNED ? 1 : BSUM_LDS];
    __shared__ long long s_w[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if constexpr (!SCANNED) {  // inclusive sums of the totals
        constexpr int PER = BSUM_LDS / 256;
        long long v[PER], run = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int b = threadIdx.x * PER + k;
            v[k] = b < nb ? bsum[b] : 0;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = run += v[k];
        const long long incl = wave_incl_scan(run, lane);
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        long long off = incl - run;
        for (int w = 0; w < wave; ++w) off += s_w[w];
#pragma unroll
        for (int k = 0; k < PER; ++k) s_b[threadIdx.x * PER + k] = v[k] + off;
        __syncthreads();
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    auto total_to = [&](int b) { return SCANNED ? bsum[b] : s_b[b]; };
    const long long total = total_to(nb - 1);
    long long t = (long long)floor((double)u_pos[i] * (double)total);
    if (t >= total) t = total - 1;
    int lo = 0, hi = nb - 1;  // first block whose inclusive total exceeds t
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (total_to(mid) > t) hi = mid; else lo = mid + 1;
    }
    const int blk = lo;
    t -= blk ? total_to(blk - 1) : 0;
    // first group whose inclusive sum exceeds t: the entries at most t are counted, eight at a
    // time (independent loads)
    const long long *gs = gsum + (size_t)blk * 64;
    int gr = 0;
#pragma unroll
    for (int k = 0; k < 7; ++k) gr += gs[8 * k + 7] <= t ? 8 : 0;
    const int g8 = gr;
#pragma unroll
    for (int k = 0; k < 7; ++k) gr += gs[g8 + k] <= t ? 1 : 0;
    t -= gr ? gs[gr - 1] : 0;
    // first pixel of the group whose cumulative weight exceeds t
    const long long p0 = (long long)blk * NLV_BLOCK + gr * NLV_GROUP;
    long long run = 0;
    int at = 0;
    if (p0 + NLV_GROUP <= n && ((uintptr_t)nlv & 15) == 0) {
        float4 q[NLV_GROUP / 4];
#pragma unroll
        for (int k = 0; k < NLV_GROUP / 4; ++k)
            q[k] = *reinterpret_cast<const float4 *>(nlv + p0 + 4 * k);
#pragma unroll
        for (int k = 0; k < NLV_GROUP; ++k) {
            run += sample_weight((&q[k / 4].x)[k % 4], base);
            at += run <= t ? 1 : 0;
        }
    } else {
        for (int k = 0; k < NLV_GROUP && p0 + k < n; ++k) {
            run += sample_weight(nlv[p0 + k], base);
            at += run <= t ? 1 : 0;
        }
    }
    const int p = (int)p0 + at, x = p % W, y = p / W;
    const double s = s_max - (s_max - s_min) * (double)nlv[p];
    float *row = params + (size_t)i * 8;
    row[0] = (float)x;
    row[1] = (float)y;
    row[2] = (float)log(s);
    row[3] = (float)(2.0 * M_PI * (double)u_theta[i]);
    row[4] = (float)nu_init;
    const size_t plane = (size_t)H * W;
    for (int c = 0; c < 3; ++c) {
        double v = (double)img[c * plane + p] + sigma_c * (double)z[(size_t)i * 3 + c];
        v = fmin(fmax(v, 1e-3), 1.0 - 1e-3);
        row[5 + c] = (float)log(v / (1.0 - v));
    }
}

// ------------------------------------------------------------------------------------------
// Noise canvas (Eq. 8): Philox4x64-10, one block per pixel
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void philox4x64_10(unsigned long long (&c)[4], unsigned long long k0,
                                              unsigned long long k1)
{
    const unsigned long long M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const unsigned long long W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const unsigned long long hi0 = __umul64hi(M0, c[0]), lo0 = M0 * c[0];
        const unsigned long long hi1 = __umul64hi(M1, c[2]), lo1 = M1 * c[2];
        const unsigned long long n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
        k0 += W0;
        k1 += W1;
    }
}

__global__ void __launch_bounds__(256)
k_noise(unsigned long long seed, unsigned long long iter, long long npix,
        float *__restrict__ bg)
{
    const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
    if (p >= npix) return;
    unsigned long long c[4] = {(unsigned long long)p, iter, 0ull, 0ull};
    philox4x64_10(c, seed, 0ull);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) bg[ch * npix + p] = (float)(c[ch] >> 40) * 0x1p-24f;
}

// ------------------------------------------------------------------------------------------
// Spatial-constraint loss (Eq. 9) and re-initialisation (Supp. Sec. S1.4.2)
// ------------------------------------------------------------------------------------------
// A grid of at most CONSTRAINT_BLOCKS workgroups strides over the pixels, four at a time (V = 4:
// 16-byte loads and stores) where the planes allow; each workgroup adds its share of the loss with
// one atomic. Atomics on one address take about 14 ns each, one after the other: with 1,920
// workgroups of one pixel per thread they were all of the 27.9 us that 768 x 640 took.
constexpr int CONSTRAINT_BLOCKS = 256;

template <int V>
__global__ void __launch_bounds__(256)
k_constraint(const float *__restrict__ I, const float *__restrict__ A,
             const float *__restrict__ t, const float *__restrict__ ta, long long npix,
             float lam, float *__restrict__ gI, float *__restrict__ gA, float *__restrict__ loss)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    float acc = 0.f;
    const float inv3 = 1.f / (3.f * (float)npix), inv1 = 1.f / (float)npix;
    auto at = [](const float *p) { return *reinterpret_cast<const vec *>(p); };
    for (long long p = ((long long)blockIdx.x * 256 + threadIdx.x) * V; p < npix;
         p += (long long)gridDim.x * 256 * V) {
        const vec tv = at(ta + p), av = at(A + p);
        vec iv[3], cv[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            iv[c] = at(I + c * npix + p);
            cv[c] = at(t + c * npix + p);
        }
        vec ga;
#pragma unroll
        for (int k = 0; k < V; ++k) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float d = tv[k] > 0.f ? iv[c][k] - cv[c][k] : 0.f;
                iv[c][k] = 2.f * d * inv3;
                acc = fmaf(d * d, inv3, acc);
            }
            const float e = av[k] - tv[k];
            ga[k] = 2.f * lam * e * inv1;
            acc = fmaf(lam * e * e, inv1, acc);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) *reinterpret_cast<vec *>(gI + c * npix + p) = iv[c];
        *reinterpret_cast<vec *>(gA + p) = ga;
    }
    if (!loss) return;
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    __shared__ float s_acc[4];
    if ((threadIdx.x & 63) == 0) s_acc[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float tot = s_acc[0] + s_acc[1] + s_acc[2] + s_acc[3];
        if (tot != 0.f) atomicAdd(loss, tot);
    }
}

__global__ void __launch_bounds__(256)
k_reinit(float *__restrict__ params, float *__restrict__ m, float *__restrict__ v,
         const float *__restrict__ prop, int N, double logit_thr, int *__restrict__ count)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N || !((double)params[(size_t)i * 8 + 4] < logit_thr)) return;
    for (int q = 0; q < 8; ++q) {
        params[(size_t)i * 8 + q] = prop[(size_t)i * 8 + q];
        if (m) m[(size_t)i * 8 + q] = 0.f;
        if (v) v[(size_t)i * 8 + q] = 0.f;
    }
    if (count) atomicAdd(count, 1);
}

// HW: the build whose window half width is h.
template <int HW = 0>
void launch_local_var(hipStream_t st, const dim3 &grid, int rows, const float *img, int H, int W,
                      int h, double *lv, unsigned long long *bmm)
{
    if (h != HW) {
        if constexpr (HW < LV_HMAX)
            launch_local_var<HW + 1>(st, grid, rows, img, H, W, h, lv, bmm);
        return;
    }
    // 32 rows as 8 waves of 4, or 4 of 8 for windows of 13 and 15, whose waves read many more rows
    // than they share (7 x 7 at 2048 x 2048: 80 and 88 us for the start; 15 x 15: 164 and 153)
    constexpr int R = HW < 6 ? 4 : 8, NW = 32 / R;
    if (rows == 32) k_local_var<HW, R, NW><<<grid, 64 * NW, 0, st>>>(img, H, W, lv, bmm);
    else k_local_var<HW, 2, 4><<<grid, 256, 0, st>>>(img, H, W, lv, bmm);
}

int launched() { return hipGetLastError() == hipSuccess ? DBMP_OK : DBMP_EHIP; }

}  // namespace
}  // namespace dbmp

using namespace dbmp;

extern "C" {

int dbmp_blur_atlas(dbmp_aids_stream stream, const void *atlas, int B, int Hb, int Wb,
                    int atlas_dtype, float sigma, float truncate, void *out)
{
    if (!atlas || !out || B < 1 || Hb < 1 || Wb < 1 || Wb > 1024) return DBMP_EINVAL;
    if (atlas_dtype != DBMP_F32 && atlas_dtype != DBMP_BF16 && atlas_dtype != DBMP_F16)
        return DBMP_EINVAL;
    if (!(sigma > 0.f && sigma <= 8.f) || !(truncate > 0.f)) return DBMP_EINVAL;
    const int r = (int)(truncate * (double)sigma + 0.5);
    if (r > BLUR_RMAX) return DBMP_EINVAL;
    const size_t esz = atlas_dtype == DBMP_F32 ? 4 : 2;
    const char *a = (const char *)atlas, *o = (const char *)out;
    const size_t bytes = esz * (size_t)B * Hb * Wb;
    if (a < o + bytes && o < a + bytes) return DBMP_EINVAL;  // overlapping buffers
    BlurTaps t{};
    t.r = r;
    double w[2 * BLUR_RMAX + 1], sum = 0.0;
    for (int d = -r; d <= r; ++d) sum += (w[d + r] = exp(-(double)d * d / (2.0 * sigma * sigma)));
    for (int d = -r; d <= r; ++d) t.w[d + r] = (float)(w[d + r] / sum);
    // The sizes accepted are those of which a row fits in 48 KB without the columns of zeros; with
    // them a band takes at most 60 KB (radius 16, 64 columns, 64 rows).
    int band = BLUR_LDS_BYTES / (8 * Wb) - 2 * r;
    if (band < 1) return DBMP_EINVAL;  // the band does not fit in LDS
    const long long fill = ((long long)B * Hb + 511) / 512;  // rows per workgroup of 512
    band = (int)std::min<long long>(std::min({band, 64, Hb}), std::max<long long>(fill, 8));
    const int bands = (Hb + band - 1) / band;
    band = (Hb + bands - 1) / bands;
    int lg = 6;  // log2 of a wave's columns
    while (lg > 0 && 1 << (lg - 1) >= Wb) --lg;
    const size_t lds = 4 * (size_t)(band + 2 * r) * (2 * Wb + 2 * r);
    const dim3 grid(bands, B);
    hipStream_t st = (hipStream_t)stream;
    auto run = [&](auto texel_of, auto kern) {
        using TexT = decltype(texel_of);
        kern<<<grid, 256, lds, st>>>((const TexT *)atlas, (TexT *)out, Hb, Wb, band, lg, t);
    };
    auto run_r = [&](auto texel_of) {
        using TexT = decltype(texel_of);
        if (lg < 6) run(texel_of, r == 3 ? k_blur<TexT, 3, true> : k_blur<TexT, 0, true>);
        else run(texel_of, r == 3 ? k_blur<TexT, 3, false> : k_blur<TexT, 0, false>);
    };
    if (atlas_dtype == DBMP_F32) run_r(float{});
    else if (atlas_dtype == DBMP_F16) run_r(_Float16{});
    else run_r(uint16_t{});
    return launched();
}

long long dbmp_sa_init_workspace_bytes(int H, int W)
{
    if (H < 1 || W < 1 || (long long)H * W >= INT_MAX) return -1;
    return (long long)sa_layout(H, W).total;
}

int dbmp_sa_init(dbmp_aids_stream stream, const float *target, int H, int W, int win,
                 double base, const float *u_pos, const float *u_theta, const float *z_col, int N,
                 double s_min, double s_max, double nu_init, double sigma_c, void *workspace,
                 long long workspace_bytes, float *nlv_out, float *params_out)
{
    if (!target || !workspace || !nlv_out || H < 1 || W < 1 || N < 0) return DBMP_EINVAL;
    if ((long long)H * W >= INT_MAX) return DBMP_EINVAL;
    if (N > 0 && (!u_pos || !u_theta || !z_col || !params_out)) return DBMP_EINVAL;
    if (win < 1 || win > 2 * LV_HMAX + 1 || !(win & 1)) return DBMP_EINVAL;
    if (!(base >= 0.0 && base <= 1.0) || !(s_min > 0.0) || !(s_max >= s_min)) return DBMP_EINVAL;
    if (!(sigma_c >= 0.0) || ((uintptr_t)workspace & 15)) return DBMP_EINVAL;
    const long long npix = (long long)H * W;
    const SaLayout L = sa_layout(H, W);
    if (workspace_bytes < (long long)L.total) return DBMP_EINVAL;
    char *ws = (char *)workspace;
    auto *minmax = (unsigned long long *)(ws + L.minmax);
    auto *bmm = (unsigned long long *)(ws + L.bmm);
    auto *lv = (double *)(ws + L.lv);
    auto *gsum = (long long *)(ws + L.gsum);
    auto *bsum = (long long *)(ws + L.bsum);
    hipStream_t st = (hipStream_t)stream;
    int lh = H, lw = W;
    lv_shape(lh, lw);
    const int rows = lv_rows(lh, lw);
    const dim3 lvg((lw + LV_W - 1) / LV_W, (lh + rows - 1) / rows);
    launch_local_var(st, lvg, rows, target, lh, lw, win / 2, lv, bmm);
    int nslots = (int)(lvg.x * lvg.y);
    if (nslots > 2048) {  // too many for every workgroup of k_nlv to read
        k_lv_minmax<<<1, 1024, 0, st>>>(bmm, nslots, minmax);
        bmm = minmax;
        nslots = 1;
    }
    const int nb = (int)((npix + NLV_BLOCK - 1) / NLV_BLOCK);
    k_nlv<<<nb, 256, 0, st>>>(lv, npix, bmm, nslots, base, nlv_out, gsum, bsum);
    if (N > 0) {
        auto run = [&](auto kern) {
            kern<<<(N + 255) / 256, 256, 0, st>>>(gsum, bsum, nb, npix, base, nlv_out, target, H, W,
                                                  u_pos, u_theta, z_col, N, s_min, s_max, nu_init,
                                                  sigma_c, params_out);
        };
        if (nb > BSUM_LDS) {
            k_scan_sums<<<1, 1024, 0, st>>>(bsum, nb);
            run(k_sa_sample<true>);
        } else {
            run(k_sa_sample<false>);
        }
    }
    return launched();
}

int dbmp_noise_canvas(dbmp_aids_stream stream, unsigned long long seed,
                      unsigned long long iteration, int H, int W, float *bg_out)
{
    if (!bg_out || H < 1 || W < 1 || (long long)H * W >= INT_MAX) return DBMP_EINVAL;
    const long long npix = (long long)H * W;
    k_noise<<<(unsigned)((npix + 255) / 256), 256, 0, (hipStream_t)stream>>>(seed, iteration,
                                                                               npix, bg_out);
    return launched();
}

int dbmp_constraint_loss(dbmp_aids_stream stream, const float *image, const float *alpha,
                         const float *target, const float *target_alpha, int H, int W,
                         float lambda, float *dL_dimage, float *dL_dalpha, float *loss)
{
    if (!image || !alpha || !target || !target_alpha || !dL_dimage || !dL_dalpha) return DBMP_EINVAL;
    if (H < 1 || W < 1 || (long long)H * W >= INT_MAX || !(lambda >= 0.f)) return DBMP_EINVAL;
    const long long npix = (long long)H * W;
    const uintptr_t all = (uintptr_t)image | (uintptr_t)alpha | (uintptr_t)target |
                          (uintptr_t)target_alpha | (uintptr_t)dL_dimage | (uintptr_t)dL_dalpha;
    const int v = npix % 4 == 0 && (all & 15) == 0 ? 4 : 1;  // whole 16-byte groups in every plane
    const long long blocks =
        std::min<long long>((npix / v + 255) / 256, CONSTRAINT_BLOCKS);
    auto run = [&](auto kern) {
        kern<<<(unsigned)blocks, 256, 0, (hipStream_t)stream>>>(image, alpha, target, target_alpha,
                                                                npix, lambda, dL_dimage, dL_dalpha,
                                                                loss);
    };
    if (v == 4) run(k_constraint<4>);
    else run(k_constraint<1>);
    return launched();
}

int dbmp_reinit_transparent(dbmp_aids_stream stream, float *params, float *m, float *v,
                            const float *proposal, int N, double threshold, int32_t *count)
{
    if (N < 0 || (N > 0 && (!params || !proposal))) return DBMP_EINVAL;
    if (!(threshold > 0.0 && threshold < 1.0)) return DBMP_EINVAL;
    if (N == 0) return DBMP_OK;
    const double thr = threshold;
    k_reinit<<<(N + 255) / 256, 256, 0, (hipStream_t)stream>>>(params, m, v, proposal, N,
                                                              log(thr / (1.0 - thr)), count);
    return launched();
}

}  // extern "C"
