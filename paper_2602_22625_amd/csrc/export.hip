// Layer export (Sec. 3.1.3; Supp. "PSD export"), declared in include/dbmp_export.h.
//
// Stage 1: one lane per primitive finds the box of export pixels its bilinear support can reach
// (float64, as the binning), then one workgroup turns the box areas into offsets (an exclusive
// int64 scan). Stage 2: a workgroup per primitive (or, of many primitives, per few of them) walks its
// box's export pixels; each lane evaluates a pixel's alpha (the forward's arithmetic: float64 coordinates, float32 bilinear
// sample) and writes it into the primitive's own packed box. Every output value has exactly one
// writer, so no atomics.
#include "dbmp_export.h"
#include "dbmp_internal.h"
#include "diffbmp.h"

#include <limits.h>
#include <math.h>

#include <algorithm>

namespace dbmp {
namespace {

// A box as the caller's int32 [N, 4] holds it: one 16-byte access, at any 4-byte address.
typedef int BoxWords __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ int4 box_at(const BoxWords *__restrict__ boxes, long long i)
{
    const BoxWords b = boxes[i];
    return make_int4(b.x, b.y, b.z, b.w);
}

// Canvas point of export pixel X: (X + 0.5) / rho - 0.5; export coordinate of canvas point x:
// rho (x + 0.5) - 0.5.
__global__ void __launch_bounds__(256)
k_export_boxes(const float *__restrict__ params, int N, int Hb, int Wb, int HH, int WW,
               double rho, BoxWords *__restrict__ boxes)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const float *p = params + (size_t)i * 8;
    bool fin = true;
    for (int q = 0; q < 8; ++q) fin = fin && isfinite(p[q]);
    int x0 = 0, y0 = 0, w = 0, h = 0;
    const double s = exp((double)p[2]);
    if (fin && s > 0.0 && isfinite(s)) {
        double st, ct;
        sincos((double)p[3], &st, &ct);
        const double cu = 0.5 * (Wb - 1), cv = 0.5 * (Hb - 1);
        double xmin = 1e300, xmax = -1e300, ymin = 1e300, ymax = -1e300;
        for (int c = 0; c < 4; ++c) {  // corners of -1 <= U <= Wb, -1 <= V <= Hb
            const double U = (c & 1) ? (double)Wb : -1.0, V = (c & 2) ? (double)Hb : -1.0;
            const double u = U / cu - 1.0, v = V / cv - 1.0;
            const double X = rho * ((double)p[0] + s * (ct * u - st * v) + 0.5) - 0.5;
            const double Y = rho * ((double)p[1] + s * (st * u + ct * v) + 0.5) - 0.5;
            xmin = fmin(xmin, X); xmax = fmax(xmax, X);
            ymin = fmin(ymin, Y); ymax = fmax(ymax, Y);
        }
        const double mg = 1e-3;  // conservative against rounding
        const double fx0 = fmax(ceil(xmin - mg), 0.0), fx1 = fmin(floor(xmax + mg), WW - 1.0);
        const double fy0 = fmax(ceil(ymin - mg), 0.0), fy1 = fmin(floor(ymax + mg), HH - 1.0);
        if (fx0 <= fx1 && fy0 <= fy1) {
            x0 = (int)fx0; y0 = (int)fy0;
            w = (int)(fx1 - fx0) + 1; h = (int)(fy1 - fy0) + 1;
        }
    }
    boxes[i] = BoxWords{x0, y0, w, h};
}

// Exclusive scan of the N areas into offsets[0 .. N], and the largest box, by one workgroup of 1024
// lanes, each taking 8 consecutive values per pass: a pass costs two barriers and a memory
// latency whatever its width (one value per lane: 14 us for 8,192 primitives, 11 now; 125 us for
// 65,536), and the largest box took atomics after a launch that cleared them.
constexpr int OFF_PER = 8;

__global__ void __launch_bounds__(1024)
k_export_offsets(const BoxWords *__restrict__ boxes, long long *__restrict__ off, int N,
                 int *__restrict__ max_wh)
{
    __shared__ long long wsum[16];
    __shared__ int s_w[16], s_h[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    long long carry = 0;
    int w = 0, h = 0;
    for (int b0 = 0; b0 < N; b0 += 1024 * OFF_PER) {
        const int i0 = b0 + threadIdx.x * OFF_PER;
        long long v[OFF_PER], run = 0;
#pragma unroll
        for (int k = 0; k < OFF_PER; ++k) {
            const int i = i0 + k;
            const int4 bx = i < N ? box_at(boxes, i) : make_int4(0, 0, 0, 0);
            w = max(w, bx.z);
            h = max(h, bx.w);
            v[k] = run;
            run += (long long)bx.z * bx.w;
        }
        long long incl = run;
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        __syncthreads();  // the previous pass has read wsum
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        long long pre = carry + incl - run;
        for (int q = 0; q < 16; ++q) {
            if (q < wave) pre += wsum[q];
            carry += wsum[q];
        }
#pragma unroll
        for (int k = 0; k < OFF_PER; ++k)
            if (i0 + k < N) off[i0 + k] = pre + v[k];
    }
    for (int o = 32; o > 0; o >>= 1) {
        w = max(w, __shfl_xor(w, o));
        h = max(h, __shfl_xor(h, o));
    }
    if (lane == 0) {
        s_w[wave] = w;
        s_h[wave] = h;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < 16; ++q) {
            w = max(w, s_w[q]);
            h = max(h, s_h[q]);
        }
        off[N] = carry;
        max_wh[0] = w;
        max_wh[1] = h;
    }
}

template <typename TexT>
__device__ __forceinline__ float tex_at(const TexT *__restrict__ bm, int Hb, int Wb, int r, int c)
{
    return (r >= 0 && r < Hb && c >= 0 && c < Wb) ? texel<TexT>(bm[(size_t)r * Wb + c]) : 0.f;
}

// The map of a primitive and its opacity scale, folded as the binning folds them (float64):
// U = aU x + bU y + eU with U = cu (u + 1), u = (cos dx + sin dy) / s (unpadded bitmap coordinates).
struct LayerMap {
    double aU, bU, eU, aV, bV, eV;
    float ka;
};

__device__ __forceinline__ LayerMap layer_map(const float *p, int Hb, int Wb, float alpha_max)
{
    LayerMap m;
    const double s = exp((double)p[2]);
    double st, ct;
    sincos((double)p[3], &st, &ct);
    const double cu = 0.5 * (Wb - 1), cv = 0.5 * (Hb - 1), inv_s = 1.0 / s;
    m.aU = cu * ct * inv_s;
    m.bU = cu * st * inv_s;
    m.aV = -cv * st * inv_s;
    m.bV = cv * ct * inv_s;
    const double px = p[0], py = p[1];
    m.eU = cu - m.aU * px - m.bU * py;
    m.eV = cv - m.aV * px - m.bV * py;
    m.ka = (float)((double)alpha_max / (1.0 + exp(-(double)p[4])));
    return m;
}

// The alpha of a point between four texels, at fractions wu, wv along the bitmap's axes.
__device__ __forceinline__ float layer_value(const LayerMap &m, float wu, float wv, float p00,
                                             float p01, float p10, float p11)
{
    const float top = fmaf(wu, p01 - p00, p00), bot = fmaf(wu, p11 - p10, p10);
    return m.ka * fmaf(wv, bot - top, top);
}

// The integer nearest zero, saturated to the range of int (a cast leaves that undefined).
__device__ __forceinline__ int sat_int(double x)
{
    int i;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(i) : "v"(x));
    return i;
}

constexpr int WAVE_VALUES = 256;  // boxes of up to this many values are taken by one wave
constexpr int EXPORT_CHUNK = 16;  // most primitives of a workgroup

// Values of one box by the nt threads t = 0 .. nt - 1, in row-major order, texels from memory.
template <typename TexT>
__device__ __forceinline__ void layer_from_memory(const LayerMap &m, const TexT *__restrict__ bm,
                                                  int Hb, int Wb, const int4 &box, double ir,
                                                  float *__restrict__ out, int t, int nt)
{
    const int bw = box.z, n = bw * box.w;
    const double x0 = box.x + 0.5, y0 = box.y + 0.5;
    const int step_y = nt / bw, step_x = nt - step_y * bw;
    int by = t / bw, bx = t - by * bw;
    for (int j = t; j < n; j += nt) {
        // canvas point of export pixel (X, Y): (X + 0.5) / rho - 0.5
        const double x = fma(x0 + bx, ir, -0.5), y = fma(y0 + by, ir, -0.5);
        const double U = fma(m.aU, x, fma(m.bU, y, m.eU)), V = fma(m.aV, x, fma(m.bV, y, m.eV));
        const double u0 = floor(U), v0 = floor(V);
        float a = 0.f;
        if (u0 >= -1.0 && u0 <= Wb - 1.0 && v0 >= -1.0 && v0 <= Hb - 1.0) {
            const int iu = (int)u0, iv = (int)v0;
            a = layer_value(m, (float)(U - u0), (float)(V - v0), tex_at(bm, Hb, Wb, iv, iu),
                            tex_at(bm, Hb, Wb, iv, iu + 1), tex_at(bm, Hb, Wb, iv + 1, iu),
                            tex_at(bm, Hb, Wb, iv + 1, iu + 1));
        }
        out[j] = a;
        bx += step_x;
        by += step_y;
        if (bx >= bw) {
            bx -= bw;
            ++by;
        }
    }
}

// The same from the copy in LDS. A position outside the bitmap is moved to a cell of zeros, and the
// pixel's place in the box is mapped straight to the bitmap, so the loop has no comparisons.
template <typename TexT>
__device__ __forceinline__ void layer_from_copy(const LayerMap &m, const TexT *s_tex, int pitch,
                                                int Hb, int Wb, const int4 &box, double ir,
                                                float *__restrict__ out, int t, int nt)
{
    const double AU = m.aU * ir, BU = m.bU * ir, AV = m.aV * ir, BV = m.bV * ir;
    const double ex = fma(box.x + 0.5, ir, -0.5), ey = fma(box.y + 0.5, ir, -0.5);
    const double EU = fma(m.aU, ex, fma(m.bU, ey, m.eU)), EV = fma(m.aV, ex, fma(m.bV, ey, m.eV));
    const int bw = box.z, n = bw * box.w;
    const int step_y = nt / bw, step_x = nt - step_y * bw;
    int by = t / bw, bx = t - by * bw;
    for (int j = t; j < n; j += nt) {
        const double U = fma(AU, (double)bx, fma(BU, (double)by, EU));
        const double V = fma(AV, (double)bx, fma(BV, (double)by, EV));
        const double u0 = floor(U), v0 = floor(V);
        // outside the bitmap and its border (as unsigned: past the end) lies a cell of zeros
        const unsigned iu = min((unsigned)sat_int(u0) + 1u, (unsigned)Wb + 1u);
        const unsigned iv = min((unsigned)sat_int(v0) + 1u, (unsigned)Hb + 1u);
        const TexT *q = s_tex + __umul24(iv, pitch) + iu;
        out[j] = layer_value(m, (float)(U - u0), (float)(V - v0), texel<TexT>(q[0]),
                             texel<TexT>(q[1]), texel<TexT>(q[pitch]), texel<TexT>(q[pitch + 1]));
        bx += step_x;
        by += step_y;
        if (bx >= bw) {
            bx -= bw;
            ++by;
        }
    }
}

__device__ __forceinline__ bool map_finite(const LayerMap &m)
{
    return isfinite(m.aU) && isfinite(m.bU) && isfinite(m.eU) && isfinite(m.aV) &&
           isfinite(m.bV) && isfinite(m.eV) && isfinite(m.ka);
}

// The copy's border: rows -1, Hb, Hb + 1 and columns -1, Wb, Wb + 1 of zeros (one wave).
template <typename TexT>
__device__ __forceinline__ void copy_border(TexT *s_tex, int pitch, int Hb, int Wb, int lane)
{
    for (int x = lane; x < Wb + 3; x += 64)
        s_tex[x] = s_tex[(Hb + 1) * pitch + x] = s_tex[(Hb + 2) * pitch + x] = TexT(0);
    for (int y = lane; y < Hb; y += 64) {
        TexT *t = s_tex + (y + 1) * pitch;
        t[0] = t[Wb + 1] = t[Wb + 2] = TexT(0);
    }
}

// Rows w, w + nw, .. of the bitmap into the copy (wave w of nw).
template <typename TexT>
__device__ __forceinline__ void copy_rows(TexT *s_tex, int pitch, const TexT *__restrict__ bm,
                                          int Hb, int Wb, int lane, int w, int nw)
{
#pragma unroll 4
    for (int y = w; y < Hb; y += nw)
        for (int x = lane; x < Wb; x += 64)
            s_tex[(y + 1) * pitch + x + 1] = bm[(size_t)y * Wb + x];
}

struct LayerArgs {
    int N, chunk;
    int copy_min;  // boxes of at least this many values take the copy in LDS
    int B, Hb, Wb, pitch;
    float alpha_max;
    double ir;  // 1 / rho
};

// One workgroup per primitive: the primitive's constants once (by one wave, while the others copy
// the bitmap), then its box's pixels in row-major order, NT at a time (coalesced stores into its
// packed box; the row and column advance by a fixed step, no division).
// LDS: the bitmap is first copied to LDS inside a border of zeros, if the box has at least half as
// many values as the bitmap texels: 64 neighbouring pixels read texels of some 40 cache lines, and
// the L1 serves one line per clock, so four loads per value from memory cost about 160 clocks per
// 64 values. Bound by instructions (82 % of the issue slots, 42 per value of which 14 in float64).
// 54 million values at 1024 x 1024 x 2, 8,192 primitives, 64 x 64 float32 bitmaps: 276 us from
// memory, 145 with comparisons in the loop over the copy (four values at a time or 512 threads
// were no faster), 113 now; 217 MB are written, 43 us. Smaller boxes read from memory.
// (A grid of (primitive, tile row, tile column) sized by the largest box launched mostly empty
// workgroups: 5.1 ms at 2048 x 2048 with 65,536 primitives against 0.59 ms; one wave per primitive
// took 1.17 ms: the largest boxes then run on 64 lanes.)
template <typename TexT, bool LDS, int NT>
__global__ void __launch_bounds__(NT)
k_export_layers(LayerArgs a, const TexT *__restrict__ atlas, const float *__restrict__ params,
                const int *__restrict__ idx, const BoxWords *__restrict__ boxes,
                const long long *__restrict__ offsets, float *__restrict__ alpha_out,
                float *__restrict__ colour_out)
{
    extern __shared__ __attribute__((aligned(16))) char s_raw[];
    __shared__ LayerMap s_map;
    __shared__ int s_fin;  // the map's constants are finite
    TexT *s_tex = reinterpret_cast<TexT *>(s_raw);
    const int i = blockIdx.x;
    const int4 box = box_at(boxes, i);
    const int n = box.z * box.w;
    const float *p = params + (size_t)i * 8;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < 3)
        colour_out[3 * i + threadIdx.x] =
            (float)(1.0 / (1.0 + exp(-(double)p[5 + threadIdx.x])));
    if (n == 0) return;
    float *out = alpha_out + offsets[i];
    const int k = idx[i];
    if (!(k >= 0 && k < a.B)) {
        for (int j = threadIdx.x; j < n; j += NT) out[j] = 0.f;
        return;
    }
    const TexT *bm = atlas + (size_t)k * a.Hb * a.Wb;
    const bool staged = LDS && n >= a.copy_min;
    if (wave == 0) {
        if (LDS && staged) copy_border(s_tex, a.pitch, a.Hb, a.Wb, lane);
        const LayerMap m = layer_map(p, a.Hb, a.Wb, a.alpha_max);
        if (lane == 0) {
            s_map = m;
            s_fin = map_finite(m);
        }
    } else if (LDS && staged) {
        copy_rows(s_tex, a.pitch, bm, a.Hb, a.Wb, lane, wave - 1, NT / 64 - 1);
    }
    __syncthreads();
    const LayerMap m = s_map;
    if (LDS && staged && s_fin)
        layer_from_copy(m, s_tex, a.pitch, a.Hb, a.Wb, box, a.ir, out, (int)threadIdx.x, NT);
    else
        layer_from_memory(m, bm, a.Hb, a.Wb, box, a.ir, out, (int)threadIdx.x, NT);
}

// Many primitives: a workgroup takes `chunk` of them, their constants in one go (a lane each, while the
// other waves copy the first bitmap), then the boxes of more than 256 values one after the other, by
// all waves, and the smaller ones a wave each. Small boxes are bound by the latency of their
// constants, and all workgroups of a launch hold the LDS that a few larger boxes need: 65,536 boxes
// of 67 values beside 16 of 9,400 (128 x 128 bfloat16 bitmaps) took 174 us with one primitive per
// workgroup of 256 (77 without LDS), 63 here; 65,536 of 470 values beside 64, 262 (204), 202.
template <typename TexT, bool LDS, int NT>
__global__ void __launch_bounds__(NT, 8)
k_export_chunks(LayerArgs a, const TexT *__restrict__ atlas, const float *__restrict__ params,
                const int *__restrict__ idx, const BoxWords *__restrict__ boxes,
                const long long *__restrict__ offsets, float *__restrict__ alpha_out,
                float *__restrict__ colour_out)
{
    extern __shared__ __attribute__((aligned(16))) char s_raw[];
    __shared__ LayerMap s_map[EXPORT_CHUNK];
    __shared__ int4 s_box[EXPORT_CHUNK];
    __shared__ long long s_off[EXPORT_CHUNK];
    __shared__ int s_k[EXPORT_CHUNK], s_fin[EXPORT_CHUNK];
    TexT *s_tex = reinterpret_cast<TexT *>(s_raw);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // strided: neighbours are often alike, and a workgroup with several large boxes ends late. Lane l
    // of every wave looks at the l-th.
    auto prim = [&](int l) { return blockIdx.x + (long long)l * gridDim.x; };
    const bool mine = lane < a.chunk && prim(lane) < a.N;
    uint64_t large, small;
    {
        float p[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        int4 box = make_int4(0, 0, 0, 0);
        int k = -1;
        if (mine) {
            if (wave == 0) {  // requested with the box: the constants are what the others wait for
#pragma unroll
                for (int q = 0; q < 5; ++q) p[q] = params[8 * prim(lane) + q];
                s_off[lane] = offsets[prim(lane)];
            }
            box = box_at(boxes, prim(lane));
            k = idx[prim(lane)];
        }
        const int n = box.z * box.w;
        large = __ballot(n > WAVE_VALUES);
        small = __ballot(n != 0 && n <= WAVE_VALUES);
        if (wave == 0) {
            if (LDS) copy_border(s_tex, a.pitch, a.Hb, a.Wb, lane);
            if (lane < a.chunk) {
                s_box[lane] = box;
                s_k[lane] = k;
                const LayerMap m = layer_map(p, a.Hb, a.Wb, a.alpha_max);
                s_map[lane] = m;
                s_fin[lane] = map_finite(m);
            }
        } else if (LDS && large) {
            const int l = (int)__builtin_ctzll(large), kl = __builtin_amdgcn_readlane(k, l);
            if (__builtin_amdgcn_readlane(n, l) >= a.copy_min && kl >= 0 && kl < a.B)
                copy_rows(s_tex, a.pitch, atlas + (size_t)kl * a.Hb * a.Wb, a.Hb, a.Wb, lane,
                          wave - 1, NT / 64 - 1);
        }
        if (wave == NT / 64 - 1 && lane < 3 * a.chunk && prim(lane / 3) < a.N) {
            const long long i = prim(lane / 3);
            const int q = lane % 3;
            colour_out[3 * i + q] = (float)(1.0 / (1.0 + exp(-(double)params[8 * i + 5 + q])));
        }
    }
    __syncthreads();
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    bool first = true;
    for (; large; large &= large - 1, first = false) {
        const int l = (int)__builtin_ctzll(large), k = uniform(s_k[l]);
        const int4 box = s_box[l];
        const int n = uniform(box.z * box.w);
        float *out = alpha_out + s_off[l];
        const TexT *bm = atlas + (size_t)k * a.Hb * a.Wb;
        if (!(k >= 0 && k < a.B)) {
            for (int j = threadIdx.x; j < n; j += NT) out[j] = 0.f;
        } else if (LDS && n >= a.copy_min && uniform(s_fin[l])) {
            if (!first) {
                __syncthreads();  // the previous copy is read
                copy_rows(s_tex, a.pitch, bm, a.Hb, a.Wb, lane, wave, NT / 64);
                __syncthreads();
            }
            layer_from_copy(s_map[l], s_tex, a.pitch, a.Hb, a.Wb, box, a.ir, out, (int)threadIdx.x, NT);
        } else {
            layer_from_memory(s_map[l], bm, a.Hb, a.Wb, box, a.ir, out, (int)threadIdx.x, NT);
        }
    }
    for (int c = 0; small; small &= small - 1, ++c) {
        if (c % (NT / 64) != wave) continue;
        const int l = (int)__builtin_ctzll(small), k = uniform(s_k[l]);
        const int4 box = s_box[l];
        float *out = alpha_out + s_off[l];
        if (k >= 0 && k < a.B) {
            layer_from_memory(s_map[l], atlas + (size_t)k * a.Hb * a.Wb, a.Hb, a.Wb, box, a.ir, out,
                              lane, 64);
        } else {
            for (int j = lane; j < box.z * box.w; j += 64) out[j] = 0.f;
        }
    }
}

int launched() { return hipGetLastError() == hipSuccess ? DBMP_OK : DBMP_EHIP; }

bool export_canvas(int H, int W, double rho, int *HH, int *WW)
{
    if (H < 1 || W < 1 || !(rho > 0.0 && rho <= 64.0)) return false;
    const double hh = nearbyint(H * rho), ww = nearbyint(W * rho);
    if (hh < 1 || ww < 1 || hh * ww >= (double)INT_MAX) return false;
    *HH = (int)hh;
    *WW = (int)ww;
    return true;
}

}  // namespace
}  // namespace dbmp

using namespace dbmp;

extern "C" {

int dbmp_export_boxes(dbmp_export_stream stream, const float *params, int N, int Hb, int Wb,
                      int H, int W, double rho, int32_t *boxes, long long *offsets,
                      int32_t *max_wh)
{
    int HH = 0, WW = 0;
    if (N < 0 || Hb < 2 || Wb < 2 || !export_canvas(H, W, rho, &HH, &WW)) return DBMP_EINVAL;
    if (!offsets || !max_wh || (N > 0 && (!params || !boxes))) return DBMP_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    if (N > 0)
        k_export_boxes<<<(N + 255) / 256, 256, 0, st>>>(params, N, Hb, Wb, HH, WW, rho,
                                                       (BoxWords *)boxes);
    k_export_offsets<<<1, 1024, 0, st>>>((const BoxWords *)boxes, offsets, N, max_wh);
    return launched();
}

int dbmp_export_layers(dbmp_export_stream stream, const float *params, const int32_t *atlas_idx,
                       int N, const void *atlas, int B, int Hb, int Wb, int atlas_dtype, int H,
                       int W, double rho, float alpha_max, const int32_t *boxes,
                       const long long *offsets, int max_w, int max_h, float *alpha_out,
                       float *colour_out)
{
    int HH = 0, WW = 0;
    if (N < 0 || B < 1 || Hb < 2 || Wb < 2 || !export_canvas(H, W, rho, &HH, &WW))
        return DBMP_EINVAL;
    if (atlas_dtype != DBMP_F32 && atlas_dtype != DBMP_BF16 && atlas_dtype != DBMP_F16)
        return DBMP_EINVAL;
    if (!(alpha_max > 0.f && alpha_max <= 1.f)) return DBMP_EINVAL;
    if (max_w < 0 || max_h < 0 || max_w > WW || max_h > HH) return DBMP_EINVAL;
    if (N == 0) return DBMP_OK;
    if (!params || !atlas_idx || !atlas || !boxes || !offsets || !colour_out) return DBMP_EINVAL;
    if (max_w > 0 && !alpha_out) return DBMP_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    // bitmaps in LDS up to 42 KB with their border (three or more workgroups per compute unit), if
    // the largest box may repay the copy; an odd pitch in 4-byte words spreads a column over the banks
    const int esz = atlas_dtype == DBMP_F32 ? 4 : 2;
    const int pitch = (((Wb + 3) * esz + 3) / 4 | 1) * (4 / esz);
    const long long lds = (long long)(Hb + 3) * pitch * esz, most = (long long)max_w * max_h;
    const long long half = ((long long)Hb * Wb + 1) / 2;
    const bool stage = lds <= 42 * 1024 && most >= half && most > WAVE_VALUES;
    const int copy_min = stage ? (int)std::max<long long>(half, WAVE_VALUES + 1) : INT_MAX;
    // Primitives of a workgroup. Boxes of a wave each want 2,048 workgroups, which are resident at
    // once; where some are larger, as many as balance the load: with 65,536 primitives, 6 each of 512
    // threads (63 us with 16 larger boxes, 4 took 77 and 8 took 56; 202 with boxes of 470 values, 198
    // and 207) and 2 each where nothing is copied (60 us for small boxes and 212 for boxes of 470
    // values; one took 79 and 197, four 223 for the latter).
    const int wgs = most <= WAVE_VALUES ? 2048 : !stage ? 32768 : lds > 20 * 1024 ? 12288 : 16384;
    const int chunk = std::min(EXPORT_CHUNK, N / wgs + (N % wgs != 0));
    const LayerArgs a{N, chunk, copy_min, B, Hb, Wb, pitch, alpha_max, 1.0 / rho};
    auto run = [&](auto texel_of, auto one, auto many, int threads) {
        using TexT = decltype(texel_of);
        const unsigned grid = (unsigned)(N / chunk + (N % chunk != 0));
        auto go = [&](auto kern) {
            kern<<<grid, threads, stage ? (size_t)lds : 0, st>>>(
                a, (const TexT *)atlas, params, atlas_idx, (const BoxWords *)boxes, offsets, alpha_out,
                colour_out);
        };
        if (chunk == 1) go(one);
        else go(many);
    };
    // above 20 KB of LDS fewer than eight workgroups fit a compute unit: 512 threads each (65,536
    // primitives, 43,000 of them copied, 100 x 100 float32 bitmaps: 770 us, 1,147 with 256)
    auto run_t = [&](auto t) {
        using T = decltype(t);
        if (stage && lds > 20 * 1024)
            run(t, k_export_layers<T, true, 512>, k_export_chunks<T, true, 512>, 512);
        else if (stage)
            run(t, k_export_layers<T, true, 256>, k_export_chunks<T, true, 256>, 256);
        else
            run(t, k_export_layers<T, false, 256>, k_export_chunks<T, false, 256>, 256);
    };
    if (atlas_dtype == DBMP_F32) run_t(float{});
    else if (atlas_dtype == DBMP_F16) run_t(_Float16{});
    else run_t(uint16_t{});
    return launched();
}

}  // extern "C"
