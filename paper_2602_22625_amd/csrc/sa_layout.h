// Workspace of the structure-aware initialisation: host logic only, with no HIP types, so the same code
// is exercised by a CPU test.
//
// Its size is part of the interface: callers may bring a workspace sized by an earlier library, so it
// stays what an int64 per pixel and one pair of extremes per 16 x 16 block came to, and what the
// kernels use now is laid out within that.
#pragma once

#include <stddef.h>

namespace dbmp {

constexpr int LV_W = 64;         // columns per workgroup of the local variance
constexpr int NLV_BLOCK = 4096;  // pixels per workgroup of the sampling weights
constexpr int NLV_GROUP = 64;    // pixels whose sampling weights are summed to one entry

struct SaLayout {
    size_t minmax, bmm, lv, gsum, bsum, used, total;  // byte offsets; bytes used; bytes to bring
};

// Rows per workgroup of the local variance: 32, or 8 (more rows of halo per output) where 32 would
// leave the chip without two workgroups per compute unit.
inline int lv_rows(int H, int W)
{
    const long long wgs = (long long)((W + LV_W - 1) / LV_W) * ((H + 31) / 32);
    return wgs >= 512 ? 32 : 8;
}

// A single column lies in memory as a single row does, whose windows are the same: the local variance
// takes it as one, 64 pixels per wave (65,536 x 1: 57 us for the start of a fit as a column, 31 as a row).
inline void lv_shape(int &H, int &W)
{
    if (W == 1) {
        W = H;
        H = 1;
    }
}

inline SaLayout sa_layout(int H, int W)
{
    lv_shape(H, W);
    const size_t npix = (size_t)H * W, nb = (npix + NLV_BLOCK - 1) / NLV_BLOCK;
    const size_t rows = (size_t)lv_rows(H, W);
    const size_t nblk = (((size_t)W + LV_W - 1) / LV_W) * (((size_t)H + rows - 1) / rows);
    const size_t blocks16 = (((size_t)W + 15) / 16) * (((size_t)H + 15) / 16);  // (symmetric)
    auto up = [](size_t x, size_t a) { return (x + a - 1) / a * a; };
    const size_t total = 256 + up(16 * blocks16, 256) + 2 * up(8 * npix, 256) +
                         up(8 * ((npix + 2047) / 2048), 256);
    auto lay = [&](size_t a) {
        SaLayout L;
        L.minmax = 0;
        L.bmm = up(16, a);
        L.lv = L.bmm + up(16 * nblk, a);
        L.gsum = L.lv + up(8 * npix, a);
        L.bsum = L.gsum + up(8 * (NLV_BLOCK / NLV_GROUP) * nb, a);
        L.used = L.bsum + 8 * nb;
        L.total = total;
        return L;
    };
    const SaLayout L = lay(256);
    return L.used <= total ? L : lay(16);  // a few pixels, or a few columns of many rows
}

}  // namespace dbmp
