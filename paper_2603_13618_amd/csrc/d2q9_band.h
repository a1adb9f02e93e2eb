// d2q9_band.h -- geometry shared by the D2Q9 kernels that advance 64-column
// bands several steps per launch (forward and adjoint): which tile a workgroup
// owns, periodic wrapping, and the ring cells around a tile.
#pragma once

#include "lks_device.h"

namespace lks {

// Whether the tiles of T cells with a ring of K along an axis of n cells reach
// at most one period beyond it on either side (what the kernels wrap).
constexpr bool tile_fits(int n, int T, int K) { return n >= K && (n - 1LL) / T * T + T + K <= 2LL * n; }

// K steps of a tile of 64 columns: eight waves (two a SIMD: six and twelve
// measured 30 % slower) of NR rows each, one lane a column.  Cells of the tile
// and a ring of H0 = K - 1 cells lie in LDS at (y + H0) W0 + x + H0, x and y
// relative to the tile.
constexpr int kBandWaves = 8;
constexpr int kBandX = kWave, kBandK = 3;
constexpr int band_y(int nr) { return nr * kBandWaves; }
constexpr bool band_fits(int nx, int ny, int nr) { return tile_fits(nx, kBandX, kBandK) && tile_fits(ny, band_y(nr), kBandK); }
constexpr int band_tiles(int nx, int ny, int nr)
{
    return ((nx + kBandX - 1) / kBandX) * ((ny + band_y(nr) - 1) / band_y(nr));
}

template <int K, int NR_> struct Band {
    static_assert(K >= 1 && K <= kBandK, "one to three steps");
    static constexpr int NW = kBandWaves, NR = NR_, TX = kBandX, TY = band_y(NR), H0 = K - 1, W0 = TX + 2 * H0;
    static constexpr int kCells = K == 1 ? 1 : W0 * (TY + 2 * H0);
    // cells of the ring of H cells: one a thread at most
    template <int H> static constexpr int ring() { return (TX + 2 * H) * (TY + 2 * H) - TX * TY; }
    static_assert(ring<H0>() <= NW * kWave, "one ring cell a thread");

    // The XCD that runs a workgroup is its id mod 8: each takes runs of eight
    // tiles along x (the grid is rounded up to 64 workgroups).
    __device__ __forceinline__ static int tile()
    {
        return blockIdx.x / 64 * 64 + blockIdx.x % 8 * 8 + blockIdx.x / 8 % 8;
    }
    // one period off at most (tile_fits)
    __device__ __forceinline__ static int wrap(int j, int n)
    {
        j += j < 0 ? n : 0;
        return j - (j >= n ? n : 0);
    }
    __device__ __forceinline__ static int cell(int x, int y) { return (y + H0) * W0 + x + H0; }
    // ring cell e of the ring of H cells: top and bottom rows, then the sides
    template <int H> __device__ __forceinline__ static void ring_cell(int e, int& x, int& y)
    {
        constexpr int W = TX + 2 * H;
        if (e < 2 * H * W) {
            const int r = e / W;
            x = e - r * W - H;
            y = r < H ? r - H : TY + r - H;
        } else {
            const int s = e - 2 * H * W, c = s % (2 * H);
            x = c < H ? c - H : TX + c - H;
            y = s / (2 * H);
        }
    }
};

} // namespace lks
