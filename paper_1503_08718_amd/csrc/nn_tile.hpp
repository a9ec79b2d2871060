// Spatial tiles of the 3x3x3 convolutions: a block stages the activations of
// an 8 x TY x TZ tile of voxels and its halo in LDS once, and every tap reads
// them from there.
#pragma once

#include "nn_device.hpp"

namespace mrt {

constexpr int TILE_X = 8;

// PITCH_: positions between neighbouring lines in LDS (at least 10).  A 16-byte
// read of the matrix operand is free of bank conflicts when its 16 voxels lie
// at 16 different positions modulo 16; a group is two lines of 8, so lines that
// are 8 modulo 16 apart: y and y + 4 at pitch 10.
template <int TY, int TZ, int PITCH_ = TILE_X + 2>
struct Tile {
    static constexpr int HX = TILE_X + 2, HY = TY + 2, HZ = TZ + 2, PITCH = PITCH_;
    static constexpr int LINES = HY * HZ;          // lines staged
    static constexpr int SPAN = PITCH * HY * HZ;   // positions in LDS
    static constexpr int PAIR = TY == 8 ? 4 : 1;   // lines of a group: y, y + PAIR

    // offset of a tap in positions
    static __host__ __device__ constexpr int tap(int t) { return ((t / 9) * HY + (t / 3) % 3) * PITCH + t % 3; }
    // line (y + TY z) of half 0 or 1 of voxel group i
    static __host__ __device__ constexpr int line(int i, int half) {
        return i / PAIR * 2 * PAIR + i % PAIR + half * PAIR;
    }

    // tile t of the launch: sample and first voxel
    int nb, x0, y0, z0;

    __device__ __forceinline__ Tile(const ConvGeom &g, unsigned t) {
        const unsigned ntx = (g.W + TILE_X - 1) / TILE_X, nty = (g.H + TY - 1) / TY, ntz = (g.D + TZ - 1) / TZ;
        x0 = (int)(t % ntx) * TILE_X;
        t /= ntx;
        y0 = (int)(t % nty) * TY;
        t /= nty;
        z0 = (int)(t % ntz) * TZ;
        nb = (int)(t / ntz);
    }

    // first voxel of the input row under halo line l (y + HY z), -1 in zero
    // padding; lines further outside (partial tiles) are not used and give any row
    __device__ __forceinline__ int row(const ConvGeom &g, int l) const {
        int y = y0 + l % HY - 1, z = z0 + l / HY - 1;
        const bool oy = y < 0 || y >= g.H, oz = z < 0 || z >= g.D;
        y = y < 0 ? g.H - 1 : (y >= g.H ? 0 : y);
        z = z < 0 ? g.D - 1 : (z >= g.D ? 0 : z);
        return (!oy || (g.circ & 2)) && (!oz || (g.circ & 4)) ? ((nb * g.D + z) * g.H + y) * g.W : -1;
    }
    // the same for position hx of a line: x, -1 in zero padding
    __device__ __forceinline__ int column(const ConvGeom &g, int hx) const {
        const int x = x0 + hx - 1;
        if (x >= 0 && x < g.W) return x;
        return g.circ & 1 ? (x < 0 ? g.W - 1 : 0) : -1;
    }

    // Staging by lines: GROUPS threads for each of a line's positions and as
    // many lines at a time as 256 threads hold, so that a thread's channels and
    // column stay and only its line changes.
    // The row of a line is worked out by one lane of each wave
    // and taken from there: worked out for every position it took more
    // instructions than the products (128 -> 128 channels: 840 vector instructions
    // a wave, 419 like this, 19.2 -> 17.2 us on 8^3; 64 -> 32 on 32^3 18.8 -> 16.8).
    template <int GROUPS>
    struct Stage {
        static_assert(LINES <= 64, "one lane for each line");
        static constexpr int WIDTH = HX * GROUPS, AT_ONCE = 256 / WIDTH, PASSES = (LINES + AT_ONCE - 1) / AT_ONCE;
        int l0, hx, cg;  // first line, position and channel group of this thread
        bool takes;

        __device__ __forceinline__ Stage() {
            l0 = threadIdx.x / WIDTH;
            const int e = threadIdx.x - l0 * WIDTH;
            hx = e / GROUPS;
            cg = e % GROUPS;
            takes = l0 < AT_ONCE;
        }
        __device__ __forceinline__ int line(int pass) const { return l0 + pass * AT_ONCE; }
        __device__ __forceinline__ bool stores(int pass) const { return takes && line(pass) < LINES; }
    };

    // voxel v (0 .. 8 TY TZ - 1) of the tile, -1 outside the volume
    __device__ __forceinline__ int inside(const ConvGeom &g, int v) const {
        const int x = x0 + v % TILE_X, y = y0 + v / TILE_X % TY, z = z0 + v / (TILE_X * TY);
        return x < g.W && y < g.H && z < g.D ? ((nb * g.D + z) * g.H + y) * g.W + x : -1;
    }
    __device__ __forceinline__ bool partial(const ConvGeom &g) const {
        return x0 + TILE_X > g.W || y0 + TY > g.H || z0 + TZ > g.D;
    }
};

inline long long tile_count(const ConvGeom &g, int ty, int tz) {
    return (long long)g.n * ((g.D + tz - 1) / tz) * ((g.H + ty - 1) / ty) * ((g.W + TILE_X - 1) / TILE_X);
}

}  // namespace mrt
