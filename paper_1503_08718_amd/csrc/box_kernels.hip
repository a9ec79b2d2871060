// Several time steps per launch for small cells.
//
// A cell of a few ten thousand nodes steps in the time of a launch (16^3 FP64:
// 2.7 us, of which the arithmetic is a tenth).  Here a block takes a tile of
// ty x tz rows (whole rows in x) and carries it through S steps: the first
// pulls from memory the tile widened by S - 1 rows on each side, the state in
// between stays in LDS as moments, each further step needs one row less on each
// side, and the last writes the tile.  Blocks exchange nothing; the halo rows
// are computed by every block that needs them, which is cheap where the launch
// is what a step waits for.
//
// One node per thread, the arithmetic of the single-step kernels operation by
// operation, so the results agree bit for bit: FP32 and FP64 moment storage,
// and FP64 population storage, whose populations are T/8 +- jhat/2 rounded from
// the moments (FP32 populations are dithered one by one and stay single-step).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "box_internal.h"
#include "lbm_device.hpp"

#pragma clang fp contract(off)

namespace mrt {

constexpr int BOX_LDS = 160 * 1024;
constexpr int BOX_CUS = 256;

// (T, jhat/2) of one node from what it pulled: T/4 of its own, the six
// populations (FP64: as they are stored or rebuilt, FP32: exact)
template <typename real>
__device__ __forceinline__ void box_collide(const Cell<real> &c, const real *tb, double f0, const double *p,
                                            unsigned long long node, real *o) {
    real jx, jy, jz;
    if constexpr (sizeof(real) == 4) {
        const double T64 = f0 + p[0] + p[1] + p[2] + p[3] + p[4] + p[5];
        jx = (float)(p[0] - p[1]) + 2.0f * c.h[0];
        jy = (float)(p[2] - p[3]) + 2.0f * c.h[1];
        jz = (float)(p[4] - p[5]) + 2.0f * c.h[2];
        o[0] = dither_to_float(T64, node);
    } else {
        const double f1 = p[0] + c.h[0], f2 = p[1] - c.h[0], f3 = p[2] + c.h[1], f4 = p[3] - c.h[1];
        const double f5 = p[4] + c.h[2], f6 = p[5] - c.h[2];
        o[0] = f0 + f1 + f2 + f3 + f4 + f5 + f6;
        jx = f1 - f2;
        jy = f3 - f4;
        jz = f5 - f6;
    }
    o[1] = fma(tb[4], jz, fma(tb[3], jy, tb[0] * jx));
    o[2] = fma(tb[5], jz, fma(tb[1], jy, tb[3] * jx));
    o[3] = fma(tb[2], jz, fma(tb[5], jy, tb[4] * jx));
}

// The population a node pulls along one axis from (T, jhat_a/2): side 0 from
// the lower neighbour (T/8 + jhat_a/2), side 1 from the upper one.  At a wall
// the node's own opposite population, reflected.
__device__ __forceinline__ double box_pop(double T, double z, int side) { return fma(T, 0.125, side ? -z : z); }

// nodes of a thread; their places and phase tables stay in registers
constexpr int BOX_NODES = 4, BOX_THREADS = 512;

// a / b for 0 <= a < 2^20, inv = 1.0f / b: the product's error is below 1/2b
__device__ __forceinline__ int box_div(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

template <typename real, int ST>
__global__ void __launch_bounds__(BOX_THREADS) k_box(Cell<real> c, int S, int ty, int tz, int nty) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nx = c.nx, ny = c.ny, nz = c.nz, w = S - 1;
    const int by = ty + 2 * w, bz = tz + 2 * w, nodes = by * bz * nx;
    real *tab = reinterpret_cast<real *>(smem_raw);  // [nphase][6]
    // two boxes of (T, jhat_x, jhat_y, jhat_z), [rz][ry][x]
    real *buf0 = tab + c.nphase * 6, *buf1 = buf0 + 4 * nodes;
    const int y0 = (int)(blockIdx.x % nty) * ty - w, z0 = (int)(blockIdx.x / nty) * tz - w;
    const long long N = c.N;
    const int plane = nx * ny;
    for (int i = threadIdx.x; i < c.nphase * 6; i += blockDim.x) tab[i] = c.tab[i / 6 * TABW + i % 6];
    struct Node {
        int l;              // place in the box
        int last;           // the last step that computes it (0: none)
        int at;             // node of the cell
        unsigned walls;     // bit 2 a + side: the neighbour is a wall
        int xl, xh;         // x neighbours in the box
        int ph;
    } nd[BOX_NODES];
    real own[BOX_NODES], in_a[BOX_NODES][6], in_b[BOX_NODES][6];
    const float inv_x = 1.0f / (float)nx, inv_y = 1.0f / (float)by;
#pragma unroll
    for (int k = 0; k < BOX_NODES; k++) {
        Node &n = nd[k];
        const int i = k * blockDim.x + threadIdx.x;
        n.l = i;
        n.last = 0;
        n.walls = 0;
        n.ph = 0;
        if (i >= nodes) continue;
        const int r = box_div(i, inv_x), x = i - r * nx, rz = box_div(r, inv_y), ry = r - rz * by;
        int y = y0 + ry, z = z0 + rz;
        // rows beyond a wall do not exist; in and behind the last tile the
        // rows past the cell's end are only halo
        int last = min(min(ry, by - 1 - ry), min(rz, bz - 1 - rz)) + 1;
        if (y >= ny || z >= nz) last = min(last, w);
        if ((y < 0 || y >= ny) && !c.per[1]) last = 0;
        if ((z < 0 || z >= nz) && !c.per[2]) last = 0;
        y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
        z = z < 0 ? z + nz : (z >= nz ? z - nz : z);
        if (y >= ny || z >= nz) last = 0;
        if (last == 0) continue;
        n.last = last;
        const int at = z * plane + y * nx + x;
        n.at = at;
        n.xl = x > 0 ? i - 1 : (c.per[0] ? i + nx - 1 : i);
        n.xh = x < nx - 1 ? i + 1 : (c.per[0] ? i - (nx - 1) : i);
        if (!c.per[0]) n.walls |= (x == 0 ? 1u : 0u) | (x == nx - 1 ? 2u : 0u);
        if (!c.per[1]) n.walls |= (y == 0 ? 4u : 0u) | (y == ny - 1 ? 8u : 0u);
        if (!c.per[2]) n.walls |= (z == 0 ? 16u : 0u) | (z == nz - 1 ? 32u : 0u);
        // everything the first step reads; a wall keeps the node itself
        n.ph = c.phase[at];
        own[k] = c.src[at];
        int nb[6] = {at + (n.xl - i), at + (n.xh - i), at - nx, at + nx, at - plane, at + plane};
        if (y == 0) nb[2] = c.per[1] ? at + plane - nx : at;
        if (y == ny - 1) nb[3] = c.per[1] ? at - (plane - nx) : at;
        if (z == 0) nb[4] = c.per[2] ? at + (int)N - plane : at;
        if (z == nz - 1) nb[5] = c.per[2] ? at - ((int)N - plane) : at;
#pragma unroll
        for (int d = 0; d < 6; d++) {
            const int side = (n.walls >> d & 1) ? !(d & 1) : (d & 1), a = d >> 1;
            if constexpr (ST == 1) {
                in_a[k][d] = c.src[nb[d]];
                in_b[k][d] = c.src[(a + 1) * N + nb[d]];
            } else {
                in_a[k][d] = c.src[(1 + 2 * a + side) * N + nb[d]];
            }
        }
    }
    auto put = [&](const Node &n, int s, const real *o, real *next) {
        if (s < S) {
#pragma unroll
            for (int q = 0; q < 4; q++) next[q * nodes + n.l] = o[q];
        } else if constexpr (ST == 1) {
#pragma unroll
            for (int q = 0; q < 4; q++) c.dst[q * N + n.at] = o[q];
        } else {
            c.dst[n.at] = o[0] * real(0.25);
#pragma unroll
            for (int a = 0; a < 3; a++) {
                c.dst[(2 * a + 1) * N + n.at] = out_pop(o[0], o[a + 1], (long long)n.at, a, 0);
                c.dst[(2 * a + 2) * N + n.at] = out_pop(o[0], o[a + 1], (long long)n.at, a, 1);
            }
        }
    };
    // reflected: sgn (T/8 -+ z) = (sgn T)/8 -+ sgn z, exactly
    auto reflect = [&](const Node &n, int d, real &T, real &z) {
        if (n.walls >> d & 1) {
            T *= c.sgn[d >> 1];
            z *= -c.sgn[d >> 1];
        }
    };
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BOX_NODES; k++) {
        const Node &n = nd[k];
        if (n.last == 0) continue;
        double p[6];
#pragma unroll
        for (int d = 0; d < 6; d++) {
            if constexpr (ST == 1) {
                reflect(n, d, in_a[k][d], in_b[k][d]);
                p[d] = box_pop(in_a[k][d], in_b[k][d], d & 1);
            } else {
                p[d] = (n.walls >> d & 1) ? c.sgn[d >> 1] * in_a[k][d] : in_a[k][d];
            }
        }
        real o[4];
        box_collide<real>(c, tab + n.ph * 6, ST == 1 ? (double)own[k] * 0.25 : (double)own[k], p,
                          (unsigned long long)n.at, o);
        put(n, 1, o, buf0);
    }
    // the others from LDS
    for (int s = 2; s <= S; s++) {
        __syncthreads();
        const real *in = s & 1 ? buf1 : buf0;
        real *next = s & 1 ? buf0 : buf1;
#pragma unroll
        for (int k = 0; k < BOX_NODES; k++) {
            const Node &n = nd[k];
            if (n.last < s) continue;
            const int l = n.l;
            int nb[6] = {n.xl, n.xh, l - nx, l + nx, l - by * nx, l + by * nx};
            if (n.walls & 4u) nb[2] = l;
            if (n.walls & 8u) nb[3] = l;
            if (n.walls & 16u) nb[4] = l;
            if (n.walls & 32u) nb[5] = l;
            double p[6];
#pragma unroll
            for (int d = 0; d < 6; d++) {
                real T = in[nb[d]], z = in[((d >> 1) + 1) * nodes + nb[d]];
                reflect(n, d, T, z);
                p[d] = box_pop(T, z, d & 1);
            }
            real o[4];
            box_collide<real>(c, tab + n.ph * 6, (double)in[l] * 0.25, p, (unsigned long long)n.at, o);
            put(n, s, o, next);
        }
    }
}

static size_t box_lds(int real_bytes, int nx, int ty, int tz, int S, int nphase) {
    const size_t nodes = (size_t)nx * (ty + 2 * (S - 1)) * (tz + 2 * (S - 1));
    return ((size_t)nphase * 6 + (S > 2 ? 2 : 1) * 4 * nodes) * real_bytes;
}

// node updates of one launch of a block
static double box_updates(int nx, int ty, int tz, int S) {
    double n = 0;
    for (int s = 1; s <= S; s++) n += (double)nx * (ty + 2 * (S - s)) * (tz + 2 * (S - s));
    return n;
}

// Time of one launch in microseconds: BOX_T0, BOX_T1 for each step (barrier, LDS
// latency, the chain of sums) and BOX_T2 for each node update of the blocks
// that share a CU.  Measured at 16^3 FP64 with (S, ty, tz): (2, 1, 1) 3.7, (3, 2, 2)
// 5.2, (4, 2, 2) 6.8, (4, 4, 4) 9.0, (5, 2, 2) 9.1; at 32^3 FP32 (2, 2, 2) 4.3.
// On top, what the boxes load beyond the 4 MB of those cells, at 3.7 TB/s, which
// the overlapping halos need: a wider FP64 cell (88 x 64 x 16) took 8.8 with
// (2, 2, 2), 3.7 of them for 20 MB, and is faster in single steps.  Counted from
// the first byte, 16^3 FP64 got (3, 2, 2) and 1.82 us per step; so it takes
// (3, 1, 2) and 1.71.
// The model errs by a tenth, so a box has to promise that much.
constexpr double BOX_T0 = 2.2, BOX_T1 = 0.7, BOX_T2 = 0.0009;

template <typename real>
BoxShape box_shape(int nx, int ny, int nz, int nphase, double other) {
    BoxShape best;
    double tmin = 0.9 * other;
    const long long N = (long long)nx * ny * nz;
    if (N > (1 << 19) || ny < 2 || nz < 2) return best;
    for (int S = 2; S <= 8 && S <= ny && S <= nz; S++)
        for (int ty = 1; ty <= 16 && ty < 2 * ny; ty *= 2)
            for (int tz = 1; tz <= 16 && tz < 2 * nz; tz *= 2) {
                const size_t lds = box_lds(sizeof(real), nx, ty, tz, S, nphase);
                if (lds > (size_t)BOX_LDS) continue;
                const double first = (double)nx * (ty + 2 * (S - 1)) * (tz + 2 * (S - 1));
                const int threads =
                    (int)std::ceil(std::max(first / BOX_NODES, std::min(first, (double)BOX_THREADS)) / 64) * 64;
                if (threads > BOX_THREADS) continue;
                const double blocks = (double)((ny + ty - 1) / ty) * ((nz + tz - 1) / tz);
                const double occ = std::min(1024 / threads, (int)(BOX_LDS / lds));
                const double k = std::min(occ, std::ceil(blocks / BOX_CUS)), rounds = std::ceil(blocks / (BOX_CUS * occ));
                const double bytes = std::max(0.0, blocks * first * sizeof(real) * (sizeof(real) == 8 ? 7 : 4) - 4e6);
                const double t =
                    (BOX_T0 + rounds * (S * BOX_T1 + k * BOX_T2 * box_updates(nx, ty, tz, S)) + bytes / 3.7e6) / S;
                if (t < tmin) {
                    tmin = t;
                    best = BoxShape{S, ty, tz, threads};
                }
            }
    return best;
}

template <typename real>
bool box_takes(const Cell<real> &c) {
    if (c.relax || (!c.storage && sizeof(real) == 4)) return false;
    for (int a = 0; a < 3; a++)
        if (c.phi[a][0] != 0 || c.phi[a][1] != 0) return false;
    return true;
}

template <typename real>
hipError_t launch_box(const Cell<real> &c, const BoxShape &g, int steps, hipStream_t s) {
    const int nty = (c.ny + g.ty - 1) / g.ty, ntz = (c.nz + g.tz - 1) / g.tz;
    const size_t lds = box_lds(sizeof(real), c.nx, g.ty, g.tz, steps, c.nphase);
    const dim3 grid((unsigned)(nty * ntz)), block(g.threads);
    if (c.storage) hipLaunchKernelGGL((k_box<real, 1>), grid, block, lds, s, c, steps, g.ty, g.tz, nty);
    else if constexpr (sizeof(real) == 8)
        hipLaunchKernelGGL((k_box<real, 0>), grid, block, lds, s, c, steps, g.ty, g.tz, nty);
    return hipGetLastError();
}

template BoxShape box_shape<float>(int, int, int, int, double);
template BoxShape box_shape<double>(int, int, int, int, double);
template bool box_takes<float>(const Cell<float> &);
template bool box_takes<double>(const Cell<double> &);
template hipError_t launch_box<float>(const Cell<float> &, const BoxShape &, int, hipStream_t);
template hipError_t launch_box<double>(const Cell<double> &, const BoxShape &, int, hipStream_t);

}  // namespace mrt
