// The two-steps-per-pass kernel of population storage (pop2_device.hpp) and how
// a cell is cut into blocks for it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pop2_device.hpp"
#include "step2_internal.h"

namespace mrt {

constexpr int POP2_LDS = 160 * 1024;
constexpr int POP2_CUS = 256;
constexpr size_t POP2_CACHE = 256u << 20;  // state beyond the last-level cache is written past it
constexpr int POP2_THREADS = 512;  // what the registers of a vector of 4 FP64 nodes allow

template <typename real, int VEC, bool RAG, int NT, int GA>
__global__ void __launch_bounds__(POP2_THREADS) k_pop2(Cell<real> c, int tr, int ntiles, int nchunks) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    // blocks go to the 8 XCDs round robin: each XCD takes a run of neighbouring tiles
    const int nb = ntiles * nchunks, per = (nb + 7) / 8;
    const int b = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
    if (b >= nb || (int)(blockIdx.x / 8u) >= per) return;
    const int tile = b % ntiles, chunk = b / ntiles;
    const int y0 = tile * tr;
    const int z0 = (int)((long long)chunk * c.nz / nchunks), z1 = (int)((long long)(chunk + 1) * c.nz / nchunks);
    march2_pop<real, VEC, RAG, NT, GA>(c, reinterpret_cast<char *>(smem_raw), tr, y0, min(tr, c.ny - y0), z0, z1 - z0);
}

// nodes per thread: a row of nx nodes has to fit one wave
static int pop2_vec(int real_bytes, int nx) { return real_bytes == 4 ? 4 : (nx <= 128 ? 2 : 4); }

template <typename real>
bool pop2_takes(const Cell<real> &c) {
    if (c.storage || c.relax) return false;
    for (int a = 0; a < 3; a++)
        if (c.phi[a][0] != 0 || c.phi[a][1] != 0) return false;
    return true;
}

// Time of one launch in microseconds: a block starts and drains in 7; a plane
// takes 0.45 and, for each wave that a SIMD has to work through, 1.75 (4 FP32
// nodes, whose dithers are most of it), 0.5 or 0.9 (2 or 4 FP64 nodes); the first
// and last plane cost half each; more blocks than the card holds take another
// round; and what the blocks load, halo included, and store moves at 7.2 TB/s
// at best.  Measured with (rows, z-chunks): FP32 96^3 (14, 32) 22.7, (6, 16)
// 23.9, (8, 12) 40; 128^3 (6, 16) 40; 192^3 (6, 8) 109; FP64 96^3 (6, 16) 22.7,
// (4, 10) 23.6, (4, 20) 26.8, (6, 24) 27.9; 128^3 (4, 8) 43.4.
static double pop2_model(int real_bytes, int vec, double nodes, int tr, int waves, long long blocks, int occ, int planes) {
    const int k = (int)std::min<long long>(occ, (blocks + POP2_CUS - 1) / POP2_CUS);
    const long long rounds = (blocks + (long long)POP2_CUS * occ - 1) / ((long long)POP2_CUS * occ);
    const double busy = (double)((waves * k + 3) / 4), per_wave = real_bytes == 4 ? 1.75 : (vec == 2 ? 0.5 : 0.9);
    const double bytes = 7.0 * real_bytes * nodes * (1.0 + (tr + 2.0) / tr * (planes + 2.0) / planes);
    const double run = rounds * (7.0 + (planes + 1) * (per_wave * busy + 0.45)), move = 3.0 + bytes / 7.2e6;
    // they overlap, though not wholly (by the maximum alone, 128 x 192 x 192 FP64
    // took fewer blocks with fewer halo bytes and 148 us; 108 like this)
    return std::max(run, move) + 0.1 * std::min(run, move);
}

template <typename real>
Step2Shape pop2_shape(int nx, int ny, int nz, int nphase) {
    Step2Shape best;
    const long long N = (long long)nx * ny * nz;
    // a row in one wave, 32-bit node numbers, dither keys and byte offsets, and
    // no extent of 1 (the halo rows and planes wrap around once)
    const int vec = pop2_vec(sizeof(real), nx);
    if (nx < vec || nx > 64 * vec || ny < 2 || nz < 2 || N * (long long)sizeof(real) >= (1LL << 31)) return best;
    const int nxv = (nx + vec - 1) / vec, rpw = 64 / nxv, len = nxv * vec, maxw = POP2_THREADS / 64;
    // two single steps: 2.4 us each and 8.6 (FP32) or 15.5 (FP64) us per million
    // nodes (FP32 64^3 4.6, 96^3 10.7, 128^3 20.2; FP64 96^3 16.0, 128^3 35.3), with
    // odd rows 9 to 17 and 17 to 32 (one node per thread; FP32 123 x 102 x 137 24.3)
    const double slope = (sizeof(real) == 4 ? 8.6 : 15.5) * (nx % 2 ? 1.3 : 1.0);
    const double single = 2.4 + slope * 1e-6 * (double)N;
    double tmin = 0.95 * 2.0 * single;
    int before = 0;
    for (int w = 1; w <= maxw; w++) {
        int tr = std::min(w * rpw - 2, ny);
        if (tr < 1) continue;
        const int ntiles = (ny + tr - 1) / tr;
        tr = (ny + ntiles - 1) / ntiles;
        if (tr == before) continue;  // as many rows from more waves
        before = tr;
        const size_t lds = (size_t)pop2_lds_bytes(sizeof(real), tr, len, nphase);
        if (lds > (size_t)POP2_LDS) continue;
        const int waves = (tr + 2 + rpw - 1) / rpw;
        // waves whose registers a SIMD holds.  Of 5 or 6 waves two share a SIMD, and a
        // second block of them does not fit beside the first (counted as if it did,
        // FP32 120^3 took blocks of 6 and 20.3 us per step; single 17.5, blocks of 8 15.8)
        const int simd = sizeof(real) * vec > 16 ? 2 : 3;
        const int occ = std::min(waves > 4 ? simd / ((waves + 3) / 4) : 4 * simd / waves, (int)(POP2_LDS / lds));
        // each possible number of chunks, with the fewest planes that give it
        for (int planes = nz, per; planes >= 1; planes = per - 1) {
            const int nchunks = (nz + planes - 1) / planes;
            per = (nz + nchunks - 1) / nchunks;
            const double t = pop2_model(sizeof(real), vec, (double)N, tr, waves, (long long)ntiles * nchunks, occ, per);
            if (t < tmin) {
                tmin = t;
                best = Step2Shape{vec, tr, ntiles, nchunks, waves * 64, lds};
            }
        }
    }
    return best;
}

template <typename real, int VEC, bool RAG, int GA>
static void launch_pop2_a(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    const dim3 grid((unsigned)((g.ntiles * g.nchunks + 7) / 8 * 8)), block(g.threads);
    if (14 * sizeof(real) * (size_t)c.N > POP2_CACHE)
        hipLaunchKernelGGL((k_pop2<real, VEC, RAG, 2, GA>), grid, block, g.lds, s, c, g.tr, g.ntiles, g.nchunks);
    else
        hipLaunchKernelGGL((k_pop2<real, VEC, RAG, 0, GA>), grid, block, g.lds, s, c, g.tr, g.ntiles, g.nchunks);
}

template <typename real, int VEC, bool RAG>
static void launch_pop2_v(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    if (c.gaxis == 0) launch_pop2_a<real, VEC, RAG, 0>(c, g, s);
    else if (c.gaxis == 1) launch_pop2_a<real, VEC, RAG, 1>(c, g, s);
    else launch_pop2_a<real, VEC, RAG, 2>(c, g, s);
}

template <typename real>
hipError_t launch_pop2(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    const bool rag = c.nx % g.vec != 0;
    if (g.vec == 4) {
        if (rag) launch_pop2_v<real, 4, true>(c, g, s);
        else launch_pop2_v<real, 4, false>(c, g, s);
    } else if constexpr (sizeof(real) == 8) {
        if (rag) launch_pop2_v<real, 2, true>(c, g, s);
        else launch_pop2_v<real, 2, false>(c, g, s);
    }
    return hipGetLastError();
}

#define MRT_INSTP(real)                                            \
    template bool pop2_takes<real>(const Cell<real> &);            \
    template Step2Shape pop2_shape<real>(int, int, int, int);      \
    template hipError_t launch_pop2<real>(const Cell<real> &, const Step2Shape &, hipStream_t);
MRT_INSTP(float)
MRT_INSTP(double)

}  // namespace mrt
