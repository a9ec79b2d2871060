// The two-steps-per-pass kernels (step2_device.hpp) for one cell and for many,
// and how cells are cut into blocks for them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "step2_device.hpp"
#include "step2_internal.h"

namespace mrt {

constexpr int STEP2_LDS = 160 * 1024;
constexpr int STEP2_CUS = 256;
// state beyond the 256 MB last-level cache is written past it
constexpr size_t STEP2_CACHE = 256u << 20;

// threads of the largest block: what the registers of a vector allow
template <typename real, int VEC>
constexpr int step2_max_threads() {
    return sizeof(real) * VEC > 16 ? 512 : 1024;
}

template <typename real, int VEC, bool RAG, int NT, int GA>
__global__ void __launch_bounds__((step2_max_threads<real, VEC>())) k_step2(Cell<real> c, int tr, int ntiles, int nchunks) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    // blocks go to the 8 XCDs round robin: each XCD takes a run of
    // neighbouring tiles, whose halo rows meet in its L2
    const int nb = ntiles * nchunks, per = (nb + 7) / 8;
    const int b = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
    if (b >= nb || (int)(blockIdx.x / 8u) >= per) return;
    const int tile = b % ntiles, chunk = b / ntiles;
    const int y0 = tile * tr;
    const int z0 = (int)((long long)chunk * c.nz / nchunks), z1 = (int)((long long)(chunk + 1) * c.nz / nchunks);
    march2<real, VEC, RAG, NT, GA>(c, reinterpret_cast<real *>(smem_raw), tr, y0, min(tr, c.ny - y0), z0, z1 - z0);
}

// Time of one launch in microseconds, as measured at 64^3 to 256^3 and with
// launches that leave the card idle (128^3 in FP32: 46.5, 36.8, 22.5 and 21.0
// with 60, 80, 255 and 256 blocks).  A block starts and drains in 7; an
// iteration takes 0.45 and the arithmetic of the waves that share a SIMD (one
// vector through both steps: 0.84 for 4 FP32 nodes, 0.48 and 0.84 for 2 and 4
// FP64 nodes); the first and last plane cost half an iteration each; more
// blocks than the card holds take another round.
static double step2_model(double per_wave, int rows, int rpw, long long blocks, int occ, int planes) {
    const int k = (int)std::min<long long>(occ, (blocks + STEP2_CUS - 1) / STEP2_CUS);
    const long long rounds = (blocks + (long long)STEP2_CUS * occ - 1) / ((long long)STEP2_CUS * occ);
    // rows + 2 rows take the first step, rows the second
    const double busy = (rows + 1.0) / rpw * k / 4.0;
    return rounds * (7.0 + (planes + 1) * (per_wave * busy + 0.45));
}

// nodes per thread: a row of nx nodes has to fit one wave
static int step2_vec(int real_bytes, int nx) { return real_bytes == 4 ? 4 : (nx <= 128 ? 2 : 4); }

template <typename real>
bool step2_takes(const Cell<real> &c) {
    if (!c.storage || c.relax) return false;
    // imposed side fluxes would add to every pulled wall population
    for (int a = 0; a < 3; a++)
        if (c.phi[a][0] != 0 || c.phi[a][1] != 0) return false;
    return true;
}

template <typename real>
Step2Shape step2_shape(int nx, int ny, int nz, int nphase) {
    Step2Shape best;
    const long long N = (long long)nx * ny * nz;
    // a row in one wave, 32-bit node numbers and byte offsets in a plane, and
    // no extent of 1 (the halo rows and planes wrap around once)
    const int vec = step2_vec(sizeof(real), nx);
    if (nx < vec || nx > 64 * vec || ny < 2 || nz < 2 || N >= (1LL << 31) || (long long)nx * ny >= (1LL << 28)) return best;
    const int nxv = (nx + vec - 1) / vec, rpw = 64 / nxv, len = nxv * vec;
    const int maxw = (sizeof(real) * vec > 16 ? 512 : 1024) / 64;
    const double per_wave = sizeof(real) == 8 && vec == 2 ? 0.48 : 0.84;
    // two single steps: 2.4 us each and 5.5 (FP32) or 9 (FP64) us per million
    // nodes with vectors of 4 and 2 nodes; with single nodes 1.7 times that and
    // as much more as a row's last block is idle, up to three times (226 random
    // cells of odd rows and under 300000 nodes, whose launches are of a block's
    // length: at three times for all, 16 of them lost more than 3% by taking
    // pairs, 57 x 509 x 4 in FP64 31%; so 4 do, by 11% at most)
    const int single_vec = nx % 4 == 0 ? 4 : (nx % 2 == 0 ? 2 : 1);
    double slope = sizeof(real) == 4 ? 5.5 : 9.0;
    if (single_vec == 1) {
        const int bx = nx > 32 ? 64 : (nx > 16 ? 32 : 16);
        slope *= std::min(3.0, 1.7 * ((nx + bx - 1) / bx * bx) / nx);
    }
    double tmin = 2.0 * (2.4 + slope * 1e-6 * (double)N);
    int before = 0;
    for (int w = 1; w <= maxw; w++) {
        int tr = std::min(w * rpw - 4, ny);
        if (tr < 1) continue;
        const int ntiles = (ny + tr - 1) / tr;
        tr = (ny + ntiles - 1) / ntiles;
        if (tr == before) continue;  // as many rows from more waves
        before = tr;
        const size_t lds = sizeof(real) * (size_t)step2_lds_reals(tr, len, nphase);
        if (lds > (size_t)STEP2_LDS) continue;
        const int waves = (tr + 4 + rpw - 1) / rpw;
        const int occ = std::min(maxw / waves, (int)(STEP2_LDS / lds));
        // each possible number of chunks, with the fewest planes that give it
        for (int planes = nz, per; planes >= 1; planes = per - 1) {
            const int nchunks = (nz + planes - 1) / planes;
            per = (nz + nchunks - 1) / nchunks;
            const double t = step2_model(per_wave, tr, rpw, (long long)ntiles * nchunks, occ, per);
            if (t < tmin) {
                tmin = t;
                best.vec = vec;
                best.tr = tr;
                best.ntiles = ntiles;
                best.nchunks = nchunks;
                best.threads = waves * 64;
                best.lds = lds;
            }
        }
    }
    return best;
}

template <typename real, int VEC, bool RAG, int GA>
static void launch_step2_a(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    const dim3 grid((unsigned)((g.ntiles * g.nchunks + 7) / 8 * 8)), block(g.threads);
    // 256^3 FP32 (537 MB): 55.2 us per step with non-temporal stores, 58.6
    // without; 192^3 (226 MB): 27.9 and 25.7; 128^3 FP64 (134 MB): 16.1 and 13.4
    if (8 * sizeof(real) * (size_t)c.N > STEP2_CACHE)
        hipLaunchKernelGGL((k_step2<real, VEC, RAG, 2, GA>), grid, block, g.lds, s, c, g.tr, g.ntiles, g.nchunks);
    else
        hipLaunchKernelGGL((k_step2<real, VEC, RAG, 0, GA>), grid, block, g.lds, s, c, g.tr, g.ntiles, g.nchunks);
}

template <typename real, int VEC, bool RAG>
static void launch_step2_v(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    if (c.gaxis == 0) launch_step2_a<real, VEC, RAG, 0>(c, g, s);
    else if (c.gaxis == 1) launch_step2_a<real, VEC, RAG, 1>(c, g, s);
    else launch_step2_a<real, VEC, RAG, 2>(c, g, s);
}

template <typename real>
hipError_t launch_step2(const Cell<real> &c, const Step2Shape &g, hipStream_t s) {
    const bool rag = c.nx % g.vec != 0;
    if constexpr (sizeof(real) == 4) {
        if (rag) launch_step2_v<real, 4, true>(c, g, s);
        else launch_step2_v<real, 4, false>(c, g, s);
    } else if (g.vec == 2) {
        if (rag) launch_step2_v<real, 2, true>(c, g, s);
        else launch_step2_v<real, 2, false>(c, g, s);
    } else {
        if (rag) launch_step2_v<real, 4, true>(c, g, s);
        else launch_step2_v<real, 4, false>(c, g, s);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// many cells
// ---------------------------------------------------------------------------

template <typename real, int VEC, bool RAG, int NT, int GA>
__global__ void __launch_bounds__((step2_max_threads<real, VEC>()))
k_batch2(const Cell<real> *__restrict__ cells, const int4 *__restrict__ tiles, int parity, int chunk) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int4 tile = tiles[(int)(blockIdx.x % 8u) * chunk + (int)(blockIdx.x / 8u)];
    const int rows = tile.w & 0xffff, planes = tile.w >> 16;
    if (rows == 0) return;
    Cell<real> c = cells[tile.x];
    if (parity) {
        const real *t = c.src;
        c.src = c.dst;
        c.dst = const_cast<real *>(t);
    }
    march2<real, VEC, RAG, NT, GA>(c, reinterpret_cast<real *>(smem_raw), rows, tile.y, rows, tile.z, planes);
}

template <typename real>
int step2_batch_rows(const Step2Batch &g, const Step2Extent &c) {
    const int rpw = 64 / ((c.nx + g.vec - 1) / g.vec);
    const int tr = std::min(g.threads / 64 * rpw - 4, c.ny);
    if (tr < 1) return 0;
    const int ntiles = (c.ny + tr - 1) / tr;
    return (c.ny + ntiles - 1) / ntiles;
}

template <typename real>
Step2Batch step2_batch_shape(const Step2Extent *cells, int n) {
    Step2Batch g;
    int vec = 0;
    bool narrow = false;  // some row is no multiple of 16 bytes: the single step takes fewer nodes per thread
    double nodes = 0;
    for (int i = 0; i < n; i++) {
        vec = std::max(vec, step2_vec(sizeof(real), cells[i].nx));
        narrow = narrow || cells[i].nx % (sizeof(real) == 4 ? 4 : 2) != 0;
    }
    g.gaxis = cells[0].gaxis;
    for (int i = 0; i < n; i++) {
        const Step2Extent &c = cells[i];
        const long long N = (long long)c.nx * c.ny * c.nz;
        // as for one cell; and one gradient axis, which the kernel is built for
        if (c.nx < vec || c.nx > 64 * vec || c.ny < 2 || c.nz < 2 || N >= (1LL << 31) ||
            (long long)c.nx * c.ny >= (1LL << 28) || c.gaxis != g.gaxis)
            return Step2Batch();
        g.ragged = g.ragged || c.nx % vec != 0;
        nodes += (double)N;
    }
    g.state_bytes = (size_t)(8.0 * sizeof(real) * nodes);
    const int maxw = (sizeof(real) * vec > 16 ? 512 : 1024) / 64;
    const double per_wave = sizeof(real) == 8 && vec == 2 ? 0.48 : 0.84;
    // two single steps: 4.4 us each (a block first reads its tile and its cell) and
    // 6.5 or 9 us per million nodes; all cells share the vector of the narrowest,
    // twice as long with 2 or 1 nodes (FP32: 4 cells of 32..64, 0.3 M nodes 8.7 us;
    // 12 of 64..128, 9.4 M 66; 8 of 46..88 x 32 x 32 in vectors of 2, 0.53 M 10.4; 12
    // of 24..64 with odd rows, 0.71 M 12.2)
    double tmin = 2.0 * (4.4 + (sizeof(real) == 4 ? 6.5 : 9.0) * (narrow ? 1.9 : 1.0) * 1e-6 * nodes);
    Step2Batch best;
    g.vec = vec;
    // 240 combinations: what depends on the cell and one of the two is worked
    // out once (1000 cells: 8 ms with the divisions in the innermost loop, 1.3 like
    // this; a batch chooses anew as cells leave it)
    constexpr int PLANES[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64}, NP = sizeof(PLANES) / sizeof(int);
    struct Chunks { double count, planes; };
    struct Rows { double tiles, busy; };
    std::vector<Chunks> chunks((size_t)NP * n);
    std::vector<Rows> rows(n);
    for (int p = 0; p < NP; p++)
        for (int i = 0; i < n; i++) {
            const int count = (cells[i].nz + PLANES[p] - 1) / PLANES[p];
            chunks[(size_t)p * n + i] = Chunks{(double)count, (double)((cells[i].nz + count - 1) / count)};
        }
    for (int w = 1; w <= maxw; w++) {
        g.threads = 64 * w;
        g.lds = 0;
        bool ok = true;
        for (int i = 0; i < n && ok; i++) {
            const Step2Extent &c = cells[i];
            const int tr = step2_batch_rows<real>(g, c), nxv = (c.nx + vec - 1) / vec;
            ok = tr > 0;
            if (!ok) break;
            g.lds = std::max(g.lds, sizeof(real) * (size_t)step2_lds_reals(tr, nxv * vec, c.nphase));
            rows[i] = Rows{(double)((c.ny + tr - 1) / tr), per_wave * (tr + 1.0) / (64 / nxv)};
        }
        if (!ok || g.lds > (size_t)STEP2_LDS) continue;
        const int occ = std::min(maxw / w, (int)(STEP2_LDS / g.lds));
        for (int p = 0; p < NP; p++) {
            const Chunks *ch = &chunks[(size_t)p * n];
            double blocks = 0;
            for (int i = 0; i < n; i++) blocks += rows[i].tiles * ch[i].count;
            const double k = std::min((double)occ, std::ceil(blocks / STEP2_CUS));
            double work = 0, longest = 0;
            for (int i = 0; i < n; i++) {
                const double t = 7.0 + (ch[i].planes + 1) * (rows[i].busy * k / 4.0 + 0.45);
                work += t * rows[i].tiles * ch[i].count;
                longest = std::max(longest, t);
            }
            // blocks start as others end: half of the longest one is lost at the end
            const double t = std::max(longest, work / (STEP2_CUS * k) + (blocks > STEP2_CUS * k ? 0.5 * longest : 0.0));
            if (t < tmin) {
                tmin = t;
                g.planes = PLANES[p];
                best = g;
            }
        }
    }
    return best;
}

template <typename real, int VEC, bool RAG, int GA>
static void launch_batch2_a(const Cell<real> *cells, const int4 *tiles, int chunk, const Step2Batch &g, int parity,
                            hipStream_t s) {
    const dim3 grid((unsigned)(8 * chunk)), block(g.threads);
    if (g.state_bytes > STEP2_CACHE)
        hipLaunchKernelGGL((k_batch2<real, VEC, RAG, 2, GA>), grid, block, g.lds, s, cells, tiles, parity, chunk);
    else
        hipLaunchKernelGGL((k_batch2<real, VEC, RAG, 0, GA>), grid, block, g.lds, s, cells, tiles, parity, chunk);
}

template <typename real, int VEC, bool RAG>
static void launch_batch2_v(const Cell<real> *cells, const int4 *tiles, int chunk, const Step2Batch &g, int parity,
                            hipStream_t s) {
    if (g.gaxis == 0) launch_batch2_a<real, VEC, RAG, 0>(cells, tiles, chunk, g, parity, s);
    else if (g.gaxis == 1) launch_batch2_a<real, VEC, RAG, 1>(cells, tiles, chunk, g, parity, s);
    else launch_batch2_a<real, VEC, RAG, 2>(cells, tiles, chunk, g, parity, s);
}

template <typename real>
hipError_t launch_batch2(const Cell<real> *cells, const int4 *tiles, int chunk, const Step2Batch &g, int parity,
                         hipStream_t s) {
    if constexpr (sizeof(real) == 4) {
        if (g.ragged) launch_batch2_v<real, 4, true>(cells, tiles, chunk, g, parity, s);
        else launch_batch2_v<real, 4, false>(cells, tiles, chunk, g, parity, s);
    } else if (g.vec == 2) {
        if (g.ragged) launch_batch2_v<real, 2, true>(cells, tiles, chunk, g, parity, s);
        else launch_batch2_v<real, 2, false>(cells, tiles, chunk, g, parity, s);
    } else {
        if (g.ragged) launch_batch2_v<real, 4, true>(cells, tiles, chunk, g, parity, s);
        else launch_batch2_v<real, 4, false>(cells, tiles, chunk, g, parity, s);
    }
    return hipGetLastError();
}

#define MRT_INST2(real)                                                                                            \
    template bool step2_takes<real>(const Cell<real> &);                                                           \
    template Step2Shape step2_shape<real>(int, int, int, int);                                                     \
    template hipError_t launch_step2<real>(const Cell<real> &, const Step2Shape &, hipStream_t);                   \
    template Step2Batch step2_batch_shape<real>(const Step2Extent *, int);                                         \
    template int step2_batch_rows<real>(const Step2Batch &, const Step2Extent &);                                  \
    template hipError_t launch_batch2<real>(const Cell<real> *, const int4 *, int, const Step2Batch &, int, hipStream_t);
MRT_INST2(float)
MRT_INST2(double)

}  // namespace mrt
