// Two time steps of population storage in one pass over memory.
//
// Single steps move seven values per node in and seven out and run at the rate
// of that copy.  As for moment storage (step2_device.hpp) a block takes a tile
// of whole rows and marches through the planes of a z-chunk: at plane p it
// applies the first step to its rows and one halo row on either side, at
// plane p - 1 the second step.  Each population is read by one node only, so the
// first step pulls straight from memory (no input rows in LDS, no outer halo
// rows); of the intermediate populations f3 and f4 go through LDS to the
// neighbours in y (double-buffered, one barrier per plane), f5 and f6 stay in
// the thread's registers, f1 and f2 are exchanged between lanes.
//
// The arithmetic of a node is that of the single-step kernels, operation by
// operation and with the same random bits, so two single steps and one double
// step agree bit for bit.  FP32 rounds all seven populations with a dither (12
// instructions each, 84 of 147 per node and step), and a block computes its
// halo rows and end planes again: at 96^3, with rows of 24 lanes, two to a wave
// of 64, that and the idle lanes make 1.85 times the arithmetic, and a block's
// start and drain add 7 us (22.4 us a pair, 21.4 two single steps, which the
// rule keeps there).
//
// Per step, single -> two per pass (MI355X): FP64 96^3 16.8 -> 12.1 us, 128^3 35.4
// -> 21.7, 128 x 192 x 192 98.0 -> 52.4, 192^3 162 -> 85, 93 x 63 x 89 15.2 -> 8.4;
// FP32 120^3 17.4 -> 15.3, 128^3 20.0 -> 17.3, 192^3 75 -> 53, 256^3 164 -> 111,
// 123 x 102 x 137 24.2 -> 15.7.
#pragma once

#include "step2_device.hpp"

#pragma clang fp contract(off)

namespace mrt {

// LDS bytes of a block of tr tile rows: phase table in FP64, then two buffers
// of tr + 2 rows of (f3, f4)
__host__ __device__ constexpr long long pop2_lds_bytes(int real_bytes, int tr, int len, int nphase) {
    return 8LL * nphase * TAB2 + 2LL * 2 * len * (tr + 2) * real_bytes;
}

// the populations a node pulls, before the gradient-axis shift
template <typename real, int VEC>
struct Pulled2 {
    real f[7][VEC];  // f0; own f1, f2 of the vector; f3 .. f6 pulled
};

// One step of a thread's vector: s as above, out the seven new populations.
// ph: phases; node: index of the first node.
template <typename real, int VEC, bool RAG, int GA>
__device__ __forceinline__ void pop2_core(const Cell<real> &c, const Lane2 &L, const double *tab,
                                          const Pulled2<real, VEC> &s, uint32_t ph, unsigned node,
                                          real (*out)[VEC]) {
    real s1 = s.f[1][VEC - 1], s2 = s.f[2][0];
    if constexpr (RAG) {
#pragma unroll
        for (int i = 0; i < VEC; i++) {
            if (i == L.tailL) s1 = s.f[1][i];
            if (i == L.tailR) s2 = s.f[2][i];
        }
    }
    real left = lane_get(s1, L.srcL), right = lane_get(s2, L.srcR);
    if (!c.per[0]) {
        if (L.wxl) left = c.sgn[0] * s.f[2][0];
        if (L.wxr) right = c.sgn[0] * s.f[1][VEC - 1];
    }
    const double h = (double)c.h[GA];
    constexpr int H = 2;
#pragma unroll
    for (int v0 = 0; v0 < VEC; v0 += H) {
#pragma unroll
        for (int u = 0; u < H; u++) {
            const int v = v0 + u;
            typedef double d2 __attribute__((ext_vector_type(2)));
            const double *tb = tab + ((ph >> (8 * v)) & 0xffu) * TAB2;
            const d2 t0 = *reinterpret_cast<const d2 *>(tb), t1 = *reinterpret_cast<const d2 *>(tb + 2),
                     t2 = *reinterpret_cast<const d2 *>(tb + 4);
            const double f0 = s.f[0][v];
            double f1 = v == 0 ? left : s.f[1][v - 1], f2 = v == VEC - 1 ? right : s.f[2][v + 1];
            double f3 = s.f[3][v], f4 = s.f[4][v], f5 = s.f[5][v], f6 = s.f[6][v];
            // the shift is zero on the other axes
            if constexpr (GA == 0) f1 += h, f2 -= h;
            else if constexpr (GA == 1) f3 += h, f4 -= h;
            else f5 += h, f6 -= h;
            const double T = ((((((f0 + f1) + f2) + f3) + f4) + f5) + f6);
            const double jx = f1 - f2, jy = f3 - f4, jz = f5 - f6;
            // half of (I - tau^-1): xx, yy | zz, xy | xz, yz
            const double hx = fma(t2[0], jz, fma(t1[1], jy, t0[0] * jx));
            const double hy = fma(t2[1], jz, fma(t0[1], jy, t1[1] * jx));
            const double hz = fma(t1[0], jz, fma(t2[1], jy, t2[0] * jx));
            if constexpr (sizeof(real) == 4) {
                const unsigned key = (node + v) * 8u;
                out[0][v] = dither2(T * 0.25, key);
                out[1][v] = dither2(fma(T, 0.125, hx), key + 1);
                out[2][v] = dither2(fma(T, 0.125, -hx), key + 2);
                out[3][v] = dither2(fma(T, 0.125, hy), key + 3);
                out[4][v] = dither2(fma(T, 0.125, -hy), key + 4);
                out[5][v] = dither2(fma(T, 0.125, hz), key + 5);
                out[6][v] = dither2(fma(T, 0.125, -hz), key + 6);
            } else {
                out[0][v] = T * 0.25;
                out[1][v] = fma(T, 0.125, hx);
                out[2][v] = fma(T, 0.125, -hx);
                out[3][v] = fma(T, 0.125, hy);
                out[4][v] = fma(T, 0.125, -hy);
                out[5][v] = fma(T, 0.125, hz);
                out[6][v] = fma(T, 0.125, -hz);
            }
        }
#pragma unroll
        for (int i = 0; i < 7; i++) settle<real, H>(out[i] + v0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// As march2: the block's rows y0 .. y0 + rows - 1 and planes z0 .. z0 + nplanes - 1,
// LDS laid out for tr rows, blockDim.x a multiple of 64 that holds tr + 2 rows of
// ceil(nx / VEC) lanes, rows whole inside a wave.  7 * N values, N * sizeof(real)
// below 2^31.
template <typename real, int VEC, bool RAG, int NT, int GA>
__device__ __forceinline__ void march2_pop(const Cell<real> &c, char *smem, int tr, int y0, int rows, int z0,
                                           int nplanes) {
    const int nx = c.nx, ny = c.ny, nz = c.nz;
    const long long N = c.N;
    const int nxv = (nx + VEC - 1) / VEC, len = nxv * VEC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rpw = 64 / nxv;
    Lane2 L;
    const int rr = lane / nxv;
    const int xv = lane - rr * nxv;
    L.r = wave * rpw + rr;
    L.act = rr < rpw && L.r < rows + 2;
    const bool xlo = xv == 0, xhi = xv == nxv - 1;
    L.slot = xv * VEC;
    L.x0 = xhi ? nx - VEC : xv * VEC;
    const int rem = nx - (nxv - 1) * VEC;  // new nodes of a row's last vector
    L.tailL = xv == nxv - 2 ? rem - 1 : VEC - 1;
    L.tailR = xhi && !xlo ? VEC - rem : 0;
    L.srcL = 4 * min(xlo ? lane + nxv - 1 : lane - 1, 63);  // min: lanes beyond the last whole row
    L.srcR = 4 * min(xhi ? lane - (nxv - 1) : lane + 1, 63);
    L.wxl = xlo && !c.per[0];
    L.wxr = xhi && !c.per[0];
    const int rl = min(L.r, rows + 1);  // idle threads shadow the last row
    int y = y0 - 1 + rl;
    // halo rows beyond a wall are never used; they stay inside the arrays
    if (c.per[1]) y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
    else y = min(max(y, 0), ny - 1);
    const bool ylo = y == 0 && !c.per[1], yhi = y == ny - 1 && !c.per[1];
    L.wave_wall = __any(ylo || yhi);
    const bool out = L.act && L.r >= 1 && L.r <= rows;
    const bool wave1 = __any(L.act), wave2 = __any(out);
    const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
    // byte offsets from the plane: own row; from f3 of the plane: the row that
    // f3 and f4 come from (a wall reflects the node's own f4 and f3)
    const unsigned nb = (unsigned)N * (unsigned)sizeof(real);
    const unsigned noff = (unsigned)y * nx + L.x0, off = noff * (unsigned)sizeof(real);
    const unsigned off3 = ylo ? off + nb : ((unsigned)ym * nx + L.x0) * (unsigned)sizeof(real);
    const unsigned off4 = yhi ? off : ((unsigned)yp * nx + L.x0) * (unsigned)sizeof(real) + nb;
    const long long plane = (long long)nx * ny;

    double *tab = reinterpret_cast<double *>(smem);
    real *mid = reinterpret_cast<real *>(smem + 8LL * c.nphase * TAB2);  // [parity][tr + 2][f3, f4][len]
    const int buf = (tr + 2) * 2 * len;
    const int own = rl * 2 * len + L.slot;
    // where the second step finds f3 and f4 (rows 1 .. rows, or a wall row itself)
    const int mid3 = ylo ? own + len : max(own - 2 * len, 0), mid4 = yhi ? own : min(rl + 1, tr + 1) * 2 * len + L.slot + len;

    constexpr bool NS = (NT & 2) != 0;
    auto plane_of = [&](int p) __attribute__((always_inline)) {
        if (c.per[2]) return (long long)(p < 0 ? p + nz : (p >= nz ? p - nz : p)) * plane;
        return (long long)min(max(p, 0), nz - 1) * plane;
    };
    const int first = z0 - 1, last = z0 + nplanes;  // planes of the first step
    Pulled2<real, VEC> in;                          // plane p
    Pulled2<real, VEC> M;                           // intermediate: f0, f1, f2 of p - 1; f5 of p - 2
    real M5[VEC];                                   // and of p - 1
    uint32_t ph, Mph = 0;
    auto load = [&](int p) __attribute__((always_inline)) {
        const long long pb = plane_of(p);
        const real *s = c.src + pb;
        const bool zlo = !c.per[2] && p == 0, zhi = !c.per[2] && p == nz - 1;
        row_load<real, VEC, RAG>(s, off, in.f[0]);
        row_load<real, VEC, RAG>(s + N, off, in.f[1]);
        row_load<real, VEC, RAG>(s + 2 * N, off, in.f[2]);
        row_load<real, VEC, RAG>(s + 3 * N, off3, in.f[3]);
        row_load<real, VEC, RAG>(s + 3 * N, off4, in.f[4]);
        row_load<real, VEC, RAG>(zlo ? s + 6 * N : c.src + 5 * N + plane_of(p - 1), off, in.f[5]);
        row_load<real, VEC, RAG>(zhi ? s + 5 * N : c.src + 6 * N + plane_of(p + 1), off, in.f[6]);
        ph = row_phase<VEC>(c.phase + pb, noff);
    };
    auto settle_in = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 7; i++) settle<real, VEC>(in.f[i]);
        asm volatile("" : "+v"(ph));
    };

    load(first);
    for (int i = threadIdx.x; i < c.nphase * 6; i += blockDim.x)
        tab[i / 6 * TAB2 + i % 6] = (double)c.tab[i / 6 * TABW + i % 6];
    settle_in();
#pragma unroll
    for (int v = 0; v < VEC; v++) M.f[0][v] = M.f[1][v] = M.f[2][v] = M.f[5][v] = M5[v] = real(0);
#pragma unroll 1
    for (int p = first; p <= last; p++) {
        // the buffer of parity p - 1 is complete, that of parity p free
        __syncthreads();
        real G[7][VEC];
        const uint32_t Gph = ph;
        if (wave1 && (c.per[2] || (p >= 0 && p < nz))) {  // the plane exists
            if (L.wave_wall) {
                if (ylo) scale_row<real, VEC>(in.f[3], c.sgn[1]);
                if (yhi) scale_row<real, VEC>(in.f[4], c.sgn[1]);
            }
            if (!c.per[2] && p == 0) scale_row<real, VEC>(in.f[5], c.sgn[2]);
            if (!c.per[2] && p == nz - 1) scale_row<real, VEC>(in.f[6], c.sgn[2]);
            unsigned node = (unsigned)plane_of(p) + noff;
            asm volatile("" : "+v"(node));
            pop2_core<real, VEC, RAG, GA>(c, L, tab, in, ph, node, G);
            if (L.act) {
                real *b = mid + (p & 1) * buf + own;
                lds_put<real, VEC>(b, G[3]);
                lds_put<real, VEC>(b + len, G[4]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // the next plane, into registers that are free now; the second step
        // hides its latency
        if (p < last) load(p + 1);
        __builtin_amdgcn_sched_barrier(0);
        const int q = p - 1;
        const bool second = wave2 && p > z0;
        real D[7][VEC];
        if (second) {
            const real *b = mid + (q & 1) * buf;
            lds_get<real, VEC>(b + mid3, M.f[3]);
            lds_get<real, VEC>(b + mid4, M.f[4]);
            if (L.wave_wall) {
                if (ylo) scale_row<real, VEC>(M.f[3], c.sgn[1]);
                if (yhi) scale_row<real, VEC>(M.f[4], c.sgn[1]);
            }
#pragma unroll
            for (int v = 0; v < VEC; v++) M.f[6][v] = !c.per[2] && p == nz ? c.sgn[2] * M5[v] : G[6][v];
            unsigned node = (unsigned)(q * plane) + noff;
            asm volatile("" : "+v"(node));
            pop2_core<real, VEC, RAG, GA>(c, L, tab, M, Mph, node, D);
        }
        // have the plane loaded by now: a wait after the stores would wait for
        // the stores too
        settle_in();
        if (second && out) {
            real *d = c.dst + q * plane;
#pragma unroll
            for (int i = 0; i < 7; i++) row_store<real, VEC, RAG, NS>(d + i * N, off, D[i]);
        }
#pragma unroll
        for (int v = 0; v < VEC; v++) {
            M.f[0][v] = G[0][v];
            M.f[1][v] = G[1][v];
            M.f[2][v] = G[2][v];
            // f5 of the plane below; a low z wall reflects f6
            M.f[5][v] = !c.per[2] && p == 0 ? c.sgn[2] * G[6][v] : M5[v];
            M5[v] = G[5][v];
        }
        Mph = Gph;
    }
}

}  // namespace mrt
