// Two time steps of moment storage in one pass over memory.
//
// The single-step kernel moves the whole state through memory once per step:
// at 256^3 in FP32 that is 5.75 TB/s, more than a copy of four arrays reaches
// (5.12), so only fewer bytes can make it faster.  Here a block takes a tile of whole rows (all x,
// `rows` rows in y) and marches through the planes of a z-chunk.  At plane p
// it applies the first step to its rows and to one halo row on either side,
// keeps the result on chip, and applies the second step to plane p - 1, whose
// neighbours are complete by then:
//   registers: a thread keeps its own vector of the input planes p - 1, p,
//     p + 1 and of the intermediate planes p - 2, p - 1, p (all it needs in z);
//   LDS: (T, jhat_y/2) of the input plane p and of the intermediate plane
//     p - 1, for the neighbours in y; double-buffered, one barrier per plane;
//   x neighbours: lane exchange, a row lies inside one wave.
// The halo rows and the chunk's first and last intermediate plane are computed
// twice (by the neighbouring blocks too); nothing is exchanged between blocks.
//
// Per step, single -> two per pass (MI355X): FP32 256^3 95.6 -> 55.2 us, 192^3
// 39.2 -> 25.6, 128^3 12.9 -> 10.5, 75 x 61 x 87 8.8 -> 5.6; FP64 256^3 195.5 ->
// 106.6, 128^3 21.6 -> 13.4; batches in FP32, 24 solves of 64..128 per axis
// 136 -> 84, 32 of 32..64 29.8 -> 22.0, 9 unit cells of 56 x 56 28.7 -> 18.2.
// What bounds it now is the arithmetic (57 vector instructions per node and
// step, 63 of 110 us at 256^3) together with the 580 MB that two steps still
// move (measured, 5.26 TB/s; 553 MB without the halo rows read again).
// Registers decide the layout: the planes of a vector of 4 leave 128 per wave
// only if each value is dropped as soon as its last use is past (see settle);
// with 140 a few spilled values made every prefetch wait, 98 us per step.
//
// The arithmetic of a node is that of the single-step kernel, operation by
// operation, so two single steps and one double step agree bit for bit:
//   FP32: populations T/8 +- jhat/2 exact in FP64, T summed in FP64 and
//     dithered to FP32, jhat from the FP32 flux;
//   FP64: populations rounded as population storage rounds them.
// A product by 1/8 is exact, so the fused T/8 + z equals the separate product
// and sum of the single-step kernel.  A wall link takes the node's own
// opposite population: T/8 + z of (sgn T, -sgn z) is sgn (T/8 - z) exactly.
#pragma once

#include "lbm_device.hpp"

#pragma clang fp contract(off)

namespace mrt {

constexpr int TAB2 = 8;  // table reals per phase in LDS: half (I - tau^-1) [6], padded

// what a thread keeps of a plane
template <typename real, int VEC>
struct TZ {
    real T[VEC], Z[VEC];
};

// Rows whose length is no multiple of VEC (RAG): the last vector of a row is
// moved back to end with the row, so that every thread holds VEC valid nodes;
// the nodes it shares with the vector before are computed twice, with the
// same result.  Global accesses are then aligned to one value only, which the
// vector memory instructions allow.
template <typename real, int VEC, bool RAG>
struct VecOf {
    typedef real type __attribute__((ext_vector_type(VEC)));
};
template <typename real, int VEC>
struct VecOf<real, VEC, true> {
    typedef real type __attribute__((ext_vector_type(VEC), aligned(sizeof(real))));
};

// base: the same for the whole block; off: this thread's byte offset (a
// uniform 64-bit base and a 32-bit offset need one register per address)
#define MRT_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T MRT_GLOBAL *uniform(T *base) {
    T MRT_GLOBAL *p = (T MRT_GLOBAL *)base;
    asm("" : "+s"(p));  // kept apart from the thread's offset
    return p;
}

template <typename real, int VEC, bool RAG>
__device__ __forceinline__ void row_load(const real *base, unsigned off, real *v) {
    typedef typename VecOf<real, VEC, RAG>::type vt;
    asm volatile("" : "+v"(off));  // extended to 64 bits by the load itself
    const vt MRT_GLOBAL *q = (const vt MRT_GLOBAL *)((const char MRT_GLOBAL *)uniform(base) + off);
    const vt t = *q;
#pragma unroll
    for (int i = 0; i < VEC; i++) v[i] = t[i];
}

template <typename real, int VEC, bool RAG, bool NT>
__device__ __forceinline__ void row_store(real *base, unsigned off, const real *v) {
    typedef typename VecOf<real, VEC, RAG>::type vt;
    asm volatile("" : "+v"(off));
    vt MRT_GLOBAL *p = (vt MRT_GLOBAL *)((char MRT_GLOBAL *)uniform(base) + off);
    vt t;
#pragma unroll
    for (int i = 0; i < VEC; i++) t[i] = v[i];
    if constexpr (NT) __builtin_nontemporal_store(t, p);
    else *p = t;
}

template <int VEC>
__device__ __forceinline__ uint32_t row_phase(const uint8_t *base, unsigned off) {
    asm volatile("" : "+v"(off));
    const uint8_t MRT_GLOBAL *p = uniform(base) + off;
    typedef uint32_t u32 __attribute__((aligned(1)));
    typedef uint16_t u16 __attribute__((aligned(1)));
    if constexpr (VEC == 4) return *(const u32 MRT_GLOBAL *)p;
    else return *(const u16 MRT_GLOBAL *)p;
}

template <typename real, int VEC>
__device__ __forceinline__ void lds_get(const real *p, real *v) {
    typedef real vt __attribute__((ext_vector_type(VEC)));
    const vt t = *reinterpret_cast<const vt *>(p);
#pragma unroll
    for (int i = 0; i < VEC; i++) v[i] = t[i];
}

template <typename real, int VEC>
__device__ __forceinline__ void lds_put(real *p, const real *v) {
    typedef real vt __attribute__((ext_vector_type(VEC)));
    vt t;
#pragma unroll
    for (int i = 0; i < VEC; i++) t[i] = v[i];
    *reinterpret_cast<vt *>(p) = t;
}

// dither_to_float for node indices below 2^32
__device__ __forceinline__ float dither2(double x, unsigned node) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned key = mix32(__builtin_amdgcn_bitop3_b32((unsigned)b, (unsigned)(b >> 32), node * 0x9E3779B9u, 0x96));
    return (float)__longlong_as_double((long long)((b + (unsigned long long)(key >> 3)) & ~0x1FFFFFFFull));
}

__device__ __forceinline__ double pop2(double T, double z) { return fma(T, 0.125, z); }

// A thread's place: its row of the tile and the x-vector it holds.
struct Lane2 {
    int r;             // 0 .. rows + 3: two halo rows on either side, the outer ones only read
    int x0, slot;      // first node of its vector; the vector's place in an LDS row
    int tailL, tailR;  // elements that the lanes right / left of it take as neighbours
    int srcL, srcR;    // four times the lanes that hold the x neighbours (wrapped)
    bool act;          // the thread holds a row of the tile
    bool wxl, wxr;     // its first / last node lies on an x wall
    bool wyl, wyh;     // the row lies on the low / high y wall
    bool wave_wall;    // some row of the wave lies on a y wall
    float h2;          // FP32: twice the gradient-axis shift
};

// the value of another lane; at: four times its number
__device__ __forceinline__ float lane_get(float v, int at) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(at, __float_as_int(v)));
}
__device__ __forceinline__ double lane_get(double v, int at) {
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(at, __double2hiint(v)),
                            __builtin_amdgcn_ds_bpermute(at, __double2loint(v)));
}

template <typename real, int n>
__device__ __forceinline__ void scale_row(real *v, real f) {
#pragma unroll
    for (int i = 0; i < n; i++) v[i] *= f;
}

// Hides where values came from, and has them computed by now.  The compiler
// would otherwise keep the FP64 copies that one iteration made of FP32 values
// for the next one, and put off the products with the phase table to where
// their results are used, an iteration later, with all operands kept: more
// registers than a wave has.
template <typename real, int VEC>
__device__ __forceinline__ void settle(real *v) {
#pragma unroll
    for (int i = 0; i < VEC; i++) asm volatile("" : "+v"(v[i]));
}

// One step of a thread's vector.  Tc, Xc: own T and jhat_x; row: LDS row of
// this thread's vector (T there, jhat_y len further, the neighbouring rows
// 2 len before and after); Tzm .. Zzp: (T, jhat_z) pulled along z, walls
// already folded in; node: index of the first node; o*: the new moments; GA:
// the gradient axis, the only one with a shift.
// The vector is worked through two nodes at a time, which bounds the registers.
template <typename real, int VEC, bool RAG, int GA>
__device__ __forceinline__ void step2_core(const Cell<real> &c, const Lane2 &L, const real *tab, const real *Tc,
                                           const real *Xc, const real *row, int len, const real *Tzm, const real *Zzm,
                                           const real *Tzp, const real *Zzp, uint32_t ph, unsigned node, real *oT,
                                           real *oX, real *oY, real *oZ) {
    // x neighbours by lane exchange
    real sRT = Tc[VEC - 1], sRX = Xc[VEC - 1], sLT = Tc[0], sLX = Xc[0];
    if constexpr (RAG) {
#pragma unroll
        for (int i = 0; i < VEC; i++) {
            if (i == L.tailL) { sRT = Tc[i]; sRX = Xc[i]; }
            if (i == L.tailR) { sLT = Tc[i]; sLX = Xc[i]; }
        }
    }
    real lT = lane_get(sRT, L.srcL), lX = lane_get(sRX, L.srcL);
    real rT = lane_get(sLT, L.srcR), rX = lane_get(sLX, L.srcR);
    if (!c.per[0]) {
        if (L.wxl) { lT = c.sgn[0] * Tc[0]; lX = -c.sgn[0] * Xc[0]; }
        if (L.wxr) { rT = c.sgn[0] * Tc[VEC - 1]; rX = -c.sgn[0] * Xc[VEC - 1]; }
    }
    const real *lo = row + (L.wyl ? 0 : -2 * len), *hi = row + (L.wyh ? 0 : 2 * len);
    constexpr int H = 2;
#pragma unroll
    for (int v0 = 0; v0 < VEC; v0 += H) {
        real Tym[H], Yym[H], Typ[H], Yyp[H];
        lds_get<real, H>(lo + v0, Tym);
        lds_get<real, H>(lo + len + v0, Yym);
        lds_get<real, H>(hi + v0, Typ);
        lds_get<real, H>(hi + len + v0, Yyp);
        if (L.wave_wall) {
            if (L.wyl) { scale_row<real, H>(Tym, c.sgn[1]); scale_row<real, H>(Yym, -c.sgn[1]); }
            if (L.wyh) { scale_row<real, H>(Typ, c.sgn[1]); scale_row<real, H>(Yyp, -c.sgn[1]); }
        }
#pragma unroll
        for (int u = 0; u < H; u++) {
            const int v = v0 + u;
            // half of (I - tau^-1): xx, yy, zz, xy | xz, yz
            typedef real r4 __attribute__((ext_vector_type(4)));
            typedef real r2 __attribute__((ext_vector_type(2)));
            const real *tb = tab + ((ph >> (8 * v)) & 0xffu) * TAB2;
            const r4 ta = *reinterpret_cast<const r4 *>(tb);
            const r2 tc = *reinterpret_cast<const r2 *>(tb + 4);
            const double p1 = v == 0 ? pop2(lT, lX) : pop2(Tc[v - 1], Xc[v - 1]);
            const double p2 = v == VEC - 1 ? pop2(rT, -(double)rX) : pop2(Tc[v + 1], -(double)Xc[v + 1]);
            const double p3 = pop2(Tym[u], Yym[u]), p4 = pop2(Typ[u], -(double)Yyp[u]);
            const double p5 = pop2(Tzm[v], Zzm[v]), p6 = pop2(Tzp[v], -(double)Zzp[v]);
            // (T/4 and its sum with p1 in one operation: the product is exact)
            if constexpr (sizeof(real) == 4) {
                const double T64 = fma((double)Tc[v], 0.25, p1) + p2 + p3 + p4 + p5 + p6;
                float jx = (float)(p1 - p2), jy = (float)(p3 - p4), jz = (float)(p5 - p6);
                if constexpr (GA == 0) jx += L.h2;
                else if constexpr (GA == 1) jy += L.h2;
                else jz += L.h2;
                oT[v] = dither2(T64, node + v);
                oX[v] = fmaf(tc[0], jz, fmaf(ta[3], jy, ta[0] * jx));
                oY[v] = fmaf(tc[1], jz, fmaf(ta[1], jy, ta[3] * jx));
                oZ[v] = fmaf(ta[2], jz, fmaf(tc[1], jy, tc[0] * jx));
            } else {
                // the shift is zero on the other axes
                const double f1 = GA == 0 ? p1 + c.h[0] : p1, f2 = GA == 0 ? p2 - c.h[0] : p2;
                const double f3 = GA == 1 ? p3 + c.h[1] : p3, f4 = GA == 1 ? p4 - c.h[1] : p4;
                const double f5 = GA == 2 ? p5 + c.h[2] : p5, f6 = GA == 2 ? p6 - c.h[2] : p6;
                const double jx = f1 - f2, jy = f3 - f4, jz = f5 - f6;
                oT[v] = fma((double)Tc[v], 0.25, f1) + f2 + f3 + f4 + f5 + f6;
                oX[v] = fma(tc[0], jz, fma(ta[3], jy, ta[0] * jx));
                oY[v] = fma(tc[1], jz, fma(ta[1], jy, ta[3] * jx));
                oZ[v] = fma(ta[2], jz, fma(tc[1], jy, tc[0] * jx));
            }
        }
        settle<real, H>(oT + v0), settle<real, H>(oX + v0), settle<real, H>(oY + v0), settle<real, H>(oZ + v0);
        // the next two nodes' operands are read after this point
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
}

// LDS reals of a block of tr tile rows: phase table, then two buffers each of
// the input plane and of the intermediate plane, tr + 4 rows of (T, jhat_y)
__host__ __device__ constexpr long long step2_lds_reals(int tr, int len, int nphase) {
    return (long long)nphase * TAB2 + 4LL * 2 * len * (tr + 4);
}

// The block's tile: rows y0 .. y0 + rows - 1 and planes z0 .. z0 + nplanes - 1
// of cell c.  tr: rows the LDS is laid out for (rows <= tr).  blockDim.x is a
// multiple of 64 and holds tr + 4 rows of ceil(nx / VEC) lanes, rows whole
// inside a wave.  NT bit 1: non-temporal stores, as for the single step.
template <typename real, int VEC, bool RAG, int NT, int GA>
__device__ __forceinline__ void march2(const Cell<real> &c, real *smem, int tr, int y0, int rows, int z0,
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
    L.act = rr < rpw && L.r < rows + 4;
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
    const int rl = min(L.r, rows + 3);  // idle threads shadow the last row
    int y = y0 - 2 + rl;
    float h2 = 2.0f * (float)c.h[GA];
    asm("" : "+v"(h2));
    L.h2 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(h2)));  // one copy per wave
    // the outer halo rows take no neighbours; as wall rows they read their own
    L.wyl = (y == 0 && !c.per[1]) || rl == 0;
    L.wyh = (y == ny - 1 && !c.per[1]) || rl == rows + 3;
    L.wave_wall = __any(L.act && ((y == 0 || y == ny - 1) && !c.per[1]));
    // halo rows beyond a wall are never used; they stay inside the arrays
    if (c.per[1]) y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
    else y = min(max(y, 0), ny - 1);
    const bool first_step = L.act && L.r >= 1 && L.r <= rows + 2;
    const bool out = L.act && L.r >= 2 && L.r <= rows + 1;
    const bool wave1 = __any(first_step), wave2 = __any(out);  // this wave has work in the first / second step
    const unsigned noff = (unsigned)y * nx + L.x0, off = noff * sizeof(real);
    const long long plane = (long long)nx * ny;

    real *tab = smem;
    const int buf = (tr + 4) * 2 * len;  // [input, intermediate][parity][tr + 4][T, Y][len]
    real *own = tab + (long long)c.nphase * TAB2 + rl * 2 * len + L.slot;

    constexpr bool NS = (NT & 2) != 0;
    // planes -2 .. nz + 1 (nz >= 2); beyond a wall: any plane, its values are not used
    auto plane_of = [&](int p) __attribute__((always_inline)) {
        if (c.per[2]) return (long long)(p < 0 ? p + nz : (p >= nz ? p - nz : p)) * plane;
        return (long long)min(max(p, 0), nz - 1) * plane;
    };
    const int first = z0 - 1, last = z0 + nplanes;  // planes of the first step
    TZ<real, VEC> A, B, C, P, Q, R;   // input planes p - 1, p, p + 1; intermediate planes p - 2, p - 1, p
    real X[VEC], QX[VEC];             // jhat_x of p and of the intermediate plane p - 1
    real Y[VEC];                      // jhat_y of p + 1
    uint32_t ph, Qph = 0;
    // the plane beyond a z wall is the wall plane with its populations
    // reflected: (sgn T, -sgn jhat_z)
    auto fold_z = [&](const TZ<real, VEC> &own_p, TZ<real, VEC> &nb) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < VEC; v++) {
            nb.T[v] = c.sgn[2] * own_p.T[v];
            nb.Z[v] = -c.sgn[2] * own_p.Z[v];
        }
    };
    auto load_tz = [&](int p, TZ<real, VEC> &v) __attribute__((always_inline)) {
        const real *s = c.src + plane_of(p);
        row_load<real, VEC, RAG>(s, off, v.T);
        if (first_step) row_load<real, VEC, RAG>(s + 3 * N, off, v.Z);
        if (!c.per[2] && (p == -1 || p == nz)) fold_z(v, v);
    };
    auto load_xy = [&](int p) __attribute__((always_inline)) {
        const long long pb = plane_of(p);
        const real *s = c.src + pb;
        row_load<real, VEC, RAG>(s + 2 * N, off, Y);
        if (first_step) {
            row_load<real, VEC, RAG>(s + N, off, X);
            ph = row_phase<VEC>(c.phase + pb, noff);
        }
    };
    auto put_in = [&](int p, const TZ<real, VEC> &v) __attribute__((always_inline)) {
        real *b = own + (p & 1) * buf;
        if (L.act) {
            lds_put<real, VEC>(b, v.T);
            lds_put<real, VEC>(b + len, Y);
        }
    };
    auto iterate = [&](int p, TZ<real, VEC> &A, TZ<real, VEC> &B, TZ<real, VEC> &C, TZ<real, VEC> &P,
                       TZ<real, VEC> &Q, TZ<real, VEC> &R) __attribute__((always_inline)) {
        // the buffers of parity p are complete, those of parity p + 1 free
        __syncthreads();
        settle<real, VEC>(A.T), settle<real, VEC>(A.Z), settle<real, VEC>(B.T);
        real RX[VEC];
        const uint32_t Rph = ph;
        if (wave1 && (c.per[2] || (p >= 0 && p < nz))) {  // the plane exists
            unsigned node = (unsigned)plane_of(p) + noff;
            asm volatile("" : "+v"(node));
            real RY[VEC];
            step2_core<real, VEC, RAG, GA>(c, L, tab, B.T, X, own + (p & 1) * buf, len, A.T, A.Z, C.T, C.Z, ph, node, R.T, RX,
                                       RY, R.Z);
            if (first_step) {
                real *b = own + (2 + ((p + 1) & 1)) * buf;
                lds_put<real, VEC>(b, R.T);
                lds_put<real, VEC>(b + len, RY);
            }
            if (!c.per[2] && p == 0) fold_z(R, Q);
        }
        // the next planes, into registers that are free now; the second step
        // hides their latency
        __builtin_amdgcn_sched_barrier(0);
        if (p < last) {
            load_xy(p + 1);
            load_tz(p + 2, A);
        }
        __builtin_amdgcn_sched_barrier(0);
        settle<real, VEC>(P.T), settle<real, VEC>(P.Z), settle<real, VEC>(Q.T);
        const int q = p - 1;
        const bool second = wave2 && p > z0;
        real oT[VEC], oX[VEC], oY[VEC], oZ[VEC];
        if (second) {
            if (!c.per[2] && p == nz) fold_z(Q, R);
            unsigned node = (unsigned)(q * plane) + noff;
            asm volatile("" : "+v"(node));
            step2_core<real, VEC, RAG, GA>(c, L, tab, Q.T, QX, own + (2 + (p & 1)) * buf, len, P.T, P.Z, R.T, R.Z, Qph, node,
                                           oT, oX, oY, oZ);
        }
        if (p < last) put_in(p + 1, C);
        // have the planes loaded by now: a wait after the stores would wait
        // for the stores too
        settle<real, VEC>(X), settle<real, VEC>(Y), settle<real, VEC>(A.T), settle<real, VEC>(A.Z);
        asm volatile("" : "+v"(ph));
        if (second && out) {
            real *d = c.dst + q * plane;
            row_store<real, VEC, RAG, NS>(d, off, oT);
            row_store<real, VEC, RAG, NS>(d + N, off, oX);
            row_store<real, VEC, RAG, NS>(d + 2 * N, off, oY);
            row_store<real, VEC, RAG, NS>(d + 3 * N, off, oZ);
        }
#pragma unroll
        for (int v = 0; v < VEC; v++) QX[v] = RX[v];
        Qph = Rph;
    };

    load_tz(first - 1, A);
    load_tz(first, B);
    load_xy(first);
    load_tz(first + 1, C);
    for (int i = threadIdx.x; i < c.nphase * 6; i += blockDim.x) tab[i / 6 * TAB2 + i % 6] = c.tab[i / 6 * TABW + i % 6];
    put_in(first, B);
    settle<real, VEC>(A.T), settle<real, VEC>(A.Z), settle<real, VEC>(B.T), settle<real, VEC>(B.Z);
    settle<real, VEC>(C.T), settle<real, VEC>(C.Z), settle<real, VEC>(X);
    asm volatile("" : "+v"(ph));
    // the planes' registers rotate with period 3
    for (int p = first;;) {
        iterate(p, A, B, C, P, Q, R);
        if (p++ == last) break;
        iterate(p, B, C, A, Q, R, P);
        if (p++ == last) break;
        iterate(p, C, A, B, R, P, Q);
        if (p++ == last) break;
    }
}

}  // namespace mrt
