// Weight and bias gradient of the 3x3x3 convolution from tiles staged in LDS.
//
// dW[co][tap cin + ci] = sum_v dy[v][co] x[v + off(tap)][ci] has the voxels as
// its inner dimension while both operands sit channels-last: the MFMA wants
// eight voxels of one channel per lane, memory gives eight channels of one
// voxel.  A block stages a tile of dy and the same tile of x with its halo
// once, as they are (planes of 16 channels), and reads every tap's operand
// from there with the transposing LDS read (16 lanes take a 4 x 16 block and
// each gets one column of it).  k_conv_wgrad_lds, which takes narrow volumes and
// other channel counts, stages a transposed copy of the x columns for each tap,
// two bytes at a time: 27 gathers and 8 LDS writes per 16 bytes.  The whole call
// (kernel, bias gradient, sum of the partials), gathered -> staged: 16 -> 16
// channels on 4 x 64^3 voxels 367 -> 56 us, 32 -> 16 there 638 -> 85, 64 -> 64 on
// 4 x 16^3 74 -> 24; a training iteration 4.37 -> 2.02 ms.  LDS reads bound it
// (two per product at 16 output channels).
//
// Partials and sums are FP32, in another order than the gathering kernel's.  Of
// gradients that cancel (mean zero, 8 to 32 channels on 4 x 64^3 voxels) the
// error against FP64 is 2.4e-7 to 2.7e-7 of their RMS where the gathering
// kernel's is 1.6e-7 to 2.4e-7; on smaller volumes, coarser levels and
// gradients of one sign it lies between four fifths and five fourths of it.
//
// A block owns CO output and CB input channels and all taps (the accumulators
// of its waves; wave w takes the 16-column tiles w, w + 4, ...) and the tiles
// of one voxel split; splits are summed afterwards in a fixed order.  The bias
// gradient is one more product, with ones, in the blocks of the first input
// channels.
#include "nn_tile.hpp"

namespace mrt {

// pitch 12: the lines that two quarters of a wave read are 128 bytes apart
// modulo the 256 of the banks
constexpr int WG_TY = 8, WG_TZ = 4, WG_PITCH = 12;
typedef Tile<WG_TY, WG_TZ, WG_PITCH> WTile;
constexpr int WG_VOX = TILE_X * WG_TY * WG_TZ;

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// One MFMA operand from a plane of 16 channels [position][16]: this lane's
// column, eight consecutive positions of its line.  p: the lane's address for
// the first four positions (row lane % 16 / 4, channels 4 (lane % 4) .. + 3);
// step: bytes of four positions.
__device__ __forceinline__ bf16x8 tr_read(const char *p, int step) {
    typedef s16x4 __attribute__((address_space(3))) *lp;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + step));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

template <int CIN, int CO>
__global__ void __launch_bounds__(256, 2) k_wgrad_tile(const bf16 *__restrict__ x, const bf16 *__restrict__ dy, ConvGeom g,
                                                    int ntiles, float *__restrict__ partials) {
    constexpr int CB = CIN < 32 ? CIN : 32;      // input channels of the block
    constexpr int XP = CB < 16 ? 1 : CB / 16;    // planes of x: 16 channels (8: one plane of 8)
    constexpr int XC = CB < 16 ? CB : 16;        // channels of an x plane
    constexpr int MT = CO / 16;
    constexpr int NT = CIN <= 16 ? (27 * CIN + 31) / 32 * 2 : 27 * XP;  // 16-column tiles (with the padding columns)
    constexpr int PW = (NT + 3) / 4;             // of one wave
    constexpr int XLINE = XC * 2;                // bytes of a position of x
    constexpr int XPLANE = WTile::SPAN * XLINE, DPLANE = WG_VOX * 32;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    char *xs = reinterpret_cast<char *>(smem_raw);
    char *ds = xs + XP * XPLANE;
    char *zs = ds + MT * DPLANE;                 // zeros: 4 positions and more
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quad = lane >> 4, j = lane & 15;
    const int cig = blockIdx.x % (CIN / CB), cog = blockIdx.x / (CIN / CB);
    const int split = blockIdx.y, nsplits = gridDim.y;
    const bool bias = cig == 0 && wave == 0;
    if (threadIdx.x < 16) *reinterpret_cast<u32x4 *>(zs + threadIdx.x * 16) = u32x4{0, 0, 0, 0};

    f32x4 acc[PW][MT], accb[MT];
#pragma unroll
    for (int m = 0; m < MT; m++) {
        accb[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < PW; t++) acc[t][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; e++) ones[e] = (bf16)1.0f;

    // byte offset of each of this wave's column tiles: plane and tap (8
    // channels: two taps, lanes with channels 8.. of the tile take the second)
    int toff[PW];
    bool tzero[PW];
#pragma unroll
    for (int t = 0; t < PW; t++) {
        const int n = t * 4 + wave;
        int tap, plane = 0;
        if constexpr (CIN == 8) tap = 2 * n + ((j & 3) >> 1);
        else if constexpr (CIN == 16) tap = n;
        else tap = n / XP, plane = n % XP;
        tzero[t] = tap >= 27;
        toff[t] = tzero[t] ? 0 : WTile::tap(tap) * XLINE + plane * XPLANE;
    }
    const int col = CIN == 8 ? (j & 1) * 8 : (j & 3) * 8;  // bytes
    const int row = j >> 2;

    typedef WTile::Stage<CB / 8> St;
    constexpr int XPER = St::PASSES;
    const St st;
    char *xto = xs + (CB < 16 ? 0 : st.cg / 2 * XPLANE + st.cg % 2 * 16) + (st.l0 * WG_PITCH + st.hx) * XLINE;
    constexpr int DG = CO / 8, DITEMS = WG_VOX * DG, DPER = DITEMS / 256;
    for (int t0 = split; t0 < ntiles; t0 += nsplits) {
        const WTile tile(g, (unsigned)t0);
        const int xc = st.takes ? tile.column(g, st.hx) : -1, lane_row = tile.row(g, lane);
        const bf16 *from = x + (long long)max(xc, 0) * CIN + cig * CB + st.cg * 8;
        bf16x8 xv[XPER], dv[DPER];
#pragma unroll
        for (int u = 0; u < XPER; u++) {
            const int r = __shfl(lane_row, st.line(u), 64);
            xv[u] = r >= 0 && xc >= 0 ? *reinterpret_cast<const bf16x8 *>(from + (long long)r * CIN) : zero8();
        }
#pragma unroll
        for (int u = 0; u < DPER; u++) {
            const int i = u * 256 + threadIdx.x;
            const int p = tile.inside(g, i / DG);
            dv[u] = p >= 0 ? *reinterpret_cast<const bf16x8 *>(dy + (long long)p * g.cout + cog * CO + i % DG * 8) : zero8();
        }
        __syncthreads();  // the tile before is read
#pragma unroll
        for (int u = 0; u < XPER; u++)
            if (st.stores(u)) *reinterpret_cast<bf16x8 *>(xto + u * St::AT_ONCE * WG_PITCH * XLINE) = xv[u];
#pragma unroll
        for (int u = 0; u < DPER; u++) {
            const int i = u * 256 + threadIdx.x, c = i % DG;
            *reinterpret_cast<bf16x8 *>(ds + c / 2 * DPLANE + i / DG * 32 + c % 2 * 16) = dv[u];
        }
        __syncthreads();
        const bool part = tile.partial(g);
        // chunks of four lines of 8 voxels: the inner dimension of a product
        for (int ch = 0; ch < WG_VOX / 32; ch++) {
            const int z = ch / (WG_TY / 4), y = ch % (WG_TY / 4) * 4 + quad;
            const char *dl = ds + ((z * WG_TY + y) * TILE_X + row) * 32 + (j & 3) * 8;
            bf16x8 a[MT];
#pragma unroll
            for (int m = 0; m < MT; m++) a[m] = tr_read(dl + m * DPLANE, 4 * 32);
            if (bias) {
#pragma unroll
                for (int m = 0; m < MT; m++) accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, accb[m], 0, 0, 0);
            }
            // voxels outside the volume have dy = 0; their x is cleared too, so
            // that what lies there (an infinity, say) does not come in
            u32x4 keep = u32x4{~0u, ~0u, ~0u, ~0u};
            if (part) {
                const bool line = tile.y0 + y < g.H && tile.z0 + z < g.D;
#pragma unroll
                for (int e = 0; e < 4; e++)
                    keep[e] = (line && tile.x0 + 2 * e < g.W ? 0xffffu : 0u) |
                              (line && tile.x0 + 2 * e + 1 < g.W ? 0xffff0000u : 0u);
            }
            const char *xl = xs + ((z * WTile::HY + y) * WG_PITCH + row) * XLINE + col;
#pragma unroll
            for (int t = 0; t < PW; t++) {
                if (t * 4 + 3 >= NT && t * 4 + wave >= NT) continue;
                bf16x8 b = tr_read(tzero[t] ? zs : xl + toff[t], tzero[t] ? 0 : 4 * XLINE);
                if (part) b = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, b) & keep);
#pragma unroll
                for (int m = 0; m < MT; m++) acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[t][m], 0, 0, 0);
            }
        }
    }

    // partial of this split: [cout][kpad], then the bias [cout]; a lane holds
    // output channels 4 quad .. + 3 of column lane % 16
    float *out = partials + (long long)split * ((long long)g.cout * g.kpad + g.cout);
#pragma unroll
    for (int t = 0; t < PW; t++) {
        const int n = t * 4 + wave;
        if (n >= NT) continue;
        const int k = CIN <= 16 ? n * 16 + j : n / XP * CIN + cig * CB + n % XP * 16 + j;
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                out[(long long)(cog * CO + m * 16 + quad * 4 + r) * g.kpad + k] = acc[t][m][r];
    }
    if (bias && j == 0) {
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                out[(long long)g.cout * g.kpad + cog * CO + m * 16 + quad * 4 + r] = accb[m][r];
    }
}

// sum over the splits in a fixed order, four consecutive values per thread of
// a 16-thread group, 16 groups of splits; the tail of a row is the bias
__global__ void __launch_bounds__(256) k_wgrad_sum(const float *__restrict__ partials, long long len, long long main_len,
                                                   int splits, float *__restrict__ dw, float *__restrict__ db) {
    __shared__ f32x4 red[16][16];
    const int o = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const long long i = ((long long)blockIdx.x * 16 + o) * 4;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i < len)
        for (int s = grp; s < splits; s += 16) acc += *reinterpret_cast<const f32x4 *>(partials + (long long)s * len + i);
    red[grp][o] = acc;
    __syncthreads();
    if (grp == 0 && i < len) {
        f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < 16; k++) sum += red[k][o];
        float *out = i < main_len ? dw + i : db + (i - main_len);
        if (i < main_len || db)
#pragma unroll
            for (int e = 0; e < 4; e++) out[e] = sum[e];
    }
}

// tr = 8 x 8 x 4 voxels of a tile; about two blocks for each CU
static int wgrad_groups(const ConvGeom &g) {
    return (g.cin / (g.cin < 32 ? g.cin : 32)) * (g.cout / (g.cout % 32 == 0 ? 32 : 16));
}

int nn_wgrad_tile_splits(const ConvGeom &g) {
    const long long tiles = tile_count(g, WG_TY, WG_TZ);
    const long long s = (512 + wgrad_groups(g) - 1) / wgrad_groups(g);
    return (int)(s < tiles ? s : tiles);
}

bool nn_wgrad_tile_takes(const ConvGeom &g) {
    const long long tiles = tile_count(g, WG_TY, WG_TZ), voxels = (long long)g.n * g.D * g.H * g.W;
    if (tiles >= (1LL << 31)) return false;
    if (g.cin != 8 && g.cin != 16 && g.cin != 32 && g.cin != 64 && g.cin != 128) return false;
    // A tile is summed over whole, so that in narrow volumes and many small ones
    // the kernel that gathers is faster, unless a few tiles are all there are
    // (2048 single voxels, 64 -> 64 channels: 22.8 us gathered, 174 in tiles; one
    // 17.0 and 13.5).  The limits lie where the two meet, over 2500 random shapes.
    return tiles < (g.cin >= 32 ? 16 : 64) || WG_VOX * tiles <= (g.cin >= 32 ? 4 : 5) * voxels;
}

template <int CIN, int CO>
static void launch_wgrad(const bf16 *x, const bf16 *dy, const ConvGeom &g, float *partials, hipStream_t s) {
    constexpr int CB = CIN < 32 ? CIN : 32;
    constexpr size_t lds = (size_t)WTile::SPAN * CB * 2 + (size_t)WG_VOX * CO * 2 + 256;
    const dim3 grid((unsigned)wgrad_groups(g), (unsigned)nn_wgrad_tile_splits(g));
    hipLaunchKernelGGL((k_wgrad_tile<CIN, CO>), grid, dim3(256), lds, s, x, dy, g, (int)tile_count(g, WG_TY, WG_TZ), partials);
}

hipError_t nn_wgrad_tile(const void *x, const void *dy, const ConvGeom &g, float *partials, float *dw, float *db,
                         hipStream_t s) {
    const bf16 *xx = (const bf16 *)x, *dd = (const bf16 *)dy;
    const bool wide = g.cout % 32 == 0;
#define WG(C) case C: wide ? launch_wgrad<C, 32>(xx, dd, g, partials, s) : launch_wgrad<C, 16>(xx, dd, g, partials, s); break
    switch (g.cin) {
        WG(8);
        WG(16);
        WG(32);
        WG(64);
        default: wide ? launch_wgrad<128, 32>(xx, dd, g, partials, s) : launch_wgrad<128, 16>(xx, dd, g, partials, s);
    }
#undef WG
    const long long main_len = (long long)g.cout * g.kpad, len = main_len + g.cout;
    hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)((len / 4 + 15) / 16)), dim3(256), 0, s, partials, len, main_len,
                       nn_wgrad_tile_splits(g), dw, db);
    return hipGetLastError();
}

}  // namespace mrt
