// Forward 3x3x3 convolution (and input gradient) of the warm-start network
// with the activations staged in LDS.
//
// out^T [cout][voxels] = w [cout][27 cin] x^T: the weights are the A operand
// and the voxels the columns, so that a lane ends with four neighbouring
// channels of one voxel and stores them together.  Each of a block's four
// waves takes MT groups of 16 voxels of the tile and NT groups of 16 channels;
// all read the same weights (L1) and their own voxels (LDS, one 16-byte read
// per product, planes of 8 channels so that neighbouring lanes read
// neighbouring 16 bytes).  Gathered from memory for each tap, as k_conv_fwd does
// (it still takes narrow volumes, other channel counts and alignments), the
// operands cost 27 reads of every activation through L1, which bound it.  The products and their order (tap, then channel, in
// chunks of 32) are those of k_conv_fwd: the results agree bit for bit.
//
// Gathered -> staged (MI355X): 16 -> 16 channels on 4 x 64^3 voxels 89 -> 40.7 us,
// on 64^3 26.8 -> 14; 32 -> 16 on 64^3 53.7 -> 17; 64 -> 64 on 16^3 29.8 -> 11;
// 128 -> 128 on 8^3 38.1 -> 18.8; one inference of a 128^3 cell 0.58 -> 0.30 ms.
// LDS reads (one per product at 16 output channels) and, on the coarse
// levels, the chain of 54 or 108 dependent products bound it now.
#include "nn_tile.hpp"

namespace mrt {

// positions of a plane of 8 channels, a zero vector behind its voxels.  The
// large tile's planes lie a multiple of 16 apart, as neighbouring quarters of
// a wave read neighbouring ones; the small tiles, where the LDS is not what a
// launch waits for, gain nothing from that (64 -> 64 on 16^3 10.8 us back to back, 11.1 with it)
template <int TY, int TZ>
constexpr int conv_plane() {
    typedef Tile<TY, TZ> T;
    return TY == 8 ? T::SPAN / 16 * 16 + 16 : T::SPAN + 1;
}

template <int CIN, int MT, int NT>
__global__ void __launch_bounds__(256) k_conv_tile(const bf16 *__restrict__ in, const bf16 *__restrict__ w,
                                                   const float *__restrict__ bias, ConvGeom g, int relu,
                                                   bf16 *__restrict__ out, float *__restrict__ out_f32) {
    constexpr int TY = MT == 4 ? 8 : 4, TZ = MT == 1 ? 2 : 4;
    typedef Tile<TY, TZ> T;
    constexpr int GROUPS = CIN / 8, PLANE = conv_plane<TY, TZ>(), PITCH = T::PITCH;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    bf16x8 *lds = reinterpret_cast<bf16x8 *>(smem_raw);
    const T tile(g, blockIdx.x);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quad = lane >> 4;

    const int n0 = blockIdx.y * (16 * NT);
    const bf16 *wrow[NT];
#pragma unroll
    for (int j = 0; j < NT; j++) wrow[j] = w + (long long)(n0 + j * 16 + (lane & 15)) * g.kpad + quad * 8;
    // weights are read a stage ahead of their products (their latency is that
    // of the L2): all of them before the tile is staged for up to 16 channels,
    // else the next row of three taps
    constexpr int CHUNKS = CIN >= 32 ? 3 * (CIN / 32) : (27 * CIN + 31) / 32;
    bf16x8 wk[NT][CHUNKS];
#pragma unroll
    for (int q = 0; q < CHUNKS; q++)
#pragma unroll
        for (int j = 0; j < NT; j++) wk[j][q] = *reinterpret_cast<const bf16x8 *>(wrow[j] + q * 32);
    f32x4 b4[NT];
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) b4[j][r] = bias ? bias[n0 + j * 16 + quad * 4 + r] : 0.0f;

    // the halo tile; neighbouring threads take neighbouring channel groups
    {
        typedef typename T::template Stage<GROUPS> St;
        const St st;
        const int x = st.takes ? tile.column(g, st.hx) : -1, lane_row = tile.row(g, lane);
        const bf16 *from = in + (long long)max(x, 0) * CIN + st.cg * 8;
        bf16x8 *to = lds + st.cg * PLANE + st.l0 * PITCH + st.hx;
        constexpr int BATCH = St::PASSES < 12 ? St::PASSES : 12;  // loads in flight per thread
#pragma unroll
        for (int i0 = 0; i0 < St::PASSES; i0 += BATCH) {
            bf16x8 v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                if (i0 + u >= St::PASSES) break;
                const int r = __shfl(lane_row, st.line(i0 + u), 64);
                v[u] = r >= 0 && x >= 0 ? *reinterpret_cast<const bf16x8 *>(from + (long long)r * CIN) : zero8();
            }
#pragma unroll
            for (int u = 0; u < BATCH; u++) {
                if (i0 + u >= St::PASSES) break;
                if (st.stores(i0 + u)) to[(i0 + u) * St::AT_ONCE * PITCH] = v[u];
            }
        }
    }
    if (threadIdx.x < GROUPS) lds[threadIdx.x * PLANE + T::SPAN] = zero8();
    __syncthreads();

    int pos[MT];  // halo position of this lane's voxel of each group, for the first tap
    int vx[MT], vy[MT], vz[MT];
#pragma unroll
    for (int i = 0; i < MT; i++) {
        const int l = T::line(wave * MT + i, (lane >> 3) & 1);
        vx[i] = lane & 7;
        vy[i] = l % TY;
        vz[i] = l / TY;
        pos[i] = (vz[i] * T::HY + vy[i]) * PITCH + vx[i];
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if constexpr (CIN >= 32) {
        const bf16x8 *base = lds + quad * PLANE;
        // rows of three taps; a chunk of 32 channels of each tap in turn
#pragma unroll 1
        for (int row = 0; row < 9; row++) {
            bf16x8 a[NT][CHUNKS];
            const int next = row < 8 ? (row + 1) * CHUNKS * 32 : 0;
#pragma unroll
            for (int q = 0; q < CHUNKS; q++)
#pragma unroll
                for (int j = 0; j < NT; j++) {
                    a[j][q] = wk[j][q];
                    wk[j][q] = *reinterpret_cast<const bf16x8 *>(wrow[j] + next + q * 32);
                }
            const bf16x8 *at = base + (row / 3 * T::HY + row % 3) * PITCH;
#pragma unroll
            for (int q = 0; q < CHUNKS; q++) {
                const int dx = q / (CIN / 32), c = q % (CIN / 32);
                bf16x8 b[MT];
#pragma unroll
                for (int i = 0; i < MT; i++) b[i] = at[pos[i] + dx + c * 4 * PLANE];
#pragma unroll
                for (int i = 0; i < MT; i++)
#pragma unroll
                    for (int j = 0; j < NT; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][q], b[i], acc[i][j], 0, 0, 0);
            }
        }
    } else {
        // a 32-wide chunk spans 32 / CIN taps; this lane's 8 channels belong to
        // tap TPC q + sub of chunk q (tap 27 and beyond: the zero vector)
        constexpr int TPC = 32 / CIN;
        const int sub = quad * 8 / CIN;
        const bf16x8 *base = lds + (quad * 8 % CIN / 8) * PLANE;
#pragma unroll
        for (int q = 0; q < (27 + TPC - 1) / TPC; q++) {
            int shift = 0;
            bool pad = false;
#pragma unroll
            for (int u = 0; u < TPC; u++)
                if (sub == u) {
                    shift = q * TPC + u < 27 ? T::tap(q * TPC + u) : 0;
                    pad = q * TPC + u >= 27;
                }
            bf16x8 b[MT];
#pragma unroll
            for (int i = 0; i < MT; i++) b[i] = base[pad ? T::SPAN : pos[i] + shift];
#pragma unroll
            for (int i = 0; i < MT; i++)
#pragma unroll
                for (int j = 0; j < NT; j++)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wk[j][q], b[i], acc[i][j], 0, 0, 0);
        }
    }

    // a lane holds channels 4 quad .. 4 quad + 3 of voxel lane % 16 of each group
#pragma unroll
    for (int i = 0; i < MT; i++) {
        const int x = tile.x0 + vx[i], y = tile.y0 + vy[i], z = tile.z0 + vz[i];
        if (x >= g.W || y >= g.H || z >= g.D) continue;
        const long long v = (((long long)tile.nb * g.D + z) * g.H + y) * g.W + x;
#pragma unroll
        for (int j = 0; j < NT; j++) {
            const int co = n0 + j * 16 + quad * 4;
            f32x4 y4 = acc[i][j];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                y4[r] += b4[j][r];
                if (relu) y4[r] = fmaxf(y4[r], 0.0f);
            }
            if (out_f32) {
                *reinterpret_cast<f32x4 *>(out_f32 + v * g.cout + co) = y4;
            } else {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; r++) o[r] = (bf16)y4[r];
                *reinterpret_cast<bf16x4 *>(out + v * g.cout + co) = o;
            }
        }
    }
}

template <int CIN, int MT, int NT>
static hipError_t launch_tile(const bf16 *in, const bf16 *w, const float *bias, const ConvGeom &g, int relu, bf16 *out,
                              float *out_f32, hipStream_t s) {
    constexpr int TY = MT == 4 ? 8 : 4, TZ = MT == 1 ? 2 : 4;
    const dim3 grid((unsigned)tile_count(g, TY, TZ), g.cout / (16 * NT));
    const size_t lds = (size_t)conv_plane<TY, TZ>() * CIN * sizeof(bf16);
    hipLaunchKernelGGL((k_conv_tile<CIN, MT, NT>), grid, dim3(256), lds, s, in, w, bias, g, relu, out, out_f32);
    return hipGetLastError();
}

// Large tiles reuse each weight and each staged voxel most; a coarse level
// (8^3 voxels, 128 channels) then fills a handful of blocks, so tiles shrink
// until a launch has two blocks for each CU or they are smallest.
struct TileChoice {
    int mt, nt;  // of a wave: 16 mt voxels, 16 nt channels
    long long tiles, blocks;
};

static TileChoice tile_choice(const ConvGeom &g) {
    TileChoice c{g.cin <= 64 ? 4 : 2, g.cout % 32 == 0 ? 2 : 1, 0, 0};
    for (;;) {
        c.tiles = tile_count(g, c.mt == 4 ? 8 : 4, c.mt == 1 ? 2 : 4);
        c.blocks = c.tiles * (g.cout / (16 * c.nt));
        if (c.blocks >= 512 || (c.nt == 1 && c.mt == 1)) return c;
        if (c.nt > 1) c.nt = 1;
        else c.mt >>= 1;
    }
}

template <int CIN>
static hipError_t conv_tile(const bf16 *in, const bf16 *w, const float *bias, const ConvGeom &g, int relu, bf16 *out,
                            float *out_f32, hipStream_t s) {
    const TileChoice c = tile_choice(g);
    const int mt = c.mt, nt = c.nt;
    if (mt == 4) {
        if constexpr (CIN <= 64) {
            return nt == 2 ? launch_tile<CIN, 4, 2>(in, w, bias, g, relu, out, out_f32, s)
                           : launch_tile<CIN, 4, 1>(in, w, bias, g, relu, out, out_f32, s);
        }
    }
    if (mt == 2)
        return nt == 2 ? launch_tile<CIN, 2, 2>(in, w, bias, g, relu, out, out_f32, s)
                       : launch_tile<CIN, 2, 1>(in, w, bias, g, relu, out, out_f32, s);
    return launch_tile<CIN, 1, 1>(in, w, bias, g, relu, out, out_f32, s);
}

bool nn_conv_tile_takes(const void *in, const void *w, const ConvGeom &g, const void *out, const void *out_f32) {
    auto off = [](const void *p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) != 0; };
    if (off(in, 16) || off(w, 16) || off(out, 8) || off(out_f32, 16)) return false;
    if (g.cin != 8 && g.cin != 16 && g.cin != 32 && g.cin != 64 && g.cin != 128) return false;
    // A tile is computed whole.  In a volume narrower than it, or many small
    // ones, that is work without a voxel, which runs beside the others' as long
    // as the blocks are few; beyond that it takes its time, and gathering from
    // memory costs less (1 x 256 x 256 x 1 voxels of 64 channels: 68 us gathered,
    // 248 in tiles 8 times as large; 128 channels on 2048 single voxels 21.6 and
    // 969).  The limits lie where the two meet, over 2500 random shapes.
    const TileChoice c = tile_choice(g);
    if (c.tiles >= (1LL << 24)) return false;  // a grid holds fewer than 2^32 threads
    const long long padded = 64LL * c.mt * c.tiles, voxels = (long long)g.n * g.D * g.H * g.W;
    const double limit = g.cin == 32 ? 2.5 : (g.cin == 8 || g.cin == 64 ? 2.0 : 1.75);
    return c.blocks < (g.cin >= 64 ? 256 : 512) || (double)padded <= limit * (double)voxels;
}

hipError_t nn_conv_tile(const void *in, const void *w, const float *bias, const ConvGeom &g, int relu, void *out,
                        float *out_f32, hipStream_t s) {
    const bf16 *i = (const bf16 *)in, *ww = (const bf16 *)w;
    bf16 *o = (bf16 *)out;
    switch (g.cin) {
        case 8: return conv_tile<8>(i, ww, bias, g, relu, o, out_f32, s);
        case 16: return conv_tile<16>(i, ww, bias, g, relu, o, out_f32, s);
        case 32: return conv_tile<32>(i, ww, bias, g, relu, o, out_f32, s);
        case 64: return conv_tile<64>(i, ww, bias, g, relu, o, out_f32, s);
        default: return conv_tile<128>(i, ww, bias, g, relu, o, out_f32, s);
    }
}

}  // namespace mrt
