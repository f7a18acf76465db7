// Weight and bias gradients of the learned warm start's 3x3x3 convolutions on gfx950's
// v_mfma_f32_16x16x32_bf16: dW[tap][cout][cin] = sum over voxels of G[v][cout] X[v + d][cin],
// a matrix product with M = output channels, N = input channels of one tap and K = voxels.
//
// What bounds it: the 27 taps share both operands, so staging them once per block (instead of
// once per tap) leaves the LDS reads of the fragments, about one 8-byte read per lane and
// MFMA.  A block owns a 256-voxel tile of the x-y plane and marches up in z.  The X planes
// z-1, z, z+1 (one-voxel halo in x and y, 16 input channels) sit in a ring of four, the
// gradient planes in two buffers; the next planes are loaded into registers during the
// products and stored after them, one barrier per plane.  Wave w takes the taps of
// dz = w % 3 - 1 (9 accumulator sets of every 16 output channels) over half of the tile's
// voxels (w / 3).  Operands lie in LDS as in memory (channel fastest) and
// ds_read_b64_tr_b16 hands every lane four voxels of one channel, so a tap is only an
// address offset.  K runs over the voxels in the order both fragments read them.
// The bias gradient is the same product with a column of ones.
//
// At 128 x 128 x 60 the ten layers take 0.28 ms and their partial sums 0.05 ms; a block per tap,
// staging both operands again (transposed with 2-byte LDS stores), took 3.04 ms, its sums and the
// bias sums 1.07 ms (loss and gradient 5.21 -> 1.43 ms).
#pragma once

#include "fx_internal.h"
#include "fx_unet_internal.h"

namespace fx {

namespace {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));
typedef int i2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));

constexpr int kWgTile = 256;            // voxels of a tile
constexpr int kWgThreads = 384;         // 3 dz x 2 halves of the tile
constexpr int kWgBlocks = 512;          // blocks aimed at: two per compute unit

// Four voxels of this lane's channel: lanes 4 r .. 4 r + 3 of each 16 point at the 16
// channels of voxel r, and lane i receives channel i of voxels 0..3.
__device__ __forceinline__ s4 tr_read(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4 *)p);
}
__device__ __forceinline__ bf8 frag(const unsigned char *lo, const unsigned char *hi) {
    const s4 a = tr_read(lo), b = tr_read(hi);
    return __builtin_bit_cast(bf8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Work of a launch: items (tile, z-chunk), shared out over gridDim.x blocks; blockIdx.y
// is the 16-channel slice of X, blockIdx.z the slice of 16 MT output channels.
struct WgGeom {
    int nx, ny, nz, ntx, nty, zl, items;
};

template <int MT, int TX, int XL>
struct WgShape {
    static constexpr int TY = kWgTile / TX, HX = TX + 2, HY = TY + 2, NV = HX * HY;
    static constexpr int XB = NV * 32;                      // one X plane
    static constexpr int GB = MT * kWgTile * 32;            // one gradient plane
    static constexpr int LDS = 4 * XB + 2 * GB;
    static constexpr int XP = XL == 4 ? NV : 2 * NV;        // pieces (8 or 16 bytes)
    static constexpr int GP = 2 * MT * kWgTile;
    static constexpr int PX = (XP + kWgThreads - 1) / kWgThreads, PG = (GP + kWgThreads - 1) / kWgThreads;
    static_assert(LDS >= 28 * 64 * 16, "the halves of the tile are added through LDS");
};

template <int MT, int TX, int XL>
__global__ __launch_bounds__(kWgThreads) void k_wgrad(const bf16_t *__restrict__ X, int ldx,
                                                      const bf16_t *__restrict__ G, WgGeom g, int cin,
                                                      int cout, float *__restrict__ part) {
    using S = WgShape<MT, TX, XL>;
    extern __shared__ __attribute__((aligned(16))) unsigned char wg_lds[];
    unsigned char *xl = wg_lds, *gl = wg_lds + 4 * S::XB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int dzi = wave % 3, hf = wave / 3;
    const int col = lane & 15, kq = lane >> 4;
    const int c0 = blockIdx.y * 16, o0 = blockIdx.z * 16 * MT;
    const bool want_bias = dzi == 1 && c0 == 0;

    f4 acc[9][MT], accb[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        accb[m] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t][m] = f4{0.f, 0.f, 0.f, 0.f};
    }
    const bf8 ones = __builtin_bit_cast(bf8, s8{0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80});
    if (XL == 4)                                            // channels 4..15 stay zero
        for (int u = tid; u < 4 * S::XB / 16; u += kWgThreads) *(i4 *)(xl + 16 * u) = i4{0, 0, 0, 0};

    for (int item = blockIdx.x; item < g.items; item += gridDim.x) {
        const int tx = item % g.ntx, q = item / g.ntx, ty = q % g.nty, zc = q / g.nty;
        const int x0 = tx * TX, y0 = ty * S::TY;
        const int z0 = zc * g.zl, z1 = min(z0 + g.zl, g.nz);
        // source offsets of this thread's pieces inside a plane (-1: zero)
        int xo[S::PX], go[S::PG];
#pragma unroll
        for (int p = 0; p < S::PX; ++p) {
            const int u = tid + p * kWgThreads;
            const int v = XL == 4 ? u : u >> 1, half = XL == 4 ? 0 : u & 1;
            const int hx = v % S::HX, hy = v / S::HX;
            int x = x0 + hx - 1, y = y0 + hy - 1;
            const bool in = u < S::XP && x <= g.nx && y <= g.ny;    // the far halo wraps
            x = x < 0 ? x + g.nx : (x >= g.nx ? x - g.nx : x);
            y = y < 0 ? y + g.ny : (y >= g.ny ? y - g.ny : y);
            xo[p] = in ? (y * g.nx + x) * ldx + (XL == 4 ? 0 : c0 + half * 8) : -1;
        }
#pragma unroll
        for (int p = 0; p < S::PG; ++p) {
            const int u = tid + p * kWgThreads;
            const int v = u / (2 * MT), c8 = u % (2 * MT);
            const int x = x0 + (v & (TX - 1)), y = y0 + v / TX;
            go[p] = u < S::GP && x < g.nx && y < g.ny ? (y * g.nx + x) * cout + o0 + c8 * 8 : -1;
        }
        const size_t xplane = (size_t)g.nx * g.ny * ldx, gplane = (size_t)g.nx * g.ny * cout;
        i4 xr[S::PX], gr[S::PG];
        auto load_x = [&](int z) {
            const bool in = z >= 0 && z < g.nz;
            const bf16_t *src = X + (in ? z : 0) * xplane;
#pragma unroll
            for (int p = 0; p < S::PX; ++p) {
                xr[p] = i4{0, 0, 0, 0};
                if (in && xo[p] >= 0) {
                    if (XL == 4) {
                        const i2 h = *(const i2 *)(src + xo[p]);
                        xr[p][0] = h[0];
                        xr[p][1] = h[1];
                    } else {
                        xr[p] = *(const i4 *)(src + xo[p]);
                    }
                }
            }
        };
        auto store_x = [&](int z) {
            unsigned char *dst = xl + (z & 3) * S::XB;
#pragma unroll
            for (int p = 0; p < S::PX; ++p) {
                const int u = tid + p * kWgThreads;
                if (u >= S::XP) continue;
                if (XL == 4) *(i2 *)(dst + u * 32) = i2{xr[p][0], xr[p][1]};
                else *(i4 *)(dst + u * 16) = xr[p];
            }
        };
        auto load_g = [&](int z) {
            const bf16_t *src = G + z * gplane;
#pragma unroll
            for (int p = 0; p < S::PG; ++p) gr[p] = go[p] >= 0 ? *(const i4 *)(src + go[p]) : i4{0, 0, 0, 0};
        };
        auto store_g = [&](int z) {
            unsigned char *dst = gl + (z & 1) * S::GB;
#pragma unroll
            for (int p = 0; p < S::PG; ++p) {
                const int u = tid + p * kWgThreads;
                if (u >= S::GP) continue;
                const int v = u / (2 * MT), c8 = u % (2 * MT);
                *(i4 *)(dst + (c8 >> 1) * (kWgTile * 32) + v * 32 + (c8 & 1) * 16) = gr[p];
            }
        };
        __syncthreads();                                    // the previous item's last plane read
        for (int z = z0 - 1; z <= z0 + 1; ++z) {
            load_x(z);
            store_x(z);
        }
        load_g(z0);
        store_g(z0);
        __syncthreads();
        for (int z = z0; z < z1; ++z) {
            const bool more = z + 1 < z1;
            if (more) {
                load_x(z + 2);
                load_g(z + 1);
            }
            const unsigned char *xp = xl + ((z + dzi - 1) & 3) * S::XB;
            const unsigned char *gp = gl + (z & 1) * S::GB;
#pragma unroll 1
            for (int pos = 4 * hf; pos < 4 * hf + 4; ++pos) {
                const int v0 = pos * 32 + 4 * kq + (col >> 2), v1 = v0 + 16, c8 = (col & 3) * 8;
                bf8 a[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    a[m] = frag(gp + m * (kWgTile * 32) + v0 * 32 + c8, gp + m * (kWgTile * 32) + v1 * 32 + c8);
                const unsigned char *b0 = xp + ((v0 / TX) * S::HX + (v0 & (TX - 1))) * 32 + c8;
                const unsigned char *b1 = xp + ((v1 / TX) * S::HX + (v1 & (TX - 1))) * 32 + c8;
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const int o = ((t / 3) * S::HX + t % 3) * 32;
                    const bf8 b = frag(b0 + o, b1 + o);
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[t][m], 0, 0, 0);
                }
                if (want_bias)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, accb[m], 0, 0, 0);
            }
            if (more) {
                store_x(z + 2);
                store_g(z + 1);
            }
            __syncthreads();
        }
    }
    // the two halves of the tile, then this block's partial sum: [27][cout][cin] and [cout]
    float *out = part + (size_t)blockIdx.x * (27 * cout * cin + cout);
    f4 *red = (f4 *)wg_lds;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        __syncthreads();
        if (hf == 1) {
#pragma unroll
            for (int t = 0; t < 9; ++t) red[(dzi * 9 + t) * 64 + lane] = acc[t][m];
            if (dzi == 1) red[27 * 64 + lane] = accb[m];
        }
        __syncthreads();
        if (hf == 0) {
            const int co = o0 + m * 16 + 4 * kq;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const f4 s = acc[t][m] + red[(dzi * 9 + t) * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) out[(size_t)((dzi * 9 + t) * cout + co + r) * cin + c0 + col] = s[r];
            }
            if (want_bias && col == 0) {
                const f4 s = accb[m] + red[27 * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) out[27 * cout * cin + co + r] = s[r];
            }
        }
    }
}

// dst[i] = sum over p of part[p][i]: 16 threads per value, each its share of p in order,
// their sums added in order (deterministic).  Bound by reading the partials once: the loads
// of a thread's share are independent (a serial sum per value took 22 us a layer).
__global__ __launch_bounds__(1024) void k_wsum(const float *__restrict__ part, int nparts, int m,
                                               float *__restrict__ dst) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, s = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    float v = 0.f;
    if (i < m) {
#pragma unroll 8
        for (int p = s; p < nparts; p += 16) v += part[(size_t)p * m + i];
    }
    red[s][lane] = v;
    __syncthreads();
    if (s == 0 && i < m) {
        float t = red[0][lane];
#pragma unroll
        for (int q = 1; q < 16; ++q) t += red[q][lane];
        dst[i] = t;
    }
}

// Tile width: of 32, 16 and 8 the one that covers the plane with the fewest voxels.
int wg_tx(int nx, int ny) {
    int best = 32;
    long long cost = 0;
    for (int tx = 32; tx >= 8; tx /= 2) {
        const int ty = kWgTile / tx;
        const long long c = (long long)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty);
        if (tx == 32 || c < cost) { best = tx; cost = c; }
    }
    return best;
}

// z-chunks so that the tiles, chunks and channel slices fill the chip about once;
// chunks of at least three planes (each loads two more).
WgGeom wg_geom(int cin, int cout, int nx, int ny, int nz, int *nparts) {
    const int tx = wg_tx(nx, ny), ty = kWgTile / tx;
    WgGeom g;
    g.nx = nx; g.ny = ny; g.nz = nz;
    g.ntx = (nx + tx - 1) / tx;
    g.nty = (ny + ty - 1) / ty;
    const int slices = (cin / 16) * (cout > 32 ? cout / 32 : 1);
    const int tiles = g.ntx * g.nty, want = (kWgBlocks + slices - 1) / slices;
    int zc = want / tiles;
    zc = zc > nz / 3 ? nz / 3 : zc;
    zc = zc < 1 ? 1 : zc;
    g.zl = (nz + zc - 1) / zc;
    g.items = tiles * ((nz + g.zl - 1) / g.zl);
    *nparts = g.items < want ? g.items : want;
    return g;
}

template <int MT, int TX, int XL>
void wg_go(const bf16_t *X, int ldx, const bf16_t *G, const WgGeom &g, int cin, int cout, int nparts, float *part,
           hipStream_t st) {
    hipLaunchKernelGGL((k_wgrad<MT, TX, XL>), dim3(nparts, cin / 16, cout / (16 * MT)), dim3(kWgThreads),
                       (WgShape<MT, TX, XL>::LDS), st, X, ldx, G, g, cin, cout, part);
}

template <int MT, int XL>
void wg_tile(int tx, const bf16_t *X, int ldx, const bf16_t *G, const WgGeom &g, int cin, int cout, int nparts,
             float *part, hipStream_t st) {
    if (tx == 32) wg_go<MT, 32, XL>(X, ldx, G, g, cin, cout, nparts, part, st);
    else if (tx == 16) wg_go<MT, 16, XL>(X, ldx, G, g, cin, cout, nparts, part, st);
    else wg_go<MT, 8, XL>(X, ldx, G, g, cin, cout, nparts, part, st);
}

}  // namespace

// dst[i] = sum over p < nparts of part[p][i], i < m, in a fixed order.
void part_sum(const float *part, int nparts, int m, float *dst, hipStream_t st) {
    hipLaunchKernelGGL(k_wsum, dim3((m + 63) / 64), dim3(1024), 0, st, part, nparts, m, dst);
}

// Weight gradient W[27][cout][cin] and, after it, bias gradient [cout] of a convolution into
// dst, from its input X (leading dimension ldx; xl = 4: four channels present, the rest of cin
// zero) and its BF16 output gradient G ([n][cout]); part: wgrad_part_floats(...) floats.
size_t wgrad_part_floats(int cin, int cout, int nx, int ny, int nz) {
    int nparts;
    (void)wg_geom(cin, cout, nx, ny, nz, &nparts);
    return (size_t)nparts * (27 * cin * cout + cout);
}

void wgrad(int cin, int cout, int xl, const bf16_t *X, int ldx, const bf16_t *G, int nx, int ny, int nz, float *part,
           float *dst, hipStream_t st) {
    int nparts;
    const WgGeom g = wg_geom(cin, cout, nx, ny, nz, &nparts);
    const int tx = wg_tx(nx, ny);
    if (xl == 4) wg_tile<1, 4>(tx, X, ldx, G, g, cin, cout, nparts, part, st);
    else if (cout == 16) wg_tile<1, 16>(tx, X, ldx, G, g, cin, cout, nparts, part, st);
    else wg_tile<2, 16>(tx, X, ldx, G, g, cin, cout, nparts, part, st);
    part_sum(part, nparts, 27 * cin * cout + cout, dst, st);
}

}  // namespace fx
