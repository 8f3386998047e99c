// Implicit-GEMM 3x3 convolution in fp32 on the bf16 matrix unit (f32x3.h), gfx950, NHWC: forward and data gradient of every
// launch whose tiles are consecutive pixels or whole patches, the contraction split over workgroups where conv_igemm.hip says so.  Views, tiles, halos and
// epilogue as in conv_igemm.hip; reference rows likewise.
//
// Workgroup: WM x WN waves, each 64 pixels x 16 NJ channels, in chunks of 32 channels.  LDS holds the chunk's halo and one
// tap's weights as three planes of bf16 parts, 64-byte rows whose 16-byte segment s lies at s ^ ((row >> 1) & 3)
// (conflict-free for the fragment reads of v_mfma_f32_16x16x32_bf16); weights in two buffers, a barrier per tap.
// Every value is split once per workgroup, on its way from a register to LDS: the weights of tap t + 1 in the middle of tap t,
// the next chunk's halo, requested before the last tap, at the chunk's end.  256-pixel tiles: eight waves, one workgroup per
// CU; 128-pixel tiles x 64 channels: four waves, two per CU.  Bound by MFMA issue at the clock that random operands allow:
// 128 -> 256 at 56x56, batch 100, 750 us = 247 TFLOP/s of fp32 products, 1.48 PFLOP/s of bf16 ones.  (The tap loop is not
// unrolled: the addresses of nine taps took ninety registers.)
#include "conv_tile.h"
#include "f32x3.h"

namespace vgg {

template <int WM, int WN, int NJ, int SA>
__global__ __launch_bounds__(WM *WN * 64, 2) void conv3x3_igemm_f32x3_kernel(ConvArgs p)
{
    typedef float T;
    constexpr int NT = WM * WN * 64, NI = 4, BM = WM * 64, BN = WN * NJ * 16, KC = 32, TAPS = 9;
    constexpr int XPLANE = SA * 64, WPLANE = BN * 64;
    constexpr int NX = SA * 8 / NT, NWT = BN * 8 / NT;       // 16-byte segments (four channels) per thread: halo, a tap's weights
    static_assert(SA * 8 % NT == 0 && BN * 8 % NT == 0, "whole segments per thread");
    extern __shared__ __align__(16) char smem[];
    int *pix = reinterpret_cast<int *>(smem);                // [SA] halo row -> input pixel or -1
    char *Xs = smem + SA * 4;                                // [3][SA][64]
    char *Ws = Xs + 3 * XPLANE;                              // [2][3][BN][64]
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv % WM, wn = wv / WM;
    const int q = lane & 15, g = lane >> 4;
    // (XCD-aware numbering: each XCD, with its own L2, works through one contiguous range of tiles)
    const int nblk = gridDim.x, xcd = blockIdx.x & 7;
    const int bid = xcd * (nblk >> 3) + min(xcd, nblk & 7) + (blockIdx.x >> 3);
    // (split contraction: the ksplit workgroups of a tile are neighbours, each with p.kchunks sixteen-channel chunks)
    const int split = bid % p.ksplit, tile = bid / p.ksplit;
    const int tile_n = tile % p.tiles_n, tile_m = tile / p.tiles_n;
    const int c_first = split * p.kchunks * 16, cspan = min(p.kchunks * 16, p.CinP - c_first);   // this workgroup's channels
    const int n0 = tile_n * BN;
    const TileOrigin org = tile_origin(p.g, tile_m);
    const int pitch = p.g.pitch;
    const size_t xrow = (size_t)p.CinP * sizeof(T);
    const int nchunks = (cspan + KC - 1) / KC;               // (the last one may be half: 16 channels)

    const int srow = tid >> 3, sseg = tid & 7;               // this thread's row (of every NT / 8) and segment of what it stages
    // four channels = 8 bytes of a plane's row
    auto lds_at = [&](int row) __attribute__((always_inline)) {
        return row * 64 + ((((sseg >> 1) ^ (row >> 1)) & 3) << 4) + (sseg & 1) * 8;
    };
    // (32-bit offsets from a scalar base that moves with tap and chunk: conv_plan keeps Cout x CinP x 4 within them)
    u32x4 wr[NWT], xr[NX];
    unsigned wvoff[NWT];
#pragma unroll
    for (int k = 0; k < NWT; ++k) wvoff[k] = (unsigned)min(n0 + srow + k * (NT / 8), p.Cout - 1) * (unsigned)xrow;   // columns past Cout are never stored
    auto load_w = [&](int t, int c) __attribute__((always_inline)) {
        const char *base = p.w + (size_t)t * p.Cout * xrow + (size_t)(c_first + c * KC) * 4;
        const unsigned col = c * KC + sseg * 4 < cspan ? sseg * 16 : 0;
#pragma unroll
        for (int k = 0; k < NWT; ++k) wr[k] = *reinterpret_cast<const u32x4 *>(base + (wvoff[k] + col));
    };
    auto store_w = [&](int c, int buf) __attribute__((always_inline)) {
        const bool in = c * KC + sseg * 4 < cspan;
#pragma unroll
        for (int k = 0; k < NWT; ++k) {
            const Parts4 s = split_parts(in ? wr[k] : u32x4{0u, 0u, 0u, 0u});
            char *dst = Ws + buf * 3 * WPLANE + lds_at(srow + k * (NT / 8));
#pragma unroll
            for (int e = 0; e < 3; ++e) *reinterpret_cast<f32x3_u32x2 *>(dst + e * WPLANE) = s.p[e];
        }
    };
    load_w(0, 0);
    for (int i = tid; i < SA; i += NT) pix[i] = i < p.g.S ? halo_pixel(p.g, org, i) : -1;
    __syncthreads();
    typedef const __attribute__((address_space(1))) u32x4 *gvec_t;
    auto load_x = [&](int c) __attribute__((always_inline)) {
        const bool in = c * KC + sseg * 4 < cspan;
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int px = pix[srow + k * (NT / 8)];
            const gvec_t src = px < 0 || !in ? (gvec_t)kZeroRow : (gvec_t)(p.x + (size_t)px * xrow + (size_t)(c_first + c * KC + sseg * 4) * 4);
            xr[k] = *src;
        }
    };
    auto store_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const Parts4 s = split_parts(xr[k]);
            char *dst = Xs + lds_at(srow + k * (NT / 8));
#pragma unroll
            for (int e = 0; e < 3; ++e) *reinterpret_cast<f32x3_u32x2 *>(dst + e * XPLANE) = s.p[e];
        }
    };
    load_x(0);
    int hrow[NI];   // halo row of tap (0,0) of this lane's pixels: lane l finds the wave's tile row l's
    {
        int m, h;
        tile_row(p.g, org, wm * 64 + lane, m, h);
#pragma unroll
        for (int i = 0; i < NI; ++i) hrow[i] = __shfl(h, i * 16 + q, kWave);
    }
    // Accumulators: lane 16 g + q holds channels 4 g .. 4 g + 3 of pixel q; they start at the bias.
    f32x4v hi[NI][NJ], lo[NI][NJ];
    {
        const int c0 = n0 + wn * NJ * 16 + g * 4;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            hi[0][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
            if (p.bias && !p.part)   // (split contraction: the finishing kernel adds the bias)
#pragma unroll
                for (int e = 0; e < 4; ++e) hi[0][j][e] = kPartsScale * p.bias[min(c0 + j * 16 + e, p.Cout - 1)];
        }
    }
    store_w(0, 0);
    load_w(1, 0);
    store_x();
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            hi[i][j] = hi[0][j];
            lo[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
        }
    __syncthreads();

    const int wlane = wn * NJ * 16 * 64 + q * 64 + (((g ^ (q >> 1)) & 3) << 4);   // this lane's weight fragment j = 0 inside a plane
    auto frag = [](const char *at) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(at)); };
    // One tap: its 24 NJ MFMAs; half-way the next tap's weights, requested a tap ago, go to the other buffer (chunk c1) and
    // those of the tap after it (tap t2 of chunk c2) are requested.  (Past the end: the last chunk again, never read.)
    auto tap = [&](int toff, int buf, int c1, int t2, int c2) __attribute__((always_inline)) {
        const char *Wt = Ws + buf * 3 * WPLANE + wlane;
        bf16x8 w[3][NJ], x[2][3];
        auto read_x = [&](int i) __attribute__((always_inline)) {
            const int row = hrow[i] + toff;
            const char *at = Xs + row * 64 + (((g ^ (row >> 1)) & 3) << 4);
#pragma unroll
            for (int e = 0; e < 3; ++e) x[i & 1][e] = frag(at + e * XPLANE);
        };
        read_x(0);
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
            for (int j = 0; j < NJ; ++j) w[e][j] = frag(Wt + e * WPLANE + j * 16 * 64);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < NI) read_x(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            auto terms = [&](f32x4v(&acc)[NJ], int we, int xe) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[we][j], x[i & 1][xe], acc[j], 0, 0, 0);
            };
            terms(hi[i], 0, 0); terms(lo[i], 0, 1); terms(lo[i], 1, 0);
            terms(lo[i], 1, 1); terms(lo[i], 0, 2); terms(lo[i], 2, 0);
            if (i == 1) {
                store_w(c1, buf ^ 1);
                load_w(t2, c2);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (not the loads in flight)
    };
    int buf = 0;
    for (int c = 0; c < nchunks; ++c) {
        const int cn = min(c + 1, nchunks - 1);
        int toff = 0, kw = 0;
#pragma nounroll
        for (int t = 0; t < TAPS - 1; ++t) {
            const bool wrap = t == TAPS - 2;
            tap(toff, buf, c, wrap ? 0 : t + 2, wrap ? cn : c);
            buf ^= 1;
            if (++kw == 3) { kw = 0; toff += pitch - 2; }
            else ++toff;
        }
        load_x(cn);
        tap(toff, buf, cn, 1, cn);
        buf ^= 1;
        if (c + 1 < nchunks) {
            store_x();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) hi[i][j][e] = join_parts(hi[i][j][e], lo[i][j][e]);
    if (p.part) {   // raw sums to the partial buffer of this range (Cout is a multiple of 4 then)
        float *part = p.part + (size_t)split * p.g.M * p.Cout;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int m = tile_pixel(p.g, org, wm * 64 + i * 16 + q);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int col = n0 + wn * NJ * 16 + j * 16 + g * 4;
                if (m >= 0 && col < p.Cout) *reinterpret_cast<f32x4v *>(part + (size_t)m * p.Cout + col) = hi[i][j];
            }
        }
        return;
    }
    conv_epilogue_impl<T, BM, BN, WM, WN>(
        [&](int i, int j0, char *epi, float low) __attribute__((always_inline)) {
            // (fp32: a pass is 32 columns; pixel block i of 32 rows = 16-pixel blocks 2 i, 2 i + 1)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const f32x4v &v = hi[2 * i + h][2 * j0 + j];
                    store4(reinterpret_cast<T *>(epi + (h * 16 + q) * kEpiRow) + j * 16 + g * 4, fmaxf(v[0], low), fmaxf(v[1], low),
                           fmaxf(v[2], low), fmaxf(v[3], low));
                }
        },
        [&](auto fn) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) fn(wm * 64 + i * 16 + q, j * 16 + g * 4 + e, hi[i][j][e]);
        },
        p, org, smem, n0);
}

template <int WM, int WN, int NJ, int SA>
static int launch(const ConvArgs &a0, const TileGeom &g, hipStream_t stream)
{
    constexpr int BN = WN * NJ * 16;
    ConvArgs a = a0;
    a.g = g;
    a.tiles_n = (a.Cout + BN - 1) / BN;
    a.rowsA = SA;
    size_t lds = (size_t)SA * 4 + (size_t)3 * SA * 64 + (size_t)2 * 3 * BN * 64;
    if (lds < (size_t)WM * WN * kEpiBytes) lds = (size_t)WM * WN * kEpiBytes;
    auto kern = conv3x3_igemm_f32x3_kernel<WM, WN, NJ, SA>;
    if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.g.ntiles * a.tiles_n * a.ksplit)), dim3(WM * WN * 64), lds, stream, a);
    return launch_status();
}

int launch_conv_f32x3(const ConvArgs &a, const TileGeom &g, bool narrow, hipStream_t stream)
{
    if (g.rows == 128) return g.S <= kDmaHaloRowsHalf ? launch<2, 2, 2, kDmaHaloRowsHalf>(a, g, stream) : launch<2, 2, 2, kF32x3HaloRowsHalfBig>(a, g, stream);
    if (g.S <= kDmaHaloRows) return narrow ? launch<4, 2, 2, kDmaHaloRows>(a, g, stream) : launch<4, 2, 4, kDmaHaloRows>(a, g, stream);
    return narrow ? launch<4, 2, 2, kDmaHaloRowsBig>(a, g, stream) : launch<4, 2, 4, kDmaHaloRowsBig>(a, g, stream);
}

}  // namespace vgg
