// Weight gradient of the 3x3 convolution in fp32 on the bf16 matrix unit (f32x3.h), gfx950, NHWC; views and reference rows as
// in conv_wgrad.hip, for launches whose tiles are patches.
//
// Workgroup, one per CU: eight waves, a 64(co) x 32(ci) block of all nine taps and a range of patches.  Wave = (ci half) x
// (co half) x (taps 0-4 | taps 5-8); each step of a tap multiplies two 16-row co fragments with one 16-column x fragment.
// (64 input channels and four co fragments per wave read the LDS less often but need 160 registers of accumulators: 140
// spilled.)  A patch is 4 rows of 16 pixels, of which the first 14 or 16 are its own, the others' g being zero, or 8 x 8; an
// MFMA step contracts 32 pixels, two rows or four.  Every value is split into three bf16 parts on its way to LDS:
//   g: a thread loads the eight pixels of a run of one channel, so that they leave transposed: [co][64 pixels], 128-byte rows
//      whose 16-byte segment s lies at s ^ ((co >> 1) & 7), one 16-byte read per fragment;
//   x: the halo (6 x 18 or 10 x 10) as it lies, [pixel][32 channels], since a tap shifts the pixels: transpose reads, the 32-byte half c of
//      row r at c ^ (r >> 3) & 1, which keeps the eight rows of half a wave on distinct banks.
// Two buffers and one barrier per patch: a wave splits and stores the next patch half-way through its own.  64 -> 128 at 50x66,
// batch 10: 69 -> 44 us (the fp32 MFMAs on 4 x 14 patches, 512 workgroups), 512 -> 512 at 28x28, batch 10, 298 -> 213.  What
// bounds it is not known; no unit is full.  On the first of these layers the matrix pipes are busy 0.31 of the time, vector instructions
// (3.6 beside each MFMA) take half of a SIMD's issue cycles, the LDS is active 0.23; a wave waits to issue 0.37 of its time, for
// counters and barriers 0.19.  Four tenths fewer LDS reads (the taps of a halo row shifted out of registers) and splitting at
// different times in a SIMD's two waves changed nothing (1.00 of the time over 27 and 32 shapes).  (A zero of g beside an infinite x makes
// a partial sum NaN here: the pass that adds them forms it again from the patches' own pixels.)
#include "f32x3.h"

namespace vgg {

namespace {

constexpr int kHalo = 6 * 18;
constexpr int kGPlane = 64 * 128, kXPlane = kHalo * 64;
constexpr int kBuf = 3 * (kGPlane + kXPlane);

typedef float f32x4w __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int x_half(int row, int c) { return ((c ^ (row >> 3)) & 1) << 5; }

struct WgradF32x3Args {
    const float *x, *g;
    float *part, *dbpart;   // [splits][9][Cout][CinP]; [splits][Cout] or null
    int N, H, W, CinP, Cout, tw;
    int tiles_co, tiles_ci, tiles_w, tiles_hw, ntiles, tiles_per_split;
    FastDiv dTilesW, dTilesHW;
};

template <int PW, int T0, int NT>
__device__ __forceinline__ void body(const WgradF32x3Args &p, char *smem, int tco, int tci, int split)
{
    constexpr int NC = 2, NX = 2, PH = 64 / PW, HP = PW + 2, HALO = (PH + 2) * HP, RPS = 32 / PW;   // RPS: patch rows of an MFMA step
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, G = lane >> 4, chalf = (wv >> 1) & 1, half = wv & 1;
    const int co0 = tco * 64, ci0 = tci * 32;

    f32x4w hi[NC][NT], lo[NC][NT];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t) hi[c][t] = lo[c][t] = f32x4w{0.f, 0.f, 0.f, 0.f};
    float gsum = 0.f;

    const int t_begin = split * p.tiles_per_split, t_end = min(t_begin + p.tiles_per_split, p.ntiles);
    // g: the wv-th run of eight pixels of the patch, channel `lane`; x: four channels of halo rows tid / 8 + 64 k
    const float *const gcol = p.g + min(co0 + lane, p.Cout - 1);
    const int xseg = tid & 7;
    const bool xin = ci0 + xseg * 4 < p.CinP;
    const float *const xcol = p.x + (xin ? ci0 + xseg * 4 : 0);
    struct Staged { unsigned g[8]; f32x3_u32x4 x[NX]; int h0, w0; };
    const int grow0 = PW == 16 ? wv >> 1 : wv, gcol0 = PW == 16 ? 8 * (wv & 1) : 0;
    auto request = [&](int tile, Staged &v) __attribute__((always_inline)) {   // (outside the image: clamped, replaced by zeros below)
        const int n = fast_div(tile, p.dTilesHW), rem = tile - n * p.tiles_hw, ty = fast_div(rem, p.dTilesW);
        v.h0 = ty * PH;
        v.w0 = (rem - ty * p.tiles_w) * p.tw;
        const size_t grow = ((size_t)n * p.H + min(v.h0 + grow0, p.H - 1)) * p.W;
#pragma unroll
        for (int j = 0; j < 8; ++j) v.g[j] = __float_as_uint(gcol[(grow + min(v.w0 + gcol0 + j, p.W - 1)) * p.Cout]);
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int row = min((tid >> 3) + 64 * k, HALO - 1), hy = row / HP, hx = row - hy * HP;
            const int h = min(max(v.h0 - 1 + hy, 0), p.H - 1), w = min(max(v.w0 - 1 + hx, 0), p.W - 1);
            v.x[k] = *reinterpret_cast<const f32x3_u32x4 *>(xcol + (((size_t)n * p.H + h) * p.W + w) * p.CinP);
        }
    };
    auto stage = [&](const Staged &v, char *buf) __attribute__((always_inline)) {
        f32x3_u32x4 a, b;
        const int own = v.h0 + grow0 < p.H ? min(p.tw, p.W - v.w0) - gcol0 : 0;   // pixels of the run that are the patch's
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a[j] = j < own ? v.g[j] : 0u;
            b[j] = j + 4 < own ? v.g[j + 4] : 0u;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) gsum += __uint_as_float(a[j]) + __uint_as_float(b[j]);
        {
            const Parts4 s = split_parts(a), t = split_parts(b);
            char *dst = buf + lane * 128 + ((wv ^ ((lane >> 1) & 7)) << 4);
#pragma unroll
            for (int e = 0; e < 3; ++e)
                *reinterpret_cast<f32x3_u32x4 *>(dst + e * kGPlane) = f32x3_u32x4{s.p[e][0], s.p[e][1], t.p[e][0], t.p[e][1]};
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int row = (tid >> 3) + 64 * k, hy = row / HP, hx = row - hy * HP;
            const int h = v.h0 - 1 + hy, w = v.w0 - 1 + hx;
            const bool in = xin && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
            const Parts4 s = split_parts(in ? v.x[k] : f32x3_u32x4{0u, 0u, 0u, 0u});
            char *dst = buf + 3 * kGPlane + row * 64 + x_half(row, xseg >> 2) + (xseg & 3) * 8;
            if (row < HALO)
#pragma unroll
                for (int e = 0; e < 3; ++e) *reinterpret_cast<f32x3_u32x2 *>(dst + e * kXPlane) = s.p[e];
        }
    };
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4 *lp;
    const int xrow0 = (PW == 16 ? (G >> 1) * HP + 8 * (G & 1) : G * HP) + (i >> 2);   // halo row that this lane points at, tap (0,0) of step 0

    Staged v;
    if (t_begin < t_end) {
        request(t_begin, v);
        stage(v, smem);
        request(min(t_begin + 1, t_end - 1), v);
    }
    for (int tile = t_begin; tile < t_end; ++tile) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // this patch's planes are visible, the other buffer is free
        const char *B = smem + ((tile - t_begin) & 1) * kBuf;
        char *other = smem + (((tile - t_begin) & 1) ^ 1) * kBuf;
#pragma nounroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 gf[3][NC];
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int row = chalf * 32 + c * 16 + i;
                    gf[e][c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x3_u32x4 *>(B + e * kGPlane + row * 128 + (((4 * s + G) ^ ((row >> 1) & 7)) << 4)));
                }
            bf16x8 xf[2][3];
            auto read_x = [&](int t) __attribute__((always_inline)) {
                const int r0 = xrow0 + (s * RPS + (T0 + t) / 3) * HP + (T0 + t) % 3, r1 = r0 + 4;
                const char *at = B + 3 * kGPlane + (i & 3) * 8;
                const char *a0 = at + r0 * 64 + x_half(r0, half), *a1 = at + r1 * 64 + x_half(r1, half);
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const s16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a0 + e * kXPlane));
                    const s16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a1 + e * kXPlane));
                    const s16x8 w = __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
                    xf[t & 1][e] = __builtin_bit_cast(bf16x8, w);
                }
            };
            read_x(0);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < NT) read_x(t + 1);
                __builtin_amdgcn_sched_barrier(0);
                auto terms = [&](bool high, int ge, int xe) __attribute__((always_inline)) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        f32x4w &acc = high ? hi[c][t] : lo[c][t];
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[ge][c], xf[t & 1][xe], acc, 0, 0, 0);
                    }
                };
                terms(true, 0, 0); terms(false, 0, 1); terms(false, 1, 0); terms(false, 1, 1); terms(false, 0, 2); terms(false, 2, 0);
            }
            if (s == 0 && tile + 1 < t_end) {
                stage(v, other);
                request(min(tile + 2, t_end - 1), v);
            }
        }
    }

    // register e of lane 16 G + i: output channel 4 G + e, input channel i
    const int ci = ci0 + half * 16 + i;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = co0 + chalf * 32 + c * 16 + G * 4 + e;
                if (co < p.Cout && ci < p.CinP)
                    p.part[(((size_t)split * 9 + T0 + t) * p.Cout + co) * p.CinP + ci] = join_parts(hi[c][t][e], lo[c][t][e]);
            }
    if (p.dbpart && tci == 0) {   // the eight runs' sums of g, in a fixed order
        float *red = reinterpret_cast<float *>(smem);
        __syncthreads();
        red[wv * 64 + lane] = gsum;
        __syncthreads();
        if (wv == 0 && co0 + lane < p.Cout) {
            float s = red[lane];
#pragma unroll
            for (int r = 1; r < 8; ++r) s += red[r * 64 + lane];
            p.dbpart[(size_t)split * p.Cout + co0 + lane] = s;
        }
    }
}

template <int PW>
__global__ __launch_bounds__(512, 2) void conv3x3_wgrad_f32x3_kernel(WgradF32x3Args p)
{
    extern __shared__ __align__(16) char smem[];
    // (each XCD, with its own L2, works through whole splits, whose blocks all read the same patches)
    const int nblk = gridDim.x, xcd = blockIdx.x & 7;
    int b = xcd * (nblk >> 3) + min(xcd, nblk & 7) + (blockIdx.x >> 3);
    const int tco = b % p.tiles_co; b /= p.tiles_co;
    const int tci = b % p.tiles_ci; b /= p.tiles_ci;
    // (wave-uniform branch: both bodies execute the same sequence of barriers)
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 8) == 0) body<PW, 0, 5>(p, smem, tco, tci, b);
    else body<PW, 5, 4>(p, smem, tco, tci, b);
}

}  // namespace

// g: patches of conv_wgrad.hip's plan, TH = 4 rows of TW = 14 or 16 pixels or 8 x 8; splits x tiles_per_split of them
int launch_wgrad_f32x3(const TileGeom &g, int CinP, int Cout, int splits, int tiles_per_split, const float *x, const float *grad, float *part,
                       float *dbpart, hipStream_t stream)
{
    WgradF32x3Args a;
    a.x = x; a.g = grad; a.part = part; a.dbpart = dbpart;
    a.N = g.N; a.H = g.H; a.W = g.W; a.CinP = CinP; a.Cout = Cout; a.tw = g.TW;
    a.tiles_co = (Cout + 63) / 64;
    a.tiles_ci = (CinP + 31) / 32;
    a.tiles_w = g.tiles_w; a.tiles_hw = g.tiles_hw; a.ntiles = g.ntiles; a.tiles_per_split = tiles_per_split;
    a.dTilesW = g.dTilesW; a.dTilesHW = g.dTilesHW;
    auto kern = g.TH == 8 ? conv3x3_wgrad_f32x3_kernel<8> : conv3x3_wgrad_f32x3_kernel<16>;
    if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.tiles_co * a.tiles_ci * splits)), dim3(512), 2 * kBuf, stream, a);
    return launch_status();
}

}  // namespace vgg
