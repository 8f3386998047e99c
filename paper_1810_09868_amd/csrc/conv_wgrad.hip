// Weight gradient of the 3x3 convolution on fp32 MFMA for gfx950, NHWC.
//
//   dw[t][co][ci] = sum_m g[m][co] * x[m + tap t][ci],   db[co] = sum_m g[m][co]
//
// (backward column of the appendix table: one more "convolution" per layer,
// plus a "reduce" for the bias).  GEMM view per tap: rows = co, columns = ci,
// contraction over the pixels m.  A workgroup owns a 64(co) x 32(ci) block of
// all nine taps and a range of pixel tiles (split-K).  Each of its eight waves
// takes one 32-row half of co, one half of a tile's pixels and five or four of
// the taps, and issues one v_mfma_f32_32x32x2_f32 per tap and pair of pixels,
// all fed from the same g fragment.
//
// Staging: the g rows and the x halo (see TileGeom) of a tile are copied
// straight into LDS by global_load_lds_dwordx4 (lane l of a wave writes bytes
// [16 l, 16 l + 16) of a 1 KB block and supplies its own source address, so
// rows outside the tensor simply read a block of zeros).  Two buffers: the
// copies of tile k+1 are issued between, and in flight during, the MFMA steps of
// tile k, one barrier per tile, no staging registers, no index tables (every lane derives the
// pixels it needs from the tile geometry with a few multiplies).  Rows are
// unpadded; the two pixels of an MFMA step sit in adjacent rows, which for
// 128-byte x rows are already 32 banks apart, and for 256-byte g rows are made
// so by swapping the two halves of every odd row.
//
// The two pixel-halves are added through LDS at the end and the block writes
// its partial sums; a second kernel adds the partials of all splits in a fixed
// order, so the result does not depend on scheduling.
#include "common.h"

namespace vgg {

constexpr int kPK = 64;         // pixels per tile
constexpr int kWaves = 8;
constexpr int kBCO = 64, kBCI = 32;
constexpr int kGRow = kBCO * 4;  // bytes per LDS row of g
constexpr int kXRow = kBCI * 4;  // bytes per LDS row of x

typedef unsigned int wg_u32x4 __attribute__((ext_vector_type(4)));
__device__ const wg_u32x4 kZeroSeg[1] = {};  // what a row outside the tensor reads

struct WgradArgs {
    const float *x;   // [M][CinP]
    const float *g;   // [M][Cout]
    float *part;      // [splits][9][Cout][CinP]
    float *dbpart;    // [splits][Cout] or null
    int CinP, Cout;
    int tiles_co, tiles_ci, splits, tiles_per_split;
    int SX;           // halo rows per buffer (geo.S rounded up to 8)
    TileGeom geo;
};

// Taps [T0, T0 + NT) of one wave: the main loop over the workgroup's tiles and the final sums.
// S0: MFMA step before which the wave prepares the next tile's copies.
template <int T0, int NT, int S0>
__device__ __forceinline__ void wgrad_body(const WgradArgs &p, char *smem)
{
    const int buf_bytes = kPK * kGRow + p.SX * kXRow;   // [kPK][256] g rows, then [SX][128] x rows

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    const int wc = wv & 1, wp = (wv >> 1) & 1;  // co half, pixel half (wv >> 2: tap group)

    int b = blockIdx.x;
    const int tco = b % p.tiles_co; b /= p.tiles_co;
    const int tci = b % p.tiles_ci; b /= p.tiles_ci;
    const int split = b;
    const int co0 = tco * kBCO, ci0 = tci * kBCI;
    const int pitch = p.geo.pitch;

    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    float gsum = 0.f;

    const int t_begin = split * p.tiles_per_split;
    const int t_end = min(t_begin + p.tiles_per_split, p.geo.ntiles);

    // Index arithmetic is kept off the lanes' critical path: a wave-wide instruction costs several
    // cycles whatever it computes, so every pixel index is derived once per tile by one lane and
    // handed to the lanes that need it (ds_bpermute / v_readlane) instead of once per user.
    //
    // Direct-to-LDS copies of a wave: 1 KB block wv + 8k of the g rows (4 rows of 16 segments; odd
    // rows hold their two halves swapped), k < kGOps, and block wv + 8k of the x halo (8 rows of
    // 8 segments), k < nxw.
    constexpr int kGOps = kPK / 4 / kWaves;
    const int nxw = ((p.SX >> 3) - wv + kWaves - 1) / kWaves;   // x blocks of this wave (SX >= 8 * kWaves)
    const int gsub = lane >> 4;                                  // row of this lane within a g block
    const int gcol = co0 + (((lane & 15) ^ ((gsub & 1) << 3)) << 2);
    const bool gok = gcol < p.Cout;
    const int xsub = lane >> 3;                                  // row of this lane within an x block
    const int xcol = ci0 + ((lane & 7) << 2);
    const bool xok = xcol < p.CinP;
    const float *zero = reinterpret_cast<const float *>(kZeroSeg);
    auto dma = [&](const float *src, char *dst) __attribute__((always_inline)) {
        const unsigned d = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)dst);
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(d), "v"(src) : "m0", "memory");
    };
    constexpr int kXBatch = 3;                 // x blocks of a wave whose copies are spread over the steps
    constexpr int kOps = kGOps + kXBatch;      // copies that are spread over the MFMA steps
    static_assert(S0 + kOps <= kPK / 4, "one copy per MFMA step");
    // lane l looks up halo row (l & 7) of this wave's x block k0 + (l >> 3) (blocks k0 .. k0 + 7)
    auto x_lookup = [&](const TileOrigin &org, int k0) __attribute__((always_inline)) {
        const int kk = k0 + (lane >> 3);
        const int i = (wv + kWaves * kk) * 8 + (lane & 7);
        return (kk < nxw && i < p.geo.S) ? halo_pixel(p.geo, org, i) : -1;
    };
    // source addresses of g copy k / of x copy k of a lookup; m_l: output pixel of tile row `lane`
    auto g_src = [&](int m_l, int k) __attribute__((always_inline)) {
        const int m = __builtin_amdgcn_ds_bpermute(((wv + kWaves * k) * 4 + gsub) << 2, m_l);
        return (gok && m >= 0) ? p.g + (size_t)m * p.Cout + gcol : zero;
    };
    auto x_src = [&](int px_l, int k) __attribute__((always_inline)) {
        const int px = __builtin_amdgcn_ds_bpermute(((k << 3) + xsub) << 2, px_l);
        return (xok && px >= 0) ? p.x + (size_t)px * p.CinP + xcol : zero;
    };
    auto g_dst = [&](char *base, int k) __attribute__((always_inline)) { return base + (wv + kWaves * k) * 1024; };
    auto x_dst = [&](char *base, int k) __attribute__((always_inline)) {
        return base + kPK * kGRow + (wv + kWaves * k) * 1024;
    };
    // x blocks beyond the first batch (large halos): issued in one go
    auto issue_rest = [&](const TileOrigin &org, char *base) __attribute__((always_inline)) {
        for (int k0 = kXBatch; k0 < nxw; k0 += 8) {
            const int px_l = x_lookup(org, k0);
            const int kn = min(nxw - k0, 8);
            for (int k = 0; k < kn; ++k) dma(x_src(px_l, k), x_dst(base, k0 + k));
        }
    };

    const int wrow0 = __builtin_amdgcn_readfirstlane(wp * (kPK / 2));
    const int nfirst = min(nxw, kXBatch);
    int hrow_l = 0;  // halo row (tap 0,0) of tile row `lane` of the tile being multiplied
    if (t_begin < t_end) {
        const TileOrigin org0 = tile_origin(p.geo, t_begin);
        int m_l;
        tile_row(p.geo, org0, lane, m_l, hrow_l);
#pragma unroll
        for (int k = 0; k < kGOps; ++k) dma(g_src(m_l, k), g_dst(smem, k));
        const int px_l = x_lookup(org0, 0);
        for (int k = 0; k < nfirst; ++k) dma(x_src(px_l, k), x_dst(smem, k));
        issue_rest(org0, smem);
    }
    for (int tile = t_begin; tile < t_end; ++tile) {
        const int buf = (tile - t_begin) & 1;
        // This tile's copies have landed (each wave waits for its own, the barrier publishes all),
        // and every wave is done with the other buffer, which the next copies overwrite.
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        // The next tile's copies are issued one per MFMA step rather than in a burst, and their
        // addresses are prepared before step S0: all waves of all workgroups on a CU run in
        // lockstep, so if every wave did this at the same point the MFMA pipes would idle meanwhile.
        const bool more = tile + 1 < t_end;
        char *nbase = smem + (buf ^ 1) * buf_bytes;
        int hrow_next = 0;
        const float *srcs[kOps];
        TileOrigin orgn;
        const int ncopy = more ? kGOps + nfirst : 0;
        auto prepare = [&]() __attribute__((always_inline)) {
            // all cross-lane reads first, then one wait: each of them has LDS latency
            orgn = tile_origin(p.geo, more ? tile + 1 : tile);
            int m_l;
            tile_row(p.geo, orgn, lane, m_l, hrow_next);
            const int px_l = x_lookup(orgn, 0);
#pragma unroll
            for (int k = 0; k < kGOps; ++k) srcs[k] = g_src(m_l, k);
#pragma unroll
            for (int k = 0; k < kXBatch; ++k) srcs[kGOps + k] = x_src(px_l, k);
        };

        const char *Gs = smem + buf * buf_bytes;
        const char *Xs = Gs + kPK * kGRow;
        // this wave: pixels [wp*32, wp*32+32) of the tile, two per MFMA step
        const char *ga = Gs + (wrow0 + kp) * kGRow + (((wc * 32 + r) ^ (kp << 5)) << 2);
        // operands of step s+1 are read from LDS before the MFMAs of step s are issued
        float a_next, b_next[NT];
        auto fetch = [&](int s) __attribute__((always_inline)) {
            a_next = *reinterpret_cast<const float *>(ga + s * 2 * kGRow);
            const int h0 = __builtin_amdgcn_readlane(hrow_l, wrow0 + 2 * s);
            const int h1 = __builtin_amdgcn_readlane(hrow_l, wrow0 + 2 * s + 1);
            const char *xb = Xs + (kp ? h1 : h0) * kXRow + r * 4;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                b_next[t] = *reinterpret_cast<const float *>(xb + (((T0 + t) / 3) * pitch + (T0 + t) % 3) * kXRow);
        };
        fetch(0);
#pragma unroll
        for (int s = 0; s < kPK / 4; ++s) {
            if (s == S0) prepare();
            if (s >= S0 && s - S0 < kOps && s - S0 < ncopy)
                dma(srcs[s - S0], s - S0 < kGOps ? g_dst(nbase, s - S0) : x_dst(nbase, s - S0 - kGOps));
            const float a = a_next;
            float bv[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[t] = b_next[t];
            if (s + 1 < kPK / 4) fetch(s + 1);
            gsum += a;
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, bv[t], acc[t], 0, 0, 0);
        }
        if (more) issue_rest(orgn, nbase);
        hrow_l = hrow_next;
    }

    // add the two pixel halves: waves with wp == 1 park their sums in LDS
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem);  // needs 2 * 9*16*64 floats = 73728 bytes
    if (wp == 1) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) red[((wc * 9 + T0 + t) * 16 + e) * 64 + lane] = acc[t][e];
    }
    __syncthreads();
    float gs_other = __shfl_xor(gsum, 32, kWave);  // the other pixel of the pair
    gsum += gs_other;
    float *dbs = reinterpret_cast<float *>(smem) + 2 * 9 * 16 * 64;  // [2][32]
    if (T0 == 0 && wp == 1 && kp == 0) dbs[wc * 32 + r] = gsum;
    if (wp == 0) {
        // accumulator layout: register e of lane l = row 8*(e/4) + 4*(l/32) + e%4 (co), column l%32 (ci)
        const int ci = ci0 + r;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int co = co0 + wc * 32 + (e >> 2) * 8 + kp * 4 + (e & 3);
                const float v = acc[t][e] + red[((wc * 9 + T0 + t) * 16 + e) * 64 + lane];
                if (co < p.Cout && ci < p.CinP)
                    p.part[(((size_t)split * 9 + T0 + t) * p.Cout + co) * p.CinP + ci] = v;
            }
    }
    __syncthreads();
    if (T0 == 0 && p.dbpart && tci == 0 && wp == 0 && kp == 0) {
        const int co = co0 + wc * 32 + r;
        if (co < p.Cout) p.dbpart[(size_t)split * p.Cout + co] = gsum + dbs[wc * 32 + r];
    }
}

// Eight waves: (co half) x (pixel half) x (taps 0-4 | taps 5-8).  Splitting the taps halves the
// accumulator registers of a wave, so four waves fit on a SIMD; a wave of each tap group lands on
// every SIMD (wave w runs on SIMD w % 4), which balances the 5:4 split; the two groups also prepare
// the next tile at different points of a tile, so a SIMD always has waves that are multiplying.
__global__ __launch_bounds__(kWaves * 64, 4) void conv3x3_wgrad_kernel(WgradArgs p)
{
    extern __shared__ __align__(16) char smem[];
    // (wave-uniform branch: both bodies execute the same sequence of barriers)
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 8) == 0) wgrad_body<0, 5, 0>(p, smem);
    else wgrad_body<5, 4, kPK / 8>(p, smem);
}

// Layers with at most three input channels (the first one): (tap, ci) pairs are the <= 27 columns
// of a single 32-wide MFMA tile, so a pair of pixels costs one MFMA per 32 output channels instead
// of nine.  Column c = tap*CI + ci of pixel m is x[m + tap][ci]: lane c reads it from the staged halo
// at a lane-constant offset.  Staging as in the general kernel.  Eight waves = (co half) x (pixel
// quarter); the quarters are added through LDS at the end.
__global__ __launch_bounds__(kWaves * 64, 4) void conv3x3_wgrad_thin_kernel(WgradArgs p, int CI)
{
    extern __shared__ __align__(16) char smem[];
    const int buf_bytes = kPK * kGRow + p.SX * kXRow;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    const int wc = wv & 1, wp = wv >> 1;  // co half, pixel quarter

    int b = blockIdx.x;
    const int tco = b % p.tiles_co; b /= p.tiles_co;
    const int split = b;
    const int co0 = tco * kBCO;
    const int pitch = p.geo.pitch;

    // this lane's column: tap and channel, as a byte offset from the halo row of tap (0,0)
    const bool cvalid = r < 9 * CI;
    const int tap = cvalid ? r / CI : 0, ci = cvalid ? r - tap * CI : 0;
    const int coff = ((tap / 3) * pitch + tap % 3) * kXRow + ci * 4;

    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    float gsum = 0.f;

    const int t_begin = split * p.tiles_per_split;
    const int t_end = min(t_begin + p.tiles_per_split, p.geo.ntiles);

    constexpr int kGOps = kPK / 4 / kWaves;
    const int nxw = ((p.SX >> 3) - wv + kWaves - 1) / kWaves;
    const int gsub = lane >> 4;
    const int gcol = co0 + (((lane & 15) ^ ((gsub & 1) << 3)) << 2);
    const bool gok = gcol < p.Cout;
    const int xsub = lane >> 3;
    const int xcol = (lane & 7) << 2;
    const bool xok = xcol < p.CinP;
    const float *zero = reinterpret_cast<const float *>(kZeroSeg);
    auto dma = [&](const float *src, char *dst) __attribute__((always_inline)) {
        const unsigned d = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)dst);
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(d), "v"(src) : "m0", "memory");
    };
    // all copies of a tile, in one go (there is little arithmetic to hide them behind)
    auto issue_tile = [&](const TileOrigin &org, char *base, int m_l) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kGOps; ++k) {
            const int q = wv + kWaves * k;
            const int m = __builtin_amdgcn_ds_bpermute((q * 4 + gsub) << 2, m_l);
            dma((gok && m >= 0) ? p.g + (size_t)m * p.Cout + gcol : zero, base + q * 1024);
        }
        for (int k0 = 0; k0 < nxw; k0 += 8) {
            const int kk = k0 + (lane >> 3);
            const int i = (wv + kWaves * kk) * 8 + (lane & 7);
            const int px_l = (kk < nxw && i < p.geo.S) ? halo_pixel(p.geo, org, i) : -1;
            const int kn = min(nxw - k0, 8);
            for (int k = 0; k < kn; ++k) {
                const int px = __builtin_amdgcn_ds_bpermute(((k << 3) + xsub) << 2, px_l);
                dma((xok && px >= 0) ? p.x + (size_t)px * p.CinP + xcol : zero,
                    base + kPK * kGRow + (wv + kWaves * (k0 + k)) * 1024);
            }
        }
    };

    const int wrow0 = __builtin_amdgcn_readfirstlane(wp * (kPK / 4));
    int hrow_l = 0;
    if (t_begin < t_end) {
        const TileOrigin org0 = tile_origin(p.geo, t_begin);
        int m_l;
        tile_row(p.geo, org0, lane, m_l, hrow_l);
        issue_tile(org0, smem, m_l);
    }
    for (int tile = t_begin; tile < t_end; ++tile) {
        const int buf = (tile - t_begin) & 1;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this tile's copies have landed
        __syncthreads();
        int hrow_next = 0;
        if (tile + 1 < t_end) {
            const TileOrigin orgn = tile_origin(p.geo, tile + 1);
            int m_l;
            tile_row(p.geo, orgn, lane, m_l, hrow_next);
            issue_tile(orgn, smem + (buf ^ 1) * buf_bytes, m_l);
        }
        const char *Gs = smem + buf * buf_bytes;
        const char *Xs = Gs + kPK * kGRow + coff;
        const char *ga = Gs + (wrow0 + kp) * kGRow + (((wc * 32 + r) ^ (kp << 5)) << 2);
        // this wave: pixels [wp*16, wp*16+16) of the tile, two per MFMA
#pragma unroll
        for (int s = 0; s < kPK / 8; ++s) {
            const int h0 = __builtin_amdgcn_readlane(hrow_l, wrow0 + 2 * s);
            const int h1 = __builtin_amdgcn_readlane(hrow_l, wrow0 + 2 * s + 1);
            const float a = *reinterpret_cast<const float *>(ga + s * 2 * kGRow);
            const float bv = *reinterpret_cast<const float *>(Xs + (kp ? h1 : h0) * kXRow);
            gsum += a;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, bv, acc, 0, 0, 0);
        }
        hrow_l = hrow_next;
    }

    // add the four pixel quarters: waves with wp > 0 park their sums in LDS
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem);            // [2][3][16][64]
    float *dbs = red + 2 * 3 * 16 * 64;                      // [2][3][32]
    gsum += __shfl_xor(gsum, 32, kWave);                     // the other pixel of the pair
    if (wp > 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) red[((wc * 3 + wp - 1) * 16 + e) * 64 + lane] = acc[e];
        if (kp == 0) dbs[(wc * 3 + wp - 1) * 32 + r] = gsum;
    }
    __syncthreads();
    if (wp == 0) {
        // accumulator layout: register e of lane l = row 8*(e/4) + 4*(l/32) + e%4 (co), column l%32 (tap, ci)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int co = co0 + wc * 32 + (e >> 2) * 8 + kp * 4 + (e & 3);
            float v = acc[e];
#pragma unroll
            for (int q = 0; q < 3; ++q) v += red[((wc * 3 + q) * 16 + e) * 64 + lane];
            if (cvalid && co < p.Cout) p.part[(((size_t)split * 9 + tap) * p.Cout + co) * p.CinP + ci] = v;
        }
        if (p.dbpart && kp == 0) {
            const int co = co0 + wc * 32 + r;
            float v = gsum;
#pragma unroll
            for (int q = 0; q < 3; ++q) v += dbs[(wc * 3 + q) * 32 + r];
            if (co < p.Cout) p.dbpart[(size_t)split * p.Cout + co] = v;
        }
    }
    // padding channels of this block's partial sums: exact zeros
    for (int i = tid; i < 9 * kBCO * (p.CinP - CI); i += kWaves * 64) {
        const int cpad = p.CinP - CI;
        const int t = i / (kBCO * cpad), rem = i - t * (kBCO * cpad), col = rem / cpad, c = CI + rem - col * cpad;
        if (co0 + col < p.Cout) p.part[(((size_t)split * 9 + t) * p.Cout + co0 + col) * p.CinP + c] = 0.f;
    }
}

// out[i] = sum over the splits of part[k][i], in a fixed order.  A thread owns four outputs (every count here is a
// multiple of four), a workgroup 1024 / RY of them; thread row y adds the splits k = y, y + RY, ... and the RY rows are
// then added through LDS, so that launches with few outputs and many splits (thin layers) still fill the chip.  Bound by
// reading the partials, 75 MB for 512 workgroups of bf16 64 x 64 blocks: 15 us; 4 bytes per lane and load took 16 to 31.
// Two sets of partials with the same number of splits (the weights' and the bias') share a launch: the quads [0, n4)
// come from part, [n4, n4 + n24) from part2.
// kReduceStep: out and out2 are master weights and biases, requested before the sums (a training step of 32 images 4272 -> 4241 us:
// the gradients, 80 MB, are neither written nor read again, and two launches less).
// kReduceRedo: partial sums of patches (conv_wgrad_f32x3.hip), which multiply zeros of g with real neighbours of x where a
// patch is narrower than the MFMA's rows or sticks out of the image.  Where that x is infinite the product is NaN and no part of
// the sum: a partial sum that is NaN is formed again from the patches' own pixels.  (Costs nothing here, where the sums are
// read anyway; a test per patch in the main kernel cost 4 to 14 % of it.  With one infinity in the last pixel, 256 -> 256 at 56x56,
// batch 100, takes 19 ms instead of 2.4, with nothing but NaN 2.4.)
enum ReduceKind { kReducePlain, kReduceStep, kReduceRedo };
struct PartRedo {
    const float *x, *g;   // null: no redo
    int H, W, CinP, Cout, TH, TW, tiles_w, tiles_hw, ntiles, tiles_per_split;
};
// Partial sums i .. i + 3 of split k, pixel by pixel in fp32 arithmetic.
__device__ __forceinline__ f32x4 redo_partial(const PartRedo &r, size_t i, int k)
{
    const int ci = (int)(i % r.CinP), co = (int)(i / r.CinP % r.Cout), tap = (int)(i / r.CinP / r.Cout);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    const int end = min((k + 1) * r.tiles_per_split, r.ntiles);
    for (int tile = k * r.tiles_per_split; tile < end; ++tile) {
        const int n = tile / r.tiles_hw, ty = tile % r.tiles_hw / r.tiles_w, tx = tile % r.tiles_hw % r.tiles_w;
        const int h1 = min((ty + 1) * r.TH, r.H), w1 = min((tx + 1) * r.TW, r.W);
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
        for (int h = ty * r.TH; h < h1; ++h)
            for (int w = tx * r.TW; w < w1; ++w) {
                const int hx = h + tap / 3 - 1, wx = w + tap % 3 - 1;
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
                if ((unsigned)hx < (unsigned)r.H && (unsigned)wx < (unsigned)r.W)
                    x = *reinterpret_cast<const f32x4 *>(r.x + (((size_t)n * r.H + hx) * r.W + wx) * r.CinP + ci);
                const float g = r.g[(((size_t)n * r.H + h) * r.W + w) * r.Cout + co];
#pragma unroll
                for (int c = 0; c < 4; ++c) t[c] = __builtin_fmaf(g, x[c], t[c]);
            }
        sum += t;
        if (sum[0] != sum[0] && sum[1] != sum[1] && sum[2] != sum[2] && sum[3] != sum[3]) break;
    }
    return sum;
}
template <int RY, int KIND>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const f32x4 *part, f32x4 *out, size_t n4, const f32x4 *part2,
                                                           f32x4 *out2, size_t n24, int splits, ConvStep step, PartRedo redo)
{
    constexpr bool STEP = KIND == kReduceStep;
    constexpr int RX = 256 / RY;
    __shared__ f32x4 red[RY > 1 ? 256 : 1];
    const int x = threadIdx.x % RX, y = threadIdx.x / RX;
    size_t i = (size_t)blockIdx.x * RX + x;
    // (threads beyond the last output read the first one's: a load under a condition is waited for where it ends)
    const bool live = i < n4 + n24, bias = live && i >= n4;
    if (bias) { i -= n4; part = part2; out = out2; n4 = n24; }
    if (!live) i = 0;
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, theta = s;
    if (STEP) theta = out[i];
#pragma unroll 8
    for (int k = y; k < splits; k += RY) s += part[(size_t)k * n4 + i];
    auto nan = [](const f32x4 &v) { return v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3]; };
    if (KIND == kReduceRedo && !bias && nan(s)) {
        s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
        for (int k = y; k < splits; k += RY) {
            f32x4 v = part[(size_t)k * n4 + i];
            if (nan(v)) {
                const f32x4 q = redo_partial(redo, i * 4, k);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = v[c] == v[c] ? v[c] : q[c];
            }
            s += v;
        }
    }
    if (RY > 1) {
        red[threadIdx.x] = s;
        __syncthreads();
        if (y) return;
        s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < RY; ++r) s += red[r * RX + x];
    }
    if (!live) return;
    if (STEP) {
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = sgd_step(theta[c], s[c], step.lr);
        if (bias) reinterpret_cast<f32x4 *>(step.bias_copy)[i] = s;
        else {
            const unsigned e = (unsigned)i * 4, row = e / (unsigned)step.CinP, tap = row / (unsigned)step.Cout;
            store4(step.copy + packed_w_index<bf16_t>((int)tap, (int)(row - tap * step.Cout), (int)(e - row * step.CinP), step.Cout,
                                                      step.CinP), s.x, s.y, s.z, s.w);
        }
    }
    out[i] = s;
}

static void launch_reduce(const float *part, float *out, size_t n, const float *part2, float *out2, size_t n2, int splits,
                          hipStream_t stream, const ConvStep &step = {}, const PartRedo &redo = {})
{
    const auto go = [&](auto plain, auto stepping, auto redoing, int rows) {
        const size_t per = 256 / rows;
        hipLaunchKernelGGL(step.copy ? stepping : redo.x ? redoing : plain, dim3((unsigned)(((n + n2) / 4 + per - 1) / per)), dim3(256), 0, stream,
                           reinterpret_cast<const f32x4 *>(part), reinterpret_cast<f32x4 *>(out), n / 4,
                           reinterpret_cast<const f32x4 *>(part2), reinterpret_cast<f32x4 *>(out2), n2 / 4, splits, step, redo);
    };
    // Rows by the number of partial results alone.  us for 4 bytes a load (as it was) / one / four / sixteen rows of quads,
    // splits x outputs: 8 x 2.4e6 15.6 / 15.4 / 15.6 / 23.7, 32 x 590e3 18.7 / 15.0 / 14.8 / 14.8, 64 x 295e3 19.9 / 15.3 /
    // 14.8 / 14.8, 128 x 147e3 24.8 / 14.6 / 15.0 / 15.2, 512 x 37e3 30.7 / 27.8 / 15.0 / 16.0, 1024 x 1728 23.0 / 51 / 18.5 / 8.4.
    if (splits >= 128) go(wgrad_reduce_kernel<16, kReducePlain>, wgrad_reduce_kernel<16, kReduceStep>, wgrad_reduce_kernel<16, kReduceRedo>, 16);
    else if (splits >= 16) go(wgrad_reduce_kernel<4, kReducePlain>, wgrad_reduce_kernel<4, kReduceStep>, wgrad_reduce_kernel<4, kReduceRedo>, 4);
    else go(wgrad_reduce_kernel<1, kReducePlain>, wgrad_reduce_kernel<1, kReduceStep>, wgrad_reduce_kernel<1, kReduceRedo>, 1);
}

// (also used by the bf16 weight-gradient kernel; part2/out2 may be null with n2 = 0)
void wgrad_launch_reduce(const float *part, float *out, size_t n, const float *part2, float *out2, size_t n2, int splits,
                         hipStream_t stream, const ConvStep &step)
{
    launch_reduce(part, out, n, part2, out2, n2, splits, stream, step);
}

int launch_wgrad_f32x3(const TileGeom &g, int CinP, int Cout, int splits, int tiles_per_split, const float *x, const float *grad, float *part,
                       float *dbpart, hipStream_t stream);   // conv_wgrad_f32x3.hip

static int wgrad_splits(int ntiles, int want, int &tiles_per_split)
{
    int splits = want < ntiles ? want : ntiles;
    if (splits < 1) splits = 1;
    tiles_per_split = (ntiles + splits - 1) / splits;
    return (ntiles + tiles_per_split - 1) / tiles_per_split;
}

// Patches of the kernel on the bf16 matrix unit: four rows of 16 or 14 pixels, or 8 x 8, sticking out of the image where they do
// not divide it; false: linear tiles on the fp32 MFMAs.  Four rows where the image width divides or they number at most 1.3 times
// the linear tiles: 0.45 to 0.9 of the time of the fp32 MFMAs on the same patches.  Otherwise the shape with fewest, from 64
// patches on and up to 2.2 times the linear tiles (what is multiplied for nothing included): over 104 shapes 0.65 of the linear kernel's time up to 1.4
// times, 0.7 to 1.6, 0.82 (0.96 at most) beyond 1.7.
static bool wgrad_patches(int N, int H, int W, int &TH, int &TW)
{
    const long tiles = ((long)N * H * W + kPK - 1) / kPK;
    const int c14 = ((W + 13) / 14) * ((H + 3) / 4), c16 = ((W + 15) / 16) * ((H + 3) / 4), c8 = ((W + 7) / 8) * ((H + 7) / 8);
    TH = 4;
    if (H >= 4) {
        TW = W % 16 == 0 ? 16 : W % 14 == 0 || (W + 13) / 14 * 14 < (W + 15) / 16 * 16 ? 14 : 16;
        if (W % TW == 0 || (long)N * (TW == 14 ? c14 : c16) * 10 <= tiles * 13) return true;
    }
    const int c = c8 <= c16 && c8 <= c14 ? c8 : c16 <= c14 ? c16 : c14;
    TH = c == c8 ? 8 : 4;
    TW = c == c8 ? 8 : c == c16 ? 16 : 14;
    return (long)N * c >= 64 && (long)N * c * 10 <= tiles * 22;
}

static bool wgrad_parts(const WgradArgs &a) { return a.geo.mode == 1; }   // (of a plan that is not the thin kernel's)

static void wgrad_plan(int N, int H, int W, int CinP, int Cout, WgradArgs &a, bool thin = false)
{
    a.geo = make_tile_geom(N, H, W, kPK);
    a.CinP = CinP; a.Cout = Cout;
    a.tiles_co = (Cout + kBCO - 1) / kBCO;
    a.tiles_ci = thin ? 1 : (CinP + kBCI - 1) / kBCI;
    const int groups = a.tiles_co * a.tiles_ci;
    // One resident round of workgroups (two per CU; on the bf16 matrix unit one, and never more partial sums than linear tiles
    // would have).  Every workgroup writes its whole block of partial sums, which the reduction reads back -- 38 MB each way for
    // 512 workgroups whatever the layer; four rounds (for balance) quadrupled that and measured 2.7 % slower over the whole stack.
    const int linear = wgrad_splits((int)(((long)N * H * W + kPK - 1) / kPK), (512 + groups - 1) / groups, a.tiles_per_split);
    int TH, TW;
    if (!thin && wgrad_patches(N, H, W, TH, TW)) {
        a.geo.mode = 1; a.geo.TH = TH; a.geo.TW = TW;
        a.geo.tiles_w = (W + TW - 1) / TW;
        a.geo.tiles_hw = a.geo.tiles_w * ((H + TH - 1) / TH);
        a.geo.dTilesW = make_fast_div(a.geo.tiles_w);
        a.geo.dTilesHW = make_fast_div(a.geo.tiles_hw);
        a.geo.ntiles = N * a.geo.tiles_hw;
        a.geo.pitch = TW + 2;
        a.geo.S = (TH + 2) * (TW + 2);
        a.splits = wgrad_splits(a.geo.ntiles, 256 / groups < linear ? 256 / groups : linear, a.tiles_per_split);
    } else {
        a.splits = wgrad_splits(a.geo.ntiles, (512 + groups - 1) / groups, a.tiles_per_split);
    }
    a.SX = (a.geo.S + 7) & ~7;
    if (a.SX < 8 * kWaves) a.SX = 8 * kWaves;  // every wave copies at least one halo block
}

// The thin kernel serves layers with at most three input channels; it tiles the pixels linearly, so its
// split count differs from the general kernel's.  Query and launch must agree on which one runs.
static bool wgrad_is_thin(int Cin, int CinP) { return Cin <= 3 && CinP <= kBCI; }

static size_t wgrad_ws_bytes(const WgradArgs &a)
{
    return round_up((size_t)a.splits * 9 * a.Cout * a.CinP * 4, 256) + round_up((size_t)a.splits * a.Cout * 4, 256);
}

size_t conv3x3_wgrad_workspace(int N, int H, int W, int Cin, int CinP, int Cout)
{
    WgradArgs a;
    wgrad_plan(N, H, W, CinP, Cout, a, wgrad_is_thin(Cin, CinP));
    return wgrad_ws_bytes(a);
}

// For inspection: {kernel (0 linear tiles, 8 / 14 / 16 patch width, 3 thin), pixel tiles, splits, tiles per split,
// workgroups}.
void conv3x3_wgrad_plan_info(int N, int H, int W, int Cin, int CinP, int Cout, int info[5])
{
    WgradArgs a;
    const bool thin = wgrad_is_thin(Cin, CinP);
    wgrad_plan(N, H, W, CinP, Cout, a, thin);
    info[0] = thin ? 3 : (!wgrad_parts(a) ? 0 : a.geo.TW);
    info[1] = a.geo.ntiles;
    info[2] = a.splits;
    info[3] = a.tiles_per_split;
    info[4] = a.tiles_co * a.tiles_ci * a.splits;
}

// x [M][CinP] fp32 (channels >= Cin are zero), g [M][Cout] fp32 -> dw [9][Cout][CinP], db [Cout] (may be null).
// ws_bytes: size of ws; the launch is refused when the partial sums of its own plan would not fit.
int conv3x3_wgrad(int N, int H, int W, int Cin, int CinP, int Cout, const float *x, const float *g, float *dw,
                  float *db, void *ws, size_t ws_bytes, hipStream_t stream)
{
    const bool thin = wgrad_is_thin(Cin, CinP);
    WgradArgs a;
    wgrad_plan(N, H, W, CinP, Cout, a, thin);
    if (ws_bytes < wgrad_ws_bytes(a)) return VGG_ERR_WORKSPACE;
    a.x = x; a.g = g;
    const size_t nw = (size_t)9 * Cout * CinP;
    a.part = static_cast<float *>(ws);
    a.dbpart = db ? reinterpret_cast<float *>(static_cast<char *>(ws) + round_up((size_t)a.splits * nw * 4, 256))
                  : nullptr;
    if (!thin && wgrad_parts(a)) {
        const int rc = launch_wgrad_f32x3(a.geo, CinP, Cout, a.splits, a.tiles_per_split, x, g, a.part, a.dbpart, stream);
        if (rc) return rc;
        const TileGeom &t = a.geo;
        launch_reduce(a.part, dw, nw, a.dbpart, db, db ? (size_t)Cout : 0, a.splits, stream, {},
                      PartRedo{x, g, H, W, CinP, Cout, t.TH, t.TW, t.tiles_w, t.tiles_hw, t.ntiles, a.tiles_per_split});
        return launch_status();
    }
    size_t lds = (size_t)2 * (kPK * kGRow + a.SX * kXRow);
    const size_t red = (size_t)2 * 9 * 16 * 64 * 4 + 64 * 4;
    if (lds < red) lds = red;
    if (lds > 160 * 1024) return VGG_ERR_UNSUPPORTED;
    if (lds > 64 * 1024 &&
        !(raise_lds_limit(reinterpret_cast<const void *>(conv3x3_wgrad_kernel)) && raise_lds_limit(reinterpret_cast<const void *>(conv3x3_wgrad_thin_kernel))))
        return VGG_ERR_LAUNCH;
    const dim3 grid((unsigned)(a.tiles_co * a.tiles_ci * a.splits));
    if (thin)
        hipLaunchKernelGGL(conv3x3_wgrad_thin_kernel, grid, dim3(kWaves * 64), lds, stream, a, Cin);
    else
        hipLaunchKernelGGL(conv3x3_wgrad_kernel, grid, dim3(kWaves * 64), lds, stream, a);
    if (hipGetLastError() != hipSuccess) return VGG_ERR_LAUNCH;
    launch_reduce(a.part, dw, nw, a.dbpart, db, db ? (size_t)Cout : 0, a.splits, stream);
    return launch_status();
}

}  // namespace vgg
