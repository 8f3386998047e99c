// Shared by the implicit-GEMM convolution kernels: their arguments, the bias, and how a tile leaves.
#pragma once
#include "common.h"

#include <type_traits>
#include <utility>

namespace vgg {

constexpr int kRowBytes = 80;  // 64 data + 16 pad
constexpr int kDataBytes = 64;
constexpr int kEpiRow = 144;              // epilogue transpose: 128 data bytes + 16 pad per row
constexpr int kEpiBytes = 32 * kEpiRow;   // per wave
constexpr int kMaxAHaloSegsPerBlock = 1536;  // 16-byte halo segments (384 rows) prefetched through registers
constexpr int kDmaHaloRows = 384;            // halo rows of the direct-to-LDS kernel: 2 workgroups of 74 KB per CU
constexpr int kDmaHaloRowsBig = 448;         // ... and of its variant for tiles that straddle images (78 KB)
constexpr int kDmaHaloRowsHalf = 192;        // ... and of the 128-pixel tiles (38 KB: four workgroups per CU)

struct ConvArgs {
    const char *x;      // [M][CinP] elements of T
    const char *w;      // [9][Cout][CinP]
    const float *bias;  // [Cout] or null
    const char *mask;   // [M][Cout] of T or null: output multiplied by (mask > 0)
    char *y;            // [M][Cout], or null when only the pooled tensor is wanted
    char *pool;         // [N][H/2][W/2][Cout] or null: 2x2 max of the result (patch tiles only)
    int CinP, Cout;
    int relu;
    int tiles_n;        // number of column tiles
    int rowsA;          // LDS rows reserved for the halo
    unsigned char *argmax;  // with pool, optional: [N][H/2][W/2][Cout], 2*dh+dw of the first maximum of each window
    float *part;        // [ksplit][M][Cout] partial sums when the contraction is split over workgroups, else null
    int ksplit;         // workgroups per tile (>= 1)
    int kchunks;        // channel chunks per workgroup
    FastDiv dTiles;     // conv3x3_small_bf16_kernel: division by the number of pixel tiles,
    int tableA;         // ... byte offset of its table of halo rows in LDS
    TileGeom g;
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
static __device__ const u32x4 kZeroRow[4] = {};  // 64 zero bytes: what a halo row outside the image reads

template <typename T> struct Mma;
template <> struct Mma<float> {
    static __device__ __forceinline__ void run(f32x16 &acc, const uint4 &a, const uint4 &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
    }
};
template <> struct Mma<bf16_t> {
    static __device__ __forceinline__ void run(f32x16 &acc, const uint4 &a, const uint4 &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                      __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
};

// The MFMAs are issued with the weight fragment as the first operand, so a 32x32 accumulator holds
// the tile transposed: register e of lane l is channel 8*(e/4) + 4*(l/32) + e%4 of pixel row l%32,
// i.e. a lane owns runs of four consecutive channels of one pixel.
//
// Accumulators start at the bias, so the epilogue has no bias to fetch or add.  init_acc only
// requests the values (into the first pixel block's registers).
template <int BN, int WN, int TM, int TN>
__device__ __forceinline__ void init_acc(f32x16 (&acc)[TM][TN], const ConvArgs &p, int n0, int wn, int khalf)
{
    // (channels past Cout are never stored: their loads are clamped into range instead of skipped;
    // one uniform branch around straight-line loads, so that none of them waits for another)
    const int c0 = n0 + wn * (BN / WN) + khalf * 4;
    if (!p.bias || p.part) {   // (split contraction: the finishing kernel adds the bias)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[0][j][e] = 0.f;
    } else if ((p.Cout & 3) == 0) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 b = *reinterpret_cast<const f32x4 *>(p.bias + min(c0 + j * 32 + a * 8, p.Cout - 4));
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[0][j][a * 4 + k] = b[k];
            }
    } else {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc[0][j][e] = p.bias[min(c0 + j * 32 + (e >> 2) * 8 + (e & 3), p.Cout - 1)];
    }
}
// Second half, called once the loads above have had time to land: the other pixel blocks start
// from the same values.
template <int TM, int TN>
__device__ __forceinline__ void spread_acc(f32x16 (&acc)[TM][TN])
{
#pragma unroll
    for (int i = 1; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc[0][j];
}

// Epilogue of a workgroup that holds only part of the contraction: raw fp32 sums to the partial
// buffer of its split (a lane owns runs of four consecutive channels of one pixel: 16-byte stores).
template <int BM, int BN, int WM, int WN>
__device__ __forceinline__ void conv_partial_epilogue(f32x16 (&acc)[BM / WM / 32][BN / WN / 32], const ConvArgs &p,
                                                      const TileOrigin &org, int n0, int split)
{
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv % WM, wn = wv / WM;
    const int r = lane & 31, khalf = lane >> 5;
    float *part = p.part + (size_t)split * p.g.M * p.Cout;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = tile_pixel(p.g, org, wm * (BM / WM) + i * 32 + r);
        if (m < 0) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int col = n0 + wn * (BN / WN) + j * 32 + a * 8 + khalf * 4;
                if (col < p.Cout) {   // Cout is a multiple of 4 when the contraction is split
                    const f32x4 v = {acc[i][j][a * 4], acc[i][j][a * 4 + 1], acc[i][j][a * 4 + 2], acc[i][j][a * 4 + 3]};
                    *reinterpret_cast<f32x4 *>(part + (size_t)m * p.Cout + col) = v;
                }
            }
    }
}

// Epilogue shared by the kernels below; called by every thread of the workgroup once all MFMAs are
// issued.  smem is the start of the workgroup's dynamic LDS, which is reused here.  How the accumulators
// are spread over lanes and registers is the caller's business: stage(i, j0, epi, lo) writes pixel block i
// (32 tile rows) x the 128 bytes of columns that start at MFMA column tile j0 of the wave into the wave's
// staging block (row r at epi + r * kEpiRow), each value raised to at least lo; each_element(f) calls
// f(tile row, column within the wave's 64- or 128-column range, value) for everything the lane holds.
template <typename T, int BM, int BN, int WM, int WN, typename Stage, typename EachElement>
__device__ __forceinline__ void conv_epilogue_impl(Stage stage, EachElement each_element, const ConvArgs &p,
                                                   const TileOrigin &org, char *smem, int n0)
{
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int wm = wv % WM, wn = wv / WM;
    // Epilogue: ReLU, optional (mask > 0) factor, convert, store (the bias is already in the sums).
    // A lane owns four-channel runs of one pixel (see init_acc).  Each wave passes 32 pixels x 128
    // bytes at a time through a private LDS block so that every lane then stores 16 contiguous bytes.
    T *y = reinterpret_cast<T *>(p.y);
    const T *mask = reinterpret_cast<const T *>(p.mask);
    constexpr int VEC = 16 / (int)sizeof(T);        // elements per 16-byte store
    constexpr int CPT = 128 / (int)sizeof(T);       // columns per transposed pass (64 bf16 / 32 fp32)
    constexpr int TJ = CPT / 32;                    // MFMA column tiles per pass
    static_assert(TN % TJ == 0, "wave tile must hold whole passes");
    __syncthreads();  // staging data no longer needed: LDS is reused
    if (p.Cout % VEC == 0) {
        char *epi = smem + wv * kEpiBytes;
        const int seg = lane & 7, rowq = lane >> 3;
        const float lo = p.relu ? 0.f : -__builtin_inff();
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j0 = 0; j0 < TN; j0 += TJ) {
                stage(i, j0, epi, lo);   // (no ReLU: maximum with -inf, one instruction either way)
                const int colbase = n0 + wn * (BN / WN) + j0 * 32 + seg * VEC;
                if (p.pool) {
                    // Patch tiles: these 32 rows are two patch rows of 16 pixels, i.e. eight whole 2x2
                    // windows; lane = (window, 16-byte segment).  Window (dx) = rows 2dx, 2dx+1, 16+2dx, 17+2dx.
                    const int win = lane >> 3;
                    T best[VEC];
                    unsigned char which[VEC];   // k = 2*dh + dw of the first maximum (replaced only by a strictly greater value)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int row = (k >> 1) * kTileW + 2 * win + (k & 1);
                        const u32x4 v = *reinterpret_cast<const u32x4 *>(epi + row * kEpiRow + seg * 16);
                        T ve[VEC];
                        __builtin_memcpy(ve, &v, 16);
#pragma unroll
                        for (int c = 0; c < VEC; ++c)
                            if (k == 0 || Elem<T>::load(ve + c) > Elem<T>::load(best + c)) { best[c] = ve[c]; which[c] = (unsigned char)k; }
                    }
                    const int j = wm * (BM / WM) + i * 32;  // first tile row of this block (even patch row)
                    const int ph = (org.h0 + j / kTileW) >> 1, pw = (org.w0 >> 1) + win;
                    if (2 * ph < p.g.H && 2 * pw < p.g.W && colbase < p.Cout) {
                        u32x4 v;
                        __builtin_memcpy(&v, best, 16);
                        T *po = reinterpret_cast<T *>(p.pool);
                        const size_t at = (((size_t)org.n * (p.g.H >> 1) + ph) * (p.g.W >> 1) + pw) * p.Cout + colbase;
                        *reinterpret_cast<u32x4 *>(po + at) = v;
                        if (p.argmax) __builtin_memcpy(p.argmax + at, which, VEC);
                    }
                }
                if (y == nullptr) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = rowq + 8 * q;
                    u32x4 v = *reinterpret_cast<const u32x4 *>(epi + row * kEpiRow + seg * 16);
                    const int m = tile_pixel(p.g, org, wm * (BM / WM) + i * 32 + row);
                    if (m >= 0 && colbase < p.Cout) {
                        const size_t o = (size_t)m * p.Cout + colbase;
                        if (mask) {
                            const u32x4 mk = *reinterpret_cast<const u32x4 *>(mask + o);
                            T ve[VEC], me[VEC];
                            __builtin_memcpy(ve, &v, 16);
                            __builtin_memcpy(me, &mk, 16);
#pragma unroll
                            for (int k = 0; k < VEC; ++k)
                                if (!(Elem<T>::load(me + k) > 0.f)) ve[k] = (T)0;
                            __builtin_memcpy(&v, ve, 16);
                        }
                        *reinterpret_cast<u32x4 *>(y + o) = v;
                    }
                }
            }
        }
        return;
    }
    // channel counts that do not allow 16-byte stores: element-wise
    each_element([&](int row, int c, float v) __attribute__((always_inline)) {
        const int m = tile_pixel(p.g, org, row);
        const int col = n0 + wn * (BN / WN) + c;
        if (m >= 0 && col < p.Cout) {
            if (p.relu) v = fmaxf(v, 0.f);
            const size_t o = (size_t)m * p.Cout + col;
            if (mask && !(Elem<T>::load(mask + o) > 0.f)) v = 0.f;
            Elem<T>::store(y + o, v);
        }
    });
}

// ... for 32x32 accumulators (see init_acc for their layout)
template <typename T, int BM, int BN, int WM, int WN>
__device__ __forceinline__ void conv_epilogue(f32x16 (&acc)[BM / WM / 32][BN / WN / 32], const ConvArgs &p,
                                              const TileOrigin &org, char *smem, int n0)
{
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int TJ = 128 / (int)sizeof(T) / 32;   // MFMA column tiles per staged pass
    const int lane = threadIdx.x & 63, wm = (threadIdx.x >> 6) % WM;
    const int r = lane & 31, khalf = lane >> 5;
    conv_epilogue_impl<T, BM, BN, WM, WN>(
        [&](int i, int j0, char *epi, float lo) __attribute__((always_inline)) {
#pragma unroll
            for (int jj = 0; jj < TJ; ++jj)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f32x16 &t = acc[i][j0 + jj];
                    store4(reinterpret_cast<T *>(epi + r * kEpiRow) + jj * 32 + a * 8 + khalf * 4, fmaxf(t[a * 4], lo),
                           fmaxf(t[a * 4 + 1], lo), fmaxf(t[a * 4 + 2], lo), fmaxf(t[a * 4 + 3], lo));
                }
        },
        [&](auto f) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        f(wm * (BM / WM) + i * 32 + r, j * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3), acc[i][j][e]);
        },
        p, org, smem, n0);
}

template <typename F, int... S>
__device__ __forceinline__ void for_each_step(F &&f, std::integer_sequence<int, S...>)
{
    (f(std::integral_constant<int, S>{}), ...);
}

typedef float f32x4v __attribute__((ext_vector_type(4)));

constexpr int kF32x3HaloRowsHalfBig = 256;   // most halo rows of the 128-pixel tiles (75 KB: two workgroups per CU)
// fp32 on tiles of g (256 or 128 pixels; narrow or 128 pixels: 64 channels, else 128), conv_f32x3.hip
int launch_conv_f32x3(const ConvArgs &a, const TileGeom &g, bool narrow, hipStream_t stream);

}  // namespace vgg
