// Dense layers on MFMA for gfx950: z = a * W^T + b (the paper's
// dense(W, x, b) = W*x + b, listing "dense", HLO "dot") and its two backward
// products.  At batch ~100 these are weight-streaming problems: every weight
// is read from HBM exactly once and the batch rows are the MFMA's M side.
#include "common.h"
#include "f32x3.h"

#include <type_traits>

namespace vgg {

template <typename T> struct FcMma;
template <> struct FcMma<float> {
    static __device__ __forceinline__ void run(f32x16 &acc, const uint4 &a, const uint4 &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
    }
};
template <> struct FcMma<bf16_t> {
    static __device__ __forceinline__ void run(f32x16 &acc, const uint4 &a, const uint4 &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                      __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
};

// ------------------------------------------------------------------ forward
// Workgroup: up to 128 batch rows (MB blocks of 32) x 128 outputs x a range of 64-byte K units.
// Wave w owns outputs [32w, 32w+32) and all row blocks.  Bound by streaming the weights (bf16) or by the MFMAs (fp32 from
// about 64 rows on).  Both operands of a step (4 units = 256 bytes per row) are loaded as whole 256-byte runs of four rows,
// and take the MFMA's layout through LDS, the weights in a block of the wave's own: loads in the MFMA's layout fetch
// 32 bytes of 32 rows each, and a cache line four times over.  25088 -> 4096, whole calls: bf16 batch 100 71 -> 56 us, batch 32
// 57 -> 39 (5.3 TB/s); fp32 batch 100 249 -> 222; bf16 4096 -> 4096, batch 100 21.3 -> 16.3.
struct FcArgs {
    const char *a;   // [N][In]
    const char *w;   // [Out][In]
    float *part;     // [splits][N][Out]
    int N, In, Out;
    int units;            // 64-byte K units per row: In * sizeof(T) / 64, rounded up
    int units_per_split;
    int tiles_n;          // column tiles
    int tiles_m;          // row tiles
};

typedef unsigned fc_u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes at byte offset `off` of a row of `rowbytes` bytes, zeros at and beyond the row's end, for rows that are not
// whole 16-byte segments: gathered element by element, so that any row length works.
template <typename T>
__device__ __forceinline__ fc_u32x4 gather_seg(const char *row, size_t off, size_t rowbytes)
{
    fc_u32x4 v;
    T e[16 / sizeof(T)];
#pragma unroll
    for (int k = 0; k < (int)(16 / sizeof(T)); ++k)
        e[k] = off + k * sizeof(T) < rowbytes ? reinterpret_cast<const T *>(row + off)[k] : (T)0;
    __builtin_memcpy(&v, e, 16);
    return v;
}

// VEC: rows are whole 16-byte segments (one load each; past the range its last segment again, replaced by zeros on the way
// to LDS: a load under a condition is waited for where the condition ends).
// MB: 32-row blocks of the batch tile.  STREAM: the weights pass the caches by.
template <typename T, bool VEC, int MB, bool STREAM>
__global__ __launch_bounds__(256, 2) void fc_fwd_kernel(FcArgs p)
{
    typedef fc_u32x4 u32x4;
    constexpr int kRow = 256 + 16;                          // LDS row of a step
    __shared__ __align__(16) char As[MB * 32 * kRow];       // [batch row]
    __shared__ __align__(16) char Ws[4 * 32 * kRow];        // [wave][output]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, khalf = lane >> 5;
    int b = blockIdx.x;
    const int tn = b % p.tiles_n; b /= p.tiles_n;
    const int tm = b % p.tiles_m; b /= p.tiles_m;
    const int split = b;
    const int row0 = tm * (MB * 32), o0 = tn * 128;
    const int u_begin = split * p.units_per_split;
    const int u_end = min(u_begin + p.units_per_split, p.units);
    const size_t rowbytes = (size_t)p.In * sizeof(T);

    const int ocol = o0 + wv * 32 + r;
    const bool ook = ocol < p.Out;
    char *const Wv = Ws + wv * (32 * kRow);

    f32x16 acc[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

    // Both operands of a step are requested one step ahead and held in registers, so the weight
    // stream from HBM never pauses for the staging and the MFMAs.  The barriers are issued without
    // the fence of __syncthreads(), which would wait for those loads.
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    constexpr int NA = MB * 32 * 16 / 256;   // activation segments per thread and step
    // Four whole 256-byte rows per load, rearranged through LDS: a load in the MFMA's layout touches 32 rows, a quarter of a
    // cache line each.  (Rows past the last are the last again, never stored.)
    const int seg = lane & 15;
    const size_t end = min((size_t)u_end * 64, rowbytes);
    auto load_w = [&](int u0, u32x4 (&wf)[8]) __attribute__((always_inline)) {
        const size_t off = (size_t)u0 * 64 + seg * 16;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const char *row = p.w + (size_t)min(o0 + wv * 32 + q * 4 + (lane >> 4), p.Out - 1) * rowbytes;
            if (VEC) {
                const u32x4 *src = reinterpret_cast<const u32x4 *>(row + min(off, end - 16));
                wf[q] = STREAM ? __builtin_nontemporal_load(src) : *src;
            } else wf[q] = gather_seg<T>(row, off, end);
        }
    };
    auto load_a = [&](int u0, u32x4 (&av)[NA]) __attribute__((always_inline)) {
        const size_t off = (size_t)u0 * 64 + seg * 16;
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            const char *row = p.a + (size_t)min(row0 + (tid >> 4) + k * 16, p.N - 1) * rowbytes;
            if (VEC) av[k] = *reinterpret_cast<const u32x4 *>(row + min(off, end - 16));
            else av[k] = gather_seg<T>(row, off, end);
        }
    };
    u32x4 w_next[8];
    u32x4 a_next[NA];
    if (u_begin < u_end) { load_a(u_begin, a_next); load_w(u_begin, w_next); }
    for (int u0 = u_begin; u0 < u_end; u0 += 4) {
        barrier();  // the previous step's fragment reads are done
        if (VEC && (size_t)(u0 + 4) * 64 > end && (size_t)u0 * 64 + seg * 16 >= end) {
#pragma unroll
            for (int k = 0; k < NA; ++k) a_next[k] = u32x4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 8; ++q) w_next[q] = u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int k = 0; k < NA; ++k) *reinterpret_cast<u32x4 *>(As + ((tid >> 4) + k * 16) * kRow + seg * 16) = a_next[k];
#pragma unroll
        for (int q = 0; q < 8; ++q) *reinterpret_cast<u32x4 *>(Wv + (q * 4 + (lane >> 4)) * kRow + seg * 16) = w_next[q];
        if (u0 + 4 < u_end) { load_a(u0 + 4, a_next); load_w(u0 + 4, w_next); }
        barrier();  // the staged activations are visible
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!VEC && u0 + u >= u_end) break;   // (zeros only; 145 x 6 -> 1863 in fp32 13.2 -> 10.7 us)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                const uint4 bf = *reinterpret_cast<const uint4 *>(Wv + r * kRow + u * 64 + g * 32 + khalf * 16);
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const uint4 af = *reinterpret_cast<const uint4 *>(As + (i * 32 + r) * kRow + u * 64 + g * 32 + khalf * 16);
                    FcMma<T>::run(acc[i], af, bf);
                }
            }
        }
    }
    if (ook) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = row0 + i * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
                if (row < p.N) p.part[((size_t)split * p.N + row) * p.Out + ocol] = acc[i][e];
            }
    }
}

// Small batches: bound by streaming the weights once.  Workgroup: 16 outputs x the whole contraction, its waves
// taking turns at 256-byte pieces of it, so that a workgroup reads 4 KB runs of its sixteen weight rows; batch rows come in
// sixteens (NB of them).  The waves' sums meet in LDS: no partial sums in memory and no second launch.
// A piece of the weights is loaded as four whole rows per load and takes the MFMA's layout through the wave's own LDS
// block, as the activations do: loaded straight in that layout every load touched sixteen rows and half of each cache
// line it fetched.  25088 -> 4096: bf16 batch 1 38.5 -> 32.7 us, batch 10 43.2 -> 35.4 (5.8 TB/s; a bare read of as many bytes
// takes 30.5); fp32 batch 10 80 -> 69, batch 20 138 -> 97.
// The lane layout is that of the 16-row MFMAs: lane 16 g + c holds 16 bytes (piece offset 64 e + 16 g) of weight row
// c and of batch row c; any fixed pairing of contraction indices between the two is a valid order.
// Sixteen waves of 128 registers, or eight of 256 for two blocks of batch rows, which do not fit 128.  A third piece in
// flight was slower (43 -> 45 us in the first form).
constexpr int fc_small_waves(int NB) { return NB == 1 ? 16 : 8; }

// Rows of whole 16-byte segments, and a shape where the split over workgroups is the slower one.  A workgroup walks its
// sixteen rows alone, at about 2.5 KB of row per us whatever the chip does besides, against the split's second launch and
// partial sums: the longest row, in KB, over 1500 shapes (time here / split up to it, and beyond):
//   up to 16 batch rows, outputs  up to 1499 10 (0.5 to 0.93; 0.97 to 1.1 at 12 KB), up to 2499 17 (0.5 to 0.96; 1.0 to 1.07 at 23 KB),
//                                 more: bf16 50 (0.54 to 1.05; 0.95 to 1.34), fp32 100 (0.52 to 1.02; 0.83 to 1.4)
//   17 to 32 (twice the activations per workgroup)  up to 2499 6.5 (0.55 to 1.0; 0.97 to 1.27 at 8 KB), up to 5000 17 (0.55 to 1.02;
//                                 0.86 to 1.3), up to 8191 6.5 (0.7 to 1.0; 1.0 to 1.2), more: never (1.04 to 1.24)
//   bf16, 8192 outputs and more, rows below 8 KB: 1.04 to 1.12
static bool fc_small(int dtype, int N, int In, int Out)
{
    const size_t rowbytes = (size_t)In * dtype_size(dtype), KB = 1024;
    if (rowbytes % 16 || N > 32) return false;
    const bool f32 = dtype == VGG_F32;
    if (N > 16) return Out < 8192 && rowbytes * 2 <= (Out >= 2500 && Out <= 5000 ? 34 : 13) * KB;
    if (!f32 && Out >= 8192 && rowbytes < 8 * KB) return false;
    return rowbytes <= (Out < 1500 ? 10 : Out < 2500 ? 17 : f32 ? 100 : 50) * KB;
}
// Weights of half the memory-side cache (256 MB) and more are not kept in any cache between two calls, and read once per call:
// nontemporal loads stream 6.6 TB/s where plain ones reach 6.0 (25088 -> 4096 bf16, 10 rows: 37.6 -> 35.4 us; 32 MB of weights,
// still cached: 8.2 -> 8.5).
static bool fc_streams(int dtype, int In, int Out) { return (size_t)In * Out * dtype_size(dtype) >= (size_t)128 << 20; }

template <typename T, typename TZ, int NB, bool STREAM>
__global__ __launch_bounds__(fc_small_waves(NB) * 64) void fc_fwd_small_kernel(const char *__restrict__ a, const char *__restrict__ w,
                                                                             const float *__restrict__ bias, TZ *__restrict__ z,
                                                                             int N, int In, int Out, int relu)
{
    typedef float f32x4m __attribute__((ext_vector_type(4)));
    constexpr int NW = fc_small_waves(NB);
    constexpr int ROW = 256 + 16;                         // LDS bytes per row of a wave's piece
    constexpr int kRed = NB * 16 * 17;                    // sums of a wave
    static_assert(kRed * 4 <= NB * 16 * ROW, "the sums take the place of the activations");
    extern __shared__ __align__(16) char smem[];          // [wave][16 weight rows, NB * 16 batch rows][ROW], later [wave][kRed]
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int o0 = blockIdx.x * 16;
    const size_t rowbytes = (size_t)In * sizeof(T);
    // (rows past the ends are clamped: what they yield is not stored)
    constexpr int kWave = (16 + NB * 16) * ROW;           // LDS bytes of a wave
    char *Ws = smem + wv * kWave, *As = Ws + 16 * ROW;
    f32x4m acc[NB];
#pragma unroll
    for (int x = 0; x < NB; ++x) acc[x] = f32x4m{0.f, 0.f, 0.f, 0.f};
    // Four whole rows of a piece per load, rearranged through the wave's own LDS block, which needs no barrier.
    typedef fc_u32x4 u32x4;
    struct Piece { u32x4 w[4], a[NB * 4]; };
    const int pieces = (int)((rowbytes + 255) / 256);
    auto load = [&](int k, Piece &v) __attribute__((always_inline)) {
        // (past the row's end: its last 16 bytes again, and zeros for both operands below)
        const size_t off = (size_t)k * 256 + c * 16, at = off < rowbytes ? off : rowbytes - 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 *src = reinterpret_cast<const u32x4 *>(w + (size_t)min(o0 + 4 * i + g, Out - 1) * rowbytes + at);
            if (STREAM) v.w[i] = __builtin_nontemporal_load(src);
            else v.w[i] = *src;
        }
#pragma unroll
        for (int i = 0; i < NB * 4; ++i) v.a[i] = *reinterpret_cast<const u32x4 *>(a + (size_t)min(4 * i + g, N - 1) * rowbytes + at);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int k, Piece &v) __attribute__((always_inline)) {
        if ((size_t)(k + 1) * 256 > rowbytes && (size_t)k * 256 + c * 16 >= rowbytes) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v.w[i] = u32x4{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < NB * 4; ++i) v.a[i] = u32x4{0, 0, 0, 0};
        }
        uint4 wf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(Ws + (4 * i + g) * ROW + c * 16) = v.w[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) wf[e] = *reinterpret_cast<const uint4 *>(Ws + c * ROW + e * 64 + g * 16);
#pragma unroll
        for (int i = 0; i < NB * 4; ++i) *reinterpret_cast<u32x4 *>(As + (4 * i + g) * ROW + c * 16) = v.a[i];
        uint4 af[NB][4];
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
            for (int e = 0; e < 4; ++e) af[x][e] = *reinterpret_cast<const uint4 *>(As + (x * 16 + c) * ROW + e * 64 + g * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                if constexpr (sizeof(T) == 2) {
                    acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[e]), __builtin_bit_cast(bf16x8, af[x][e]), acc[x], 0, 0, 0);
                } else {
                    const f32x4 wv4 = __builtin_bit_cast(f32x4, wf[e]), xf = __builtin_bit_cast(f32x4, af[x][e]);
#pragma unroll
                    for (int k4 = 0; k4 < 4; ++k4) acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv4[k4], xf[k4], acc[x], 0, 0, 0);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    // two sets of registers taken in turn, a piece each, the next requested before the current one is multiplied
    Piece v0, v1;
    const int last = pieces - 1;
    if (wv < pieces) load(wv, v0);
    for (int k = wv; k < pieces; k += 2 * NW) {   // (past the end: the last piece again, not used)
        load(min(k + NW, last), v1);
        multiply(k, v0);
        if (k + NW >= pieces) break;
        load(min(k + 2 * NW, last), v0);
        multiply(k + NW, v1);
    }
    // register e of lane 16 g + c: output o0 + 4 g + e of batch row c (a wave's sums go to its own LDS block)
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wv * (kWave / 4) + (x * 16 + c) * 17 + 4 * g + e] = acc[x][e];
    __syncthreads();
    for (int i = tid; i < NB * 256; i += NW * 64) {
        const int n = i >> 4, o = i & 15;
        if (n >= N || o0 + o >= Out) continue;
        float s = bias ? bias[o0 + o] : 0.f;
#pragma unroll
        for (int v = 0; v < NW; ++v) s += red[v * (kWave / 4) + n * 17 + o];
        if (relu) s = fmaxf(s, 0.f);
        Elem<TZ>::store(z + (size_t)n * Out + o0 + o, s);
    }
}

template <typename T, typename TZ>
static int launch_fc_small(const void *a, const void *w, const float *bias, void *z, int N, int In, int Out, int relu, hipStream_t s)
{
    const int nb = N <= 16 ? 1 : 2;
    auto launch = [&](auto kern) {
        if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return (int)VGG_ERR_LAUNCH;
        const int waves = fc_small_waves(nb);
        const size_t lds = (size_t)waves * (16 + nb * 16) * (256 + 16);
        hipLaunchKernelGGL(kern, dim3((unsigned)((Out + 15) / 16)), dim3(waves * 64), lds, s, (const char *)a, (const char *)w,
                           bias, (TZ *)z, N, In, Out, relu);
        return launch_status();
    };
    const bool stream = fc_streams(sizeof(T) == 2 ? VGG_BF16 : VGG_F32, In, Out);
    if (nb == 1) return stream ? launch(fc_fwd_small_kernel<T, TZ, 1, true>) : launch(fc_fwd_small_kernel<T, TZ, 1, false>);
    return stream ? launch(fc_fwd_small_kernel<T, TZ, 2, true>) : launch(fc_fwd_small_kernel<T, TZ, 2, false>);
}

// z = f(bias + sum over splits), converted to TZ.  Bound by reading the partial sums, eight of them in flight (one at a time
// was a chain of loads: 16 splits of 100 x 4096 8.8 -> 6 us).
template <typename TZ>
__global__ __launch_bounds__(256) void fc_finish_kernel(const float *__restrict__ part, const float *__restrict__ bias, TZ *__restrict__ z,
                                                        int N, int Out, int splits, int relu)
{
    const size_t n = (size_t)N * Out;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float s = bias ? bias[i % Out] : 0.f;
#pragma unroll 8
    for (int k = 0; k < splits; ++k) s += part[(size_t)k * n + i];
    if (relu) s = fmaxf(s, 0.f);
    Elem<TZ>::store(z + i, s);
}

// launch: the query sizes the workspace for two workgroups per CU; the launch takes one per CU for rows of up to 32 KB, where
// writing and reading the partial sums costs as much as streaming the weights (bf16 4096 -> 4096, batch 100: 20.0 -> 17.5 us;
// 25088 -> 4096 bf16 54 / 55, fp32 217 / 230: there two share the CU's memory latency).
static void fc_plan(int dtype, int N, int In, int Out, FcArgs &a, bool launch)
{
    a.N = N; a.In = In; a.Out = Out;
    a.units = (In * dtype_size(dtype) + 63) / 64;
    a.tiles_n = (Out + 127) / 128;
    a.tiles_m = (N + 127) / 128;
    const int tiles = a.tiles_n * a.tiles_m;
    const int want = launch && a.units <= 512 && (dtype == VGG_BF16 || N <= 32) ? 256 : 512;
    int splits = (want + tiles - 1) / tiles;
    const int max_splits = (a.units + 7) / 8;  // at least two steps per split
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    a.units_per_split = ((a.units + splits - 1) / splits + 3) / 4 * 4;
}

static int fc_splits(const FcArgs &a) { return (a.units + a.units_per_split - 1) / a.units_per_split; }

size_t fc_workspace(int dtype, int N, int In, int Out)
{
    FcArgs a;
    fc_plan(dtype, N, In, Out, a, false);
    return round_up((size_t)fc_splits(a) * N * Out * 4, 256);
}

int fc_forward(int dtype, int N, int In, int Out, const void *a_, const void *w, const float *bias, void *z, int z_dtype,
               int relu, void *ws, hipStream_t s)
{
    if (fc_small(dtype, N, In, Out)) {
        if (dtype == VGG_BF16)
            return z_dtype == VGG_BF16 ? launch_fc_small<bf16_t, bf16_t>(a_, w, bias, z, N, In, Out, relu, s)
                                       : launch_fc_small<bf16_t, float>(a_, w, bias, z, N, In, Out, relu, s);
        return z_dtype == VGG_BF16 ? launch_fc_small<float, bf16_t>(a_, w, bias, z, N, In, Out, relu, s)
                                   : launch_fc_small<float, float>(a_, w, bias, z, N, In, Out, relu, s);
    }
    FcArgs a;
    fc_plan(dtype, N, In, Out, a, true);
    const int splits = fc_splits(a);
    a.a = static_cast<const char *>(a_);
    a.w = static_cast<const char *>(w);
    a.part = static_cast<float *>(ws);
    const dim3 grid((unsigned)(a.tiles_n * a.tiles_m * splits));
    const bool vec = (size_t)In * dtype_size(dtype) % 16 == 0;
    const bool stream = a.tiles_m == 1 && fc_streams(dtype, In, Out);
    const int mb = N > 96 ? 4 : (N + 31) / 32;
    auto launch = [&](auto elem, auto vc, auto st) {
        typedef decltype(elem) T;
        constexpr bool V = decltype(vc)::value, ST = decltype(st)::value;
        switch (mb) {
        case 1: hipLaunchKernelGGL((fc_fwd_kernel<T, V, 1, ST>), grid, dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL((fc_fwd_kernel<T, V, 2, ST>), grid, dim3(256), 0, s, a); break;
        case 3: hipLaunchKernelGGL((fc_fwd_kernel<T, V, 3, ST>), grid, dim3(256), 0, s, a); break;
        default: hipLaunchKernelGGL((fc_fwd_kernel<T, V, 4, ST>), grid, dim3(256), 0, s, a);
        }
    };
    auto launch_t = [&](auto elem) {
        if (!vec) launch(elem, std::false_type{}, std::false_type{});
        else if (stream) launch(elem, std::true_type{}, std::true_type{});
        else launch(elem, std::true_type{}, std::false_type{});
    };
    if (dtype == VGG_BF16) launch_t(bf16_t{});
    else launch_t(float{});
    if (hipGetLastError() != hipSuccess) return VGG_ERR_LAUNCH;
    const size_t n = (size_t)N * Out;
    const dim3 g2((unsigned)((n + 255) / 256));
    if (z_dtype == VGG_BF16)
        hipLaunchKernelGGL(fc_finish_kernel<bf16_t>, g2, dim3(256), 0, s, a.part, bias, (bf16_t *)z, N, Out, splits, relu);
    else
        hipLaunchKernelGGL(fc_finish_kernel<float>, g2, dim3(256), 0, s, a.part, bias, (float *)z, N, Out, splits, relu);
    return launch_status();
}

// ------------------------------------------------- backward: dW = dz^T * a
// fp32, up to 40 batch rows; bound by its MFMAs and, under them, by writing dW.  Workgroup: 128 (o) x 128 (i) block of dW; the batch is
// the contraction index, staged through LDS 32 rows at a time, and multiplied eight rows (four MFMA steps) at a time
// up to the last one: 33 rows cost 40.  Wave w owns outputs [32 w, 32 w + 32) and all 128 inputs: lane r reads four
// consecutive inputs with one 16-byte LDS read and feeds them to four MFMA column tiles, so accumulator tile j of lane r
// holds input 4 r + j and the stores are 16 bytes, 512 contiguous per row; 64 accumulator registers, so that four
// workgroups share a CU and some store while others multiply.  (Operands straight from L2 without LDS: the loads between
// the MFMAs hold up their issue.)  25088 -> 4096: 10 rows 77 us, 32 rows 87 (4.8 TB/s of dW), 40 rows 111; from 41 rows on the
// kernel below takes over.
// VEC: In is a multiple of 4; otherwise the four inputs are written one by one.

// Four floats row[c..c+3], zeros at and beyond column C.  vec: the row is 16-byte aligned (C a multiple of 4).
__device__ __forceinline__ f32x4 load_row4(const float *row, int c, int C, bool vec)
{
    if (vec && c + 3 < C) return *reinterpret_cast<const f32x4 *>(row + c);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (c < C) v[0] = row[c];
    if (c + 1 < C) v[1] = row[c + 1];
    if (c + 2 < C) v[2] = row[c + 2];
    if (c + 3 < C) v[3] = row[c + 3];
    return v;
}

template <bool VEC>
__global__ __launch_bounds__(256, 4) void fc_dw_kernel(const float *__restrict__ a, const float *__restrict__ dz,
                                                       float *__restrict__ dw, int N, int In, int Out)
{
    constexpr int ROW = 128 * 4 + 16;
    __shared__ __align__(16) char lds[66 * ROW];
    char *const Ds = lds, *const As = lds + 32 * ROW;   // 32 rows each (and two that are read but not used)
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    const int tiles_i = (In + 127) / 128;
    const int i0 = (blockIdx.x % tiles_i) * 128, o0 = (blockIdx.x / tiles_i) * 128;

    f32x16 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

    // The 32 batch rows of a pass are requested one pass ahead; barriers without the fence of
    // __syncthreads(), which would wait for those loads.
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const int seg = tid & 31, row_t = tid >> 5;
    f32x4 vd[4], va[4];
    auto request = [&](int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = n0 + row_t + 8 * q;
            vd[q] = va[q] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row < N) {
                vd[q] = load_row4(dz + (size_t)row * Out, o0 + seg * 4, Out, (Out & 3) == 0);
                va[q] = load_row4(a + (size_t)row * In, i0 + seg * 4, In, (In & 3) == 0);
            }
        }
    };
    request(0);
    for (int n0 = 0; n0 < N; n0 += 32) {
        barrier();  // the previous pass's fragment reads are done
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = row_t + 8 * q;
            *reinterpret_cast<f32x4 *>(Ds + row * ROW + seg * 16) = vd[q];
            *reinterpret_cast<f32x4 *>(As + row * ROW + seg * 16) = va[q];
        }
        barrier();  // the staged rows are visible
        if (n0 + 32 < N) request(n0 + 32);
        // Four steps at a time (rows past the batch are zeros), each one's operands read while the step before it is
        // multiplied; the last read of a pass is one step past what it needs (LDS past Ds is As; past As: padding).
        const char *ds = Ds + kp * ROW + (wv * 32 + r) * 4, *as = As + kp * ROW + r * 16;
        const int steps = min((N - n0 + 1) / 2, 16);
        float d = *reinterpret_cast<const float *>(ds);
        f32x4 x = *reinterpret_cast<const f32x4 *>(as);
        for (int s = 0; s < steps; s += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float dc = d;
                const f32x4 xc = x;
                d = *reinterpret_cast<const float *>(ds + 2 * (s + k + 1) * ROW);
                x = *reinterpret_cast<const f32x4 *>(as + 2 * (s + k + 1) * ROW);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(dc, xc[j], acc[j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    const int ic = i0 + 4 * r;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int o = o0 + wv * 32 + (e >> 2) * 8 + kp * 4 + (e & 3);
        if (o >= Out) continue;
        float *dst = dw + (size_t)o * In + ic;
        // (streamed out: 411 MB for the first dense layer, re-read only by the update, long after it has left every cache)
        if (VEC) {
            if (ic < In) __builtin_nontemporal_store(f32x4{acc[0][e], acc[1][e], acc[2][e], acc[3][e]}, reinterpret_cast<f32x4 *>(dst));
        } else
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (ic + j < In) __builtin_nontemporal_store(acc[j][e], dst + j);
    }
}

// The same on the bf16 matrix unit (f32x3.h), for more than 40 batch rows where dz is not in parts ahead; bound by splitting the operands, the MFMAs and
// writing dW together.  Workgroup: 128 (o) x 128 (i) block of dW; the batch is the contraction index, staged through LDS 32 rows
// at a time as three planes of bf16 parts, and multiplied sixteen rows at a time up to the last one: 100 rows cost 112.  A
// thread loads sixteen batch rows of one output and of one input, so that they leave for LDS already transposed: rows of 32
// batch rows = 64 bytes, segment s at s ^ ((row >> 1) & 3), one 16-byte read per fragment (two transpose reads each, from rows
// as they lie, were slower at every size).  Wave (wo, wi) owns 64 x 64 = 2 x 2 MFMA tiles; input 2 r + y of its 64 lies in column r of tile y,
// so that a lane stores two neighbouring inputs and 32 lanes 256 bytes.
template <bool VEC>
__global__ __launch_bounds__(256, 2) void fc_dw_f32x3_kernel(const float *__restrict__ a, const float *__restrict__ dz,
                                                       float *__restrict__ dw, int N, int In, int Out)
{
    constexpr int PLANE = 128 * 64;
    __shared__ __align__(16) char lds[6 * PLANE];
    char *const Ds = lds, *const As = lds + 3 * PLANE;   // [part][output / input][32 batch rows]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    const int wo = wv & 1, wi = wv >> 1;
    const int tiles_i = (In + 127) / 128;
    const int i0 = (blockIdx.x % tiles_i) * 128, o0 = (blockIdx.x / tiles_i) * 128;

    f32x16 hi[2][2], lo[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) hi[x][y][e] = lo[x][y][e] = 0.f;

    // The 32 batch rows of a pass are requested one pass ahead, sixteen rows of one output and of one input per thread (past
    // the ends: the last ones again); barriers without the fence of __syncthreads(), which would wait for those loads.
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const int col = tid & 127, half = __builtin_amdgcn_readfirstlane(tid >> 7);
    const float *const dcol = dz + min(o0 + col, Out - 1), *const xcol = a + min(i0 + col, In - 1);
    unsigned vd[16], va[16];
    auto request = [&](int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const size_t row = min(n0 + half * 16 + j, N - 1);
            vd[j] = __float_as_uint(dcol[row * Out]);
            va[j] = __float_as_uint(xcol[row * In]);
        }
    };
    // eight batch rows of one column: a 16-byte segment of every part
    auto store8 = [&](char *plane, int row, int seg, const unsigned *v, int valid) __attribute__((always_inline)) {
        f32x3_u32x4 x, y;
#pragma unroll
        for (int j = 0; j < 4; ++j) { x[j] = v[j]; y[j] = v[j + 4]; }
        if (valid < 8) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { x[j] = j < valid ? x[j] : 0u; y[j] = j + 4 < valid ? y[j] : 0u; }
        }
        const Parts4 s = split_parts(x), t = split_parts(y);
#pragma unroll
        for (int e = 0; e < 3; ++e)
            *reinterpret_cast<f32x3_u32x4 *>(plane + e * PLANE + row * 64 + (((seg ^ (row >> 1)) & 3) << 4)) =
                f32x3_u32x4{s.p[e][0], s.p[e][1], t.p[e][0], t.p[e][1]};
    };
    const int arow = (col & 64) + (col & 1) * 32 + ((col & 63) >> 1);
    request(0);
    for (int n0 = 0; n0 < N; n0 += 32) {
        barrier();  // the previous pass's fragment reads are done
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int valid = N - n0 - half * 16 - h * 8;
            store8(Ds, col, half * 2 + h, vd + h * 8, valid);
            store8(As, arow, half * 2 + h, va + h * 8, valid);
        }
        barrier();  // the staged rows are visible
        if (n0 + 32 < N) request(n0 + 32);
        const int steps = min((N - n0 + 15) / 16, 2);
        for (int s = 0; s < steps; ++s) {
            bf16x8 df[3][2], af[3][2];
            auto frag = [&](const char *plane, int row) __attribute__((always_inline)) {
                return __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x3_u32x4 *>(plane + row * 64 + ((((2 * s + kp) ^ (row >> 1)) & 3) << 4)));
            };
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    df[e][x] = frag(Ds + e * PLANE, wo * 64 + x * 32 + r);
                    af[e][x] = frag(As + e * PLANE, wi * 64 + x * 32 + r);
                }
            auto terms = [&](f32x16(&acc)[2][2], int de, int ae) __attribute__((always_inline)) {
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df[de][x], af[ae][y], acc[x][y], 0, 0, 0);
            };
            terms(hi, 0, 0); terms(lo, 0, 1); terms(lo, 1, 0); terms(lo, 1, 1); terms(lo, 0, 2); terms(lo, 2, 0);
        }
    }
    const int ic = i0 + wi * 64 + 2 * r;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int o = o0 + wo * 64 + x * 32 + (e >> 2) * 8 + kp * 4 + (e & 3);
            if (o >= Out) continue;
            typedef float f32x2_t __attribute__((ext_vector_type(2)));
            const f32x2_t v = {join_parts(hi[x][0][e], lo[x][0][e]), join_parts(hi[x][1][e], lo[x][1][e])};
            float *dst = dw + (size_t)o * In + ic;
            // (streamed out: 411 MB for the first dense layer, re-read only by the update, long after it has left every cache)
            if (VEC) {
                if (ic < In) __builtin_nontemporal_store(v, reinterpret_cast<f32x2_t *>(dst));
            } else
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (ic + j < In) __builtin_nontemporal_store(v[j], dst + j);
        }
}

// db[o] = sum_n dz[n][o].  A workgroup owns 64 outputs; each of its four waves sums every fourth row and
// the four partial sums are added in a fixed order (one thread per output walking all rows alone was a
// chain of N dependent loads on sixteen CUs: 29 us for 4096 outputs).
__global__ __launch_bounds__(256) void fc_db_kernel(const float *__restrict__ dz, float *__restrict__ db, int N, int Out)
{
    __shared__ float part[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int o = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (o < Out) {
#pragma unroll 4
        for (int n = wv; n < N; n += 4) s += dz[(size_t)n * Out + o];
    }
    part[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && o < Out) db[o] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

// --------------------------------------------------- backward: da = dz * W
// fp32, up to 40 batch rows; bound by streaming W.  Workgroup: 16 NB batch rows x 256 inputs x
// a range of outputs (the contraction index); wave w owns 64 of the inputs.  v_mfma_f32_16x16x4_f32: rows come in
// sixteens, so ten cost 16.  A weight is used by one lane only and goes straight to
// its register, sixteen outputs per unit, a unit ahead; the dz rows, which all four waves need, go through LDS 64
// outputs (four units) at a time.  (Straight from the caches they held up the MFMAs' issue: 16 segments of 64 bytes
// per load.)  Lane 16 g + c loads inputs 4 c .. 4 c + 3 of weight row o = 4 g + e with one 16-byte load and feeds
// them to four MFMA column tiles, and outputs 4 g .. 4 g + 3 of batch row c: step e contracts outputs 4 g + e.
// Accumulator tile j of lane c holds input 4 c + j: the stores are 16 bytes.  25088 -> 4096, batch 10: 69 us, 5.9 TB/s.
struct FcDaArgs {
    const float *dz;  // [N][Out]
    const float *w;   // [Out][In]
    float *part;      // [splits][N][In]
    int N, In, Out;
    int tiles_i, tiles_m, o_per_split;
    int nb;           // 16-row blocks per row tile
};

// VEC: In is a multiple of 4, so a lane's four inputs are one aligned 16-byte load and store; otherwise
// they are read and written one by one.
template <int NB, bool VEC>
__global__ __launch_bounds__(256, 2) void fc_da_kernel(FcDaArgs p)
{
    constexpr int AHEAD = 1;   // units of weights in flight
    constexpr int ROW = 64 * 4 + 16, Q = NB * 4;   // LDS row of 64 outputs; values of a pass per thread
    __shared__ __align__(16) char Ds[2][NB * 16 * ROW];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    int b = blockIdx.x;
    const int ti = b % p.tiles_i; b /= p.tiles_i;
    const int tm = b % p.tiles_m; b /= p.tiles_m;
    const int split = b;
    const int row0 = tm * NB * 16;
    const int ic = ti * 256 + wv * 64 + 4 * c;  // first of this lane's 4 inputs (clamped where there are none)
    const int o_begin = split * p.o_per_split, o_end = min(o_begin + p.o_per_split, p.Out);
    const float *wp = p.w + (VEC ? min(ic, p.In - 4) : 0);

    typedef float f32x4m __attribute__((ext_vector_type(4)));
    f32x4m acc[NB][4];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[x][j] = f32x4m{0.f, 0.f, 0.f, 0.f};

    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // dz, outputs o .. o + 63, to registers and on to LDS, one value per lane and load: a wave reads 256 contiguous
    // bytes of a row whatever its alignment (past the range: zeros; rows past the batch: the last row, never stored)
    float dn[Q];
    auto load_dz = [&](int o) __attribute__((always_inline)) {
        const int col = min(o + lane, p.Out - 1);
#pragma unroll
        for (int k = 0; k < Q; ++k) dn[k] = p.dz[(size_t)min(row0 + wv + 4 * k, p.N - 1) * p.Out + col];
    };
    auto store_dz = [&](int o, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < Q; ++k)
            *reinterpret_cast<float *>(Ds[buf] + (wv + 4 * k) * ROW + lane * 4) = o + lane < o_end ? dn[k] : 0.f;
    };
    // weights of outputs o .. o + 15 (past the range: its last row again; dz is zero there, see below for the weight)
    struct Unit { f32x4 w[4]; };
    auto load_w = [&](int o, Unit &v) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *src = wp + (size_t)min(o + 4 * g + e, o_end - 1) * p.In;
            if (VEC) v.w[e] = *reinterpret_cast<const f32x4 *>(src);
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) v.w[e][j] = src[min(ic + j, p.In - 1)];
        }
        __builtin_amdgcn_sched_barrier(0);   // (the scheduler would move the requests behind the MFMAs that follow)
    };
    auto multiply = [&](const Unit &v, int buf, int h) __attribute__((always_inline)) {
        // (each block's dz fragment is read while the block before it is multiplied)
        const char *d0 = Ds[buf] + c * ROW + h * 64 + g * 16;
        f32x4 d[2];
        d[0] = *reinterpret_cast<const f32x4 *>(d0);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            if (x + 1 < NB) d[(x + 1) & 1] = *reinterpret_cast<const f32x4 *>(d0 + (x + 1) * 16 * ROW);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[x][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[x & 1][e], v.w[e][j], acc[x][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (o_begin < o_end) {
        Unit v[4];   // (two or three of the four are in use at a time)
        load_dz(o_begin);
#pragma unroll
        for (int h = 0; h < AHEAD; ++h) load_w(o_begin + 16 * h, v[h]);
        store_dz(o_begin, 0);
        barrier();
        int buf = 0;
        for (int o = o_begin; o < o_end; o += 64, buf ^= 1) {
            const bool more = o + 64 < o_end;
            if (more) load_dz(o + 64);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                load_w(o + 16 * (h + AHEAD), v[(h + AHEAD) & 3]);
                if (o + 64 > o_end) {   // the range's last pass: weights past its end are zero, whatever the last row holds
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o + 16 * h + 4 * g + e >= o_end) v[h].w[e] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                multiply(v[h], buf, h);
            }
            if (more) store_dz(o + 64, buf ^ 1);
            barrier();   // every wave is done with this pass's rows, the next pass's are visible
        }
    }
    // accumulator layout: register e of lane 16 g + c = row 4 g + e, column c
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = row0 + x * 16 + 4 * g + e;
            if (row >= p.N) continue;
            float *dst = p.part + ((size_t)split * p.N + row) * p.In + ic;
            if (VEC) {
                if (ic < p.In) *reinterpret_cast<f32x4 *>(dst) = f32x4{acc[x][0][e], acc[x][1][e], acc[x][2][e], acc[x][3][e]};
            } else
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (ic + j < p.In) dst[j] = acc[x][j][e];
        }
}

// The same on the bf16 matrix unit (f32x3.h), where the dW kernel above runs.  Workgroup, one per CU: eight waves, 16 NB batch rows x 256 inputs x a range of
// outputs (the contraction index), 32 at a time.  Both operands go through LDS as three planes of bf16 parts, rows of 32
// outputs = 64 bytes whose 16-byte segment s lies at s ^ ((row >> 1) & 3); a thread loads sixteen outputs of one input, so
// that they leave for LDS already transposed.  Two buffers and one barrier per step: one wave of a SIMD splits and stores
// while the other multiplies.  Wave w owns inputs 32 w .. 32 w + 31 as two tiles of sixteen, the weights as first operand, so
// that a lane holds four neighbouring inputs of a batch row and stores 16 bytes.
template <int NB, bool DVEC>
__global__ __launch_bounds__(512, 2) void fc_da_f32x3_kernel(FcDaArgs p)
{
    typedef float f32x4m __attribute__((ext_vector_type(4)));
    constexpr int WPLANE = 256 * 64, DPLANE = NB * 16 * 64, BUF = 3 * (WPLANE + DPLANE);
    constexpr int ND = (NB * 16 * 8 + 511) / 512;         // 16-byte segments of dz per thread
    extern __shared__ __align__(16) char lds[];           // [2][weights: part][256][64], [dz: part][NB * 16][64]
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane & 15, g = lane >> 4;
    int b = blockIdx.x;
    const int ti = b % p.tiles_i; b /= p.tiles_i;
    const int tm = b % p.tiles_m; b /= p.tiles_m;
    const int split = b;
    const int row0 = tm * NB * 16, i0 = ti * 256;
    const int o_begin = split * p.o_per_split, o_end = min(o_begin + p.o_per_split, p.Out);
    const bool wvec = (p.In & 3) == 0;

    f32x4m hi[NB][2], lo[NB][2];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) hi[x][y] = lo[x][y] = f32x4m{0.f, 0.f, 0.f, 0.f};
    // weights: outputs 16 half .. 16 half + 15 of input `col`; dz: outputs 4 dseg .. of batch rows drow, drow + 64
    // (inputs and rows past the ends: the last ones again, never stored; outputs past the range: zeros)
    const int col = tid & 255, half = __builtin_amdgcn_readfirstlane(tid >> 8), dseg = tid & 7, drow = tid >> 3;
    const float *const wcol = p.w + min(i0 + col, p.In - 1);
    struct Step { unsigned w[16]; f32x4 d[ND]; };
    auto request = [&](int o, Step &v) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 16; ++j) v.w[j] = __float_as_uint(wcol[(size_t)min(o + half * 16 + j, p.Out - 1) * p.In]);
#pragma unroll
        for (int k = 0; k < ND; ++k) {   // (unconditional: a load under a condition is waited for where the condition ends)
            const float *src = p.dz + (size_t)min(row0 + drow + 64 * k, p.N - 1) * p.Out;
            if (DVEC) v.d[k] = *reinterpret_cast<const f32x4 *>(src + min(o + dseg * 4, p.Out - 4));
            else
#pragma unroll
                for (int e = 0; e < 4; ++e) v.d[k][e] = src[min(o + dseg * 4 + e, p.Out - 1)];
        }
    };
    auto stage = [&](int o, const Step &v, char *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x3_u32x4 x, y;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[j] = o + half * 16 + h * 8 + j < o_end ? v.w[h * 8 + j] : 0u;
                y[j] = o + half * 16 + h * 8 + 4 + j < o_end ? v.w[h * 8 + 4 + j] : 0u;
            }
            const Parts4 s = split_parts(x), t = split_parts(y);
#pragma unroll
            for (int e = 0; e < 3; ++e)
                *reinterpret_cast<f32x3_u32x4 *>(buf + e * WPLANE + col * 64 + ((((half * 2 + h) ^ (col >> 1)) & 3) << 4)) =
                    f32x3_u32x4{s.p[e][0], s.p[e][1], t.p[e][0], t.p[e][1]};
        }
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const int row = drow + 64 * k;
            f32x3_u32x4 x = __builtin_bit_cast(f32x3_u32x4, v.d[k]);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = o + dseg * 4 + e < o_end ? x[e] : 0u;
            const Parts4 s = split_parts(x);
            if (row < NB * 16)
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    *reinterpret_cast<f32x3_u32x2 *>(buf + 3 * WPLANE + e * DPLANE + row * 64 + ((((dseg >> 1) ^ (row >> 1)) & 3) << 4) + (dseg & 1) * 8) = s.p[e];
        }
    };
    auto frag = [&](const char *plane, int row) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x3_u32x4 *>(plane + row * 64 + (((g ^ (row >> 1)) & 3) << 4)));
    };
    // The step at o: the next one, requested a step ago, goes to the other buffer, and the one beyond it is requested (past the
    // range: its last rows again, staged as zeros and not used).
    Step v;
    auto step = [&](int o, char *buf, char *other) __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // this step's planes are visible, the other buffer is free
        // (each block's dz is read while the block before it is multiplied)
        bf16x8 w[3][2], d[2][3];
        auto read_d = [&](int x) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 3; ++e) d[x & 1][e] = frag(buf + 3 * WPLANE + e * DPLANE, x * 16 + q);
        };
        read_d(0);
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
            for (int y = 0; y < 2; ++y) w[e][y] = frag(buf + e * WPLANE, wv * 32 + y * 16 + q);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            __builtin_amdgcn_sched_barrier(0);
            if (x + 1 < NB) read_d(x + 1);
            __builtin_amdgcn_sched_barrier(0);
            auto terms = [&](f32x4m(&acc)[2], int we, int de) __attribute__((always_inline)) {
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[we][y], d[x & 1][de], acc[y], 0, 0, 0);
            };
            terms(hi[x], 0, 0); terms(lo[x], 0, 1); terms(lo[x], 1, 0); terms(lo[x], 1, 1); terms(lo[x], 0, 2); terms(lo[x], 2, 0);
            if (x == NB / 2) {
                stage(o + 32, v, other);
                request(o + 64, v);
            }
        }
    };
    if (o_begin < o_end) {
        request(o_begin, v);
        stage(o_begin, v, lds);
        request(o_begin + 32, v);
        int cur = 0;
        for (int o = o_begin; o < o_end; o += 32, cur ^= BUF) step(o, lds + cur, lds + (BUF - cur));
    }
    // register e of lane 16 g + q: input 4 g + e of batch row q
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        const int row = row0 + x * 16 + q;
        if (row >= p.N) continue;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int ic = i0 + wv * 32 + y * 16 + 4 * g;
            float *dst = p.part + ((size_t)split * p.N + row) * p.In + ic;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = join_parts(hi[x][y][e], lo[x][y][e]);
            if (wvec) {
                if (ic < p.In) *reinterpret_cast<f32x4 *>(dst) = v;
            } else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ic + e < p.In) dst[e] = v[e];
        }
    }
}

// ------------------------------------ fp32 backward on the bf16 matrix unit, dz in parts ahead (fc_bwd_staged)
// dz in parts (f32x3.h), once per call, in the layouts that the two products' fragments have: per 32 outputs ("step") blocks of
// 1 KB, which a wave's 64 lanes read 16 bytes each, in order.  25088 -> 4096: 6 us, db among them (4.7 alone).  With it the bias gradient, in fc_db_kernel's order.
//   rows (da): [step][16-row block][part], lane 16 g + q: outputs 8 g .. 8 g + 7 of row q
//   cols (dW): [step][16-row block][part], lane 32 k + r: rows 8 k .. 8 k + 7 of output r
// Rows and outputs past the ends are zeros.
__global__ __launch_bounds__(512) void fc_dz_parts_kernel(const float *__restrict__ dz, char *__restrict__ rows, char *__restrict__ cols,
                                                          float *__restrict__ db, int N, int Out, int nb)
{
    const int tid = threadIdx.x, step = blockIdx.x, o0 = step * 32;
    auto store = [&](char *dst, const float(&v)[8]) __attribute__((always_inline)) {
        f32x3_u32x4 x, y;
#pragma unroll
        for (int j = 0; j < 4; ++j) { x[j] = __float_as_uint(v[j]); y[j] = __float_as_uint(v[j + 4]); }
        const Parts4 s = split_parts(x), t = split_parts(y);
#pragma unroll
        for (int e = 0; e < 3; ++e)
            *reinterpret_cast<f32x3_u32x4 *>(dst + e * 1024) = f32x3_u32x4{s.p[e][0], s.p[e][1], t.p[e][0], t.p[e][1]};
    };
    for (int u = tid; u < nb * 128; u += 512) {
        const bool by_row = u < nb * 64;
        const int w = by_row ? u : u - nb * 64;
        const int row = by_row ? w >> 2 : (w >> 5) * 8, o = o0 + (by_row ? (w & 3) * 8 : w & 31);
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = dz[(size_t)min(row + (by_row ? 0 : j), N - 1) * Out + min(o + (by_row ? j : 0), Out - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = row + (by_row ? 0 : j) < N && o + (by_row ? j : 0) < Out ? v[j] : 0.f;
        if (by_row) store(rows + ((size_t)step * nb + (w >> 6)) * 3072 + ((w & 3) * 16 + ((w >> 2) & 15)) * 16, v);
        else store(cols + ((size_t)step * nb + (w >> 6)) * 3072 + (w & 63) * 16, v);
    }
    if (!db) return;
    __shared__ float part[4][32];
    const int col = tid & 31, wv = tid >> 5, o = o0 + col;
    if (wv < 4) {
        float s = 0.f;
        if (o < Out) {
#pragma unroll 8
            for (int n = wv; n < N; n += 4) s += dz[(size_t)n * Out + o];
        }
        part[wv][col] = s;
    }
    __syncthreads();
    if (wv == 0 && o < Out) db[o] = (part[0][col] + part[1][col]) + (part[2][col] + part[3][col]);
}

// The steps of dz that both products walk: 3 NB blocks of 1 KB, copied straight to one of four LDS buffers by the eight waves, three
// steps ahead.  The barrier of a step lies in its middle: it says that the next step's copies are there, so that a step begins, with
// its first fragments read during the one before, without a wait; and that the last step's buffer is free.  Global loads and
// stores of a wave complete in order: "at most n younger ones outstanding" means that a copy is there.
template <int NB>
struct DzSteps {
    static constexpr int BYTES = NB * 3072, BUFFERS = 4;
    const char *src;     // + lane * 16
    unsigned lds;        // of the first buffer
    int wv;
    __device__ __forceinline__ DzSteps(const char *planes, const char *buf)
        : src(planes + (threadIdx.x & 63) * 16),
          lds(__builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)buf)),
          wv(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {}
    __device__ __forceinline__ void copy(int step, int buffer) const
    {
        const char *s = src + (size_t)step * BYTES;
#pragma unroll
        for (int k = 0; k < (3 * NB + 7) / 8; ++k) {
            const int b = wv + 8 * k;
            if (b < 3 * NB) {
                const unsigned dst = __builtin_amdgcn_readfirstlane(lds + (buffer & (BUFFERS - 1)) * BYTES + b * 1024);
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(s + b * 1024) : "m0", "memory");
            }
        }
    }
    template <int YOUNGER> static __device__ __forceinline__ void wait()
    {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(YOUNGER) : "memory");
    }
};
// a buffer of `bytes` bytes at `base`: loads beyond it give zero, stores beyond it are dropped
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, int bytes)
{
    // (the compiler takes some of these for different in every lane, and would loop over them)
    const uintptr_t b = reinterpret_cast<uintptr_t>(base);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>((uintptr_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// dW = dz^T a, up to 128 batch rows; bound by the MFMAs (six per product; pipes busy 0.61 of the time below) and by writing dW.  Eight waves, one workgroup per CU; wave w
// owns inputs 32 w .. 32 w + 31 of a tile of 256, whose batch rows it keeps in registers, split, in the MFMA's layout; 32
// outputs of dz at a time come through LDS.  So a value of the input is split once per tile and workgroup, not once per 128 x 128 block
// of dW, and nothing but MFMAs, fragment reads and stores is left in the loop.  The (tile, 32 outputs) units are shared out evenly.
// Stores: 32 lanes write 128 bytes of a row.  25088 -> 4096, 100 rows: 109 us (196 with both operands split per block), the MFMAs alone 97.
template <int NB>
__global__ __launch_bounds__(512, 2) void fc_dw_parts_kernel(const float *__restrict__ a, const char *__restrict__ cols,
                                                             float *__restrict__ dw, int N, int In, int Out, int units)
{
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, r = lane & 31, kp = lane >> 5;
    const DzSteps<NB> dz(cols, lds);
    const int steps = (Out + 31) / 32;
    const int begin = (int)((long)units * blockIdx.x / gridDim.x), end = (int)((long)units * (blockIdx.x + 1) / gridDim.x);
    if (begin >= end) return;
    int t = begin, tile = begin / steps, s = begin - tile * steps;
    auto next = [&](int v) __attribute__((always_inline)) { return v + 1 == steps ? 0 : v + 1; };
    dz.copy(s, 0);
    if (t + 1 < end) dz.copy(next(s), 1);
    if (t + 2 < end) dz.copy(next(next(s)), 2);
    dz.template wait<0>();
    bf16x8 df[2][3];
    auto read = [&](int unit, int k, bf16x8(&to)[3]) __attribute__((always_inline)) {
        const char *const plane = lds + ((unit - begin) & (DzSteps<NB>::BUFFERS - 1)) * DzSteps<NB>::BYTES + k * 3072 + lane * 16;
#pragma unroll
        for (int e = 0; e < 3; ++e) to[e] = *reinterpret_cast<const bf16x8 *>(plane + e * 1024);
    };
    while (t < end) {
        const int col = tile * 256 + dz.wv * 32 + r;
        bf16x8 af[NB][3];
        {
            // (rows past the end are beyond the buffer: zeros; inputs past the end: other values, never stored)
            f32x3_u32x4 raw[NB][2];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const auto rows = buffer_of(a + (size_t)min(k * 16, N) * In, max(min(16, N - k * 16), 0) * In * 4);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    raw[k][j >> 2][j & 3] = __builtin_amdgcn_raw_buffer_load_b32(rows, (int)((unsigned)col * 4u + (kp * 8 + j) * 4u * In), 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const f32x3_u32x4(&v)[2] = raw[k];
                const Parts4 x = split_parts(v[0]), y = split_parts(v[1]);
#pragma unroll
                for (int e = 0; e < 3; ++e) af[k][e] = __builtin_bit_cast(bf16x8, f32x3_u32x4{x.p[e][0], x.p[e][1], y.p[e][0], y.p[e][1]});
            }
        }
        // (inputs past the end: beyond every buffer below, with any row added)
        const unsigned at = (col < In ? (unsigned)col * 4u : 0x80000000u) + (unsigned)kp * 16u * In;
        // A step multiplies into one set of accumulators while the other set, the step before, is added up and stored between
        // its MFMAs: the waves of a workgroup walk in step, and would leave the matrix unit idle together.
        const int last = min(end, t + steps - s);
        auto store = [&](__amdgpu_buffer_rsrc_t out, const f32x16 &hi, const f32x16 &lo, int e) __attribute__((always_inline)) {
            // (nt: streamed out, 411 MB for the first dense layer)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(join_parts(hi[e], lo[e])), out, (int)(at + ((e >> 2) * 8 + (e & 3)) * 4u * In), 0, 2);
        };
        auto rows_of = [&](int step) __attribute__((always_inline)) { return buffer_of(dw + (size_t)step * 32 * In, min(32, Out - step * 32) * In * 4); };
        auto out = buffer_of(dw, 0);   // of the step before (none: the stores are dropped)
        auto step = [&](f32x16 &hi, f32x16 &lo, const f32x16 &hi0, const f32x16 &lo0, auto odd) __attribute__((always_inline)) {
            constexpr int P = decltype(odd)::value * NB;   // (fragments alternate between two sets of registers, also across steps)
#pragma unroll
            for (int e = 0; e < 16; ++e) hi[e] = lo[e] = 0.f;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                __builtin_amdgcn_sched_barrier(0);
                if (k == NB / 2) {
                    // younger than the next step's copies, three steps old, are the 16 stores of each of the last two steps
                    if (t <= begin + 2) dz.template wait<0>();
                    else dz.template wait<32>();
                    if (t + 3 < end) dz.copy(next(next(next(s))), t + 3 - begin);
                }
                if (k + 1 < NB) read(t, k + 1, df[(k + 1 + P) & 1]);
                else read(t + 1, 0, df[(NB + P) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                auto term = [&](f32x16 &acc, int de, int ae, int m) __attribute__((always_inline)) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df[(k + P) & 1][de], af[k][ae], acc, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (e * (6 * NB) / 16 == k * 6 + m) {
                            store(out, hi0, lo0, e);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                };
                term(lo, 0, 1, 0); term(hi, 0, 0, 1); term(lo, 1, 0, 2); term(lo, 1, 1, 3); term(lo, 0, 2, 4); term(lo, 2, 0, 5);
            }
            out = rows_of(s);
            s = next(s);
            ++t;
        };
        f32x16 hi[2], lo[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) hi[1][e] = lo[1][e] = 0.f;
        read(t, 0, df[0]);
        while (true) {
            step(hi[0], lo[0], hi[1], lo[1], std::integral_constant<int, 0>());
            if (t == last) {
#pragma unroll
                for (int e = 0; e < 16; ++e) store(out, hi[0], lo[0], e);
                break;
            }
            step(hi[1], lo[1], hi[0], lo[0], std::integral_constant<int, 1>());
            if (t == last) {
#pragma unroll
                for (int e = 0; e < 16; ++e) store(out, hi[1], lo[1], e);
                break;
            }
        }
        ++tile;
    }
}

// da = dz W.  Eight waves, one workgroup per CU; 16 NB batch rows x 256 inputs x a range of outputs (the contraction index), 32 at
// a time; bound by the MFMAs (six per product; pipes busy 0.50 of the time below), splitting the weights and streaming them.  A weight is used by one wave only:
// lane 16 g + q loads outputs 8 g .. 8 g + 7 of inputs 2 q and 2 q + 1 of the wave's 32 (128 bytes of four rows per load) straight to
// its register, a step ahead, and splits them between the MFMAs of the step before; dz comes in parts through LDS.  The weights are
// the first operand, so that a lane holds eight neighbouring inputs of a batch row.  25088 -> 4096, 100 rows: 128 us (158 with weights and dz
// split on their way through LDS); 121 with all weights in L2, 117 without splitting.
template <int NB, bool VEC>   // VEC: In is even
__global__ __launch_bounds__(512, 2) void fc_da_parts_kernel(FcDaArgs p, const char *__restrict__ rows)
{
    typedef float f32x4m __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, q = lane & 15, g = lane >> 4, b = blockIdx.x;
    const int ti = b % p.tiles_i, split = b / p.tiles_i;
    const int o_begin = split * p.o_per_split, o_end = min(o_begin + p.o_per_split, p.Out);
    const int begin = o_begin / 32, end = (o_end + 31) / 32;
    const DzSteps<NB> dz(rows, lds);
    const int col = ti * 256 + dz.wv * 32 + 2 * q;

    f32x4m hi[NB][2], lo[NB][2];
#pragma unroll
    for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) hi[x][y] = lo[x][y] = f32x4m{0.f, 0.f, 0.f, 0.f};
    dz.copy(begin, 0);
    if (begin + 1 < end) dz.copy(begin + 1, 1);
    if (begin + 2 < end) dz.copy(begin + 2, 2);
    // Weights: unit u holds rows 2 u, 2 u + 1 of the lane's eight.  Rows past the range are beyond the buffer, zeros (and no traffic);
    // columns past the end read some other weight or zero and are never stored.
    const unsigned at = (unsigned)g * 32u * p.In + (unsigned)col * 4u;
    auto weights = [&](int step) __attribute__((always_inline)) {
        const int o0 = min(step, end) * 32;
        return buffer_of(p.w + (size_t)o0 * p.In, max(min(32, o_end - o0), 0) * p.In * 4);
    };
    unsigned raw[4][4];   // [unit][2 * input + row]
    auto request = [&](__amdgpu_buffer_rsrc_t w, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int off = (int)(at + (2 * u + k) * 4u * p.In);
            if constexpr (VEC) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(w, off, 0, 2);
                raw[u][k] = v[0];
                raw[u][2 + k] = v[1];
            } else {
                raw[u][k] = __builtin_amdgcn_raw_buffer_load_b32(w, off, 0, 2);
                raw[u][2 + k] = __builtin_amdgcn_raw_buffer_load_b32(w, off + 4, 0, 2);
            }
        }
    };
    struct Frag { f32x3_u32x4 v[3][2]; };   // [part][input of the pair]
    auto split_unit = [&](Frag &f, int u) __attribute__((always_inline)) {
        const Parts4 s = split_parts(f32x3_u32x4{raw[u][0], raw[u][1], raw[u][2], raw[u][3]});
#pragma unroll
        for (int e = 0; e < 3; ++e) { f.v[e][0][u] = s.p[e][0]; f.v[e][1][u] = s.p[e][1]; }
    };
    Frag w[2];
    {
        const auto first = weights(begin), second = weights(begin + 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) request(first, u);
#pragma unroll
        for (int u = 0; u < 4; ++u) { split_unit(w[0], u); request(second, u); }
    }
    bf16x8 d[2][3];
    auto read = [&](int step, int x, bf16x8(&to)[3]) __attribute__((always_inline)) {
        const char *const plane = lds + ((step - begin) & (DzSteps<NB>::BUFFERS - 1)) * DzSteps<NB>::BYTES + x * 3072 + lane * 16;
#pragma unroll
        for (int e = 0; e < 3; ++e) to[e] = *reinterpret_cast<const bf16x8 *>(plane + e * 1024);
    };
    int s = begin;
    auto step = [&](const Frag &w, Frag &n, auto odd) __attribute__((always_inline)) {
        constexpr int P = decltype(odd)::value * NB;   // (fragments of dz alternate between two sets of registers, also across steps)
        const auto ahead = weights(s + 2);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            __builtin_amdgcn_sched_barrier(0);
            if (x == NB / 2) {
                // (younger than the next step's copies, three steps old, are the eight weight loads of each of the last two steps)
                if (s <= begin + 2) dz.template wait<0>();
                else dz.template wait<16>();
                if (s + 3 < end) dz.copy(s + 3, s + 3 - begin);
            }
            if (x + 1 < NB) read(s, x + 1, d[(x + 1 + P) & 1]);
            else read(s + 1, 0, d[(NB + P) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            auto terms = [&](f32x4m(&acc)[2], int we, int de) __attribute__((always_inline)) {
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w.v[we][y]), d[(x + P) & 1][de], acc[y], 0, 0, 0);
            };
            terms(hi[x], 0, 0); terms(lo[x], 0, 1); terms(lo[x], 1, 0); terms(lo[x], 1, 1); terms(lo[x], 0, 2); terms(lo[x], 2, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u * NB / 4 == x) { split_unit(n, u); request(ahead, u); }
        }
        ++s;
    };
    dz.template wait<0>();
    read(begin, 0, d[0]);
    while (true) {
        step(w[0], w[1], std::integral_constant<int, 0>());
        if (s >= end) break;
        step(w[1], w[0], std::integral_constant<int, 1>());
        if (s >= end) break;
    }
    // register e of lane 16 g + q, pair member y: input 8 g + 2 e + y of batch row q
    const int ic = ti * 256 + dz.wv * 32 + 8 * g;
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        const int row = x * 16 + q;
        if (row >= p.N) continue;
        float *dst = p.part + ((size_t)split * p.N + row) * p.In + ic;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = join_parts(hi[x][e & 1][e >> 1], lo[x][e & 1][e >> 1]);
        if ((p.In & 3) == 0) {
            if (ic < p.In) store4(dst, v[0], v[1], v[2], v[3]);
            if (ic + 4 < p.In) store4(dst + 4, v[4], v[5], v[6], v[7]);
        } else
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (ic + e < p.In) dst[e] = v[e];
    }
}

// da = (sum over splits) [* (a > 0)], V values per thread (V divides n)
template <int V>
__global__ void fc_da_finish_kernel(const float *__restrict__ part, const float *__restrict__ a, float *__restrict__ da, size_t n,
                                    int splits, int relu_mask)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n / V) return;
    vec s = reinterpret_cast<const vec *>(part)[i];
    for (int k = 1; k < splits; ++k) s += reinterpret_cast<const vec *>(part + (size_t)k * n)[i];
    if (relu_mask) {
        const vec m = reinterpret_cast<const vec *>(a)[i];
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (!(m[v] > 0.f)) s[v] = 0.f;
    }
    reinterpret_cast<vec *>(da)[i] = s;
}

// launch: how many workgroups to aim at.  The workspace query takes 512 rounded up to whole splits of the tiles, the
// launch 512 rounded down: 512 is what two workgroups per CU hold, and 588 instead of 490 (25088 -> 4096) would
// leave a second round of 76.
static void fc_da_plan(int N, int In, int Out, FcDaArgs &a, bool launch)
{
    a.N = N; a.In = In; a.Out = Out;
    a.tiles_i = (In + 255) / 256;
    a.tiles_m = (N + 127) / 128;
    a.nb = ((N + 15) / 16 + a.tiles_m - 1) / a.tiles_m;
    const int tiles = a.tiles_i * a.tiles_m;
    int splits = launch ? 512 / tiles : (512 + tiles - 1) / tiles;
    const int max_splits = (Out + 63) / 64;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    a.o_per_split = ((Out + splits - 1) / splits + 15) / 16 * 16;
}
static int fc_da_splits(const FcDaArgs &a) { return (a.Out + a.o_per_split - 1) / a.o_per_split; }

// dz in parts ahead of both products: 41 to 128 rows (one row tile, since the input's batch rows fill the registers; with two, 0.96 to
// 1.10 of the time of 18 shapes) and 32-bit offsets inside 32 rows of W and dW.  Against the kernels that split dz themselves, same
// bits, over 1968 shapes (25088 -> 4096, batch 100, 355 -> 255 us): up to one (tile, 32 outputs) unit of dW per workgroup 0.76 to 1.01 of the
// time.  With more, splitting dz ahead (3 us) and a tile's first step have to be paid by what those kernels lose, which is little while all
// their blocks of 128 x 128 run at once, two per CU: up to 512 blocks 0.85 to 1.16, 1.01 on average (83 rows, 1360 -> 2496 36 / 41 us).
// Beyond, 0.63 to 0.99 above 64 rows.  With fewer, writing dW counts as much as the MFMAs, and a wave's 128 bytes per row cost more
// where rows do not begin at whole ones: 32 | In 0.70 to 1.01, 16 | In 0.80 to 1.04 (beyond 1024 blocks at most 0.96), other
// multiples of four 0.87 to 1.15 (46 rows, 4296 -> 7526 88 / 101); on other rows those kernels store 4 bytes at a time too, 0.73 to 1.03, one 1.05.
// (25 to 40 rows stay on the fp32 MFMAs, as dW without da does: from 1024 outputs on 0.69 to 1.01 of the time here, but values of 2^-116
// would be 4e-6 off.)
static bool fc_bwd_staged(int N, int In, int Out)
{
    if (N <= 40 || N > 128 || In >= (1 << 24) - 256) return false;
    const long units = (long)((In + 255) / 256) * ((Out + 31) / 32), blocks = (long)((In + 127) / 128) * ((Out + 127) / 128);
    if (units <= 256) return true;
    return blocks > 512 && (N > 64 || In % 4 || In % 32 == 0 || (In % 16 == 0 && blocks > 1024));
}
// bytes of one of the two copies of dz in parts
static size_t fc_dz_parts_bytes(const FcDaArgs &a) { return (size_t)((a.Out + 31) / 32) * a.nb * 3072; }

// least: what a call has to bring, the partial sums of da; with less than the whole, the products split dz themselves.
size_t fc_bwd_workspace(int N, int In, int Out, bool least)
{
    FcDaArgs a;
    fc_da_plan(N, In, Out, a, false);
    return round_up((size_t)fc_da_splits(a) * N * In * 4, 256) + (!least && fc_bwd_staged(N, In, Out) ? 2 * fc_dz_parts_bytes(a) : 0);
}

// The launch of the kernel on the bf16 matrix unit, one workgroup per CU: of the splits that the workspace holds it takes
// the one with the least of rounds over 256 workgroups and partial sums, both in units of streaming the weights.
static void fc_da_parts_plan(int N, int In, int Out, FcDaArgs &a)
{
    fc_da_plan(N, In, Out, a, false);
    const int most = fc_da_splits(a), tiles = a.tiles_i * a.tiles_m;
    int best = 1;
    float least = 0.f;
    for (int s = 1; s <= most; ++s) {
        const float cost = (float)((tiles * (long)s + 255) / 256) * 256.f / ((float)tiles * s) + 2.f * N * s / Out;
        if (s == 1 || cost < least) { best = s; least = cost; }
    }
    a.o_per_split = ((Out + best - 1) / best + 31) / 32 * 32;
}
template <int NB>
static int launch_fc_da_f32x3(const FcDaArgs &p, int splits, hipStream_t s)
{
    if (p.nb != NB) {
        if constexpr (NB > 3) return launch_fc_da_f32x3<NB - 1>(p, splits, s);   // (more than 40 rows: at least three blocks)
        return VGG_ERR_LAUNCH;
    }
    auto kern = p.Out % 4 == 0 ? fc_da_f32x3_kernel<NB, true> : fc_da_f32x3_kernel<NB, false>;
    if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    const size_t lds = (size_t)2 * 3 * (256 + NB * 16) * 64;
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_i * p.tiles_m * splits)), dim3(512), lds, s, p);
    return launch_status();
}

// dz in parts, both products (da: its partial sums), one row tile of three to eight blocks of sixteen.
template <int NB>
static int launch_fc_bwd_parts(const FcDaArgs &p, int splits, const float *a, float *dw, float *db, hipStream_t s)
{
    if constexpr (NB > 3)
        if (p.nb != NB) return launch_fc_bwd_parts<NB - 1>(p, splits, a, dw, db, s);
    const int steps = (p.Out + 31) / 32, units = p.tiles_i * steps;
    char *const rows = reinterpret_cast<char *>(p.part) + round_up((size_t)splits * p.N * p.In * 4, 256), *const cols = rows + fc_dz_parts_bytes(p);
    hipLaunchKernelGGL(fc_dz_parts_kernel, dim3((unsigned)steps), dim3(512), 0, s, p.dz, rows, cols, db, p.N, p.Out, NB);
    const size_t lds = DzSteps<NB>::BUFFERS * DzSteps<NB>::BYTES;
    if (!raise_lds_limit(reinterpret_cast<const void *>(fc_dw_parts_kernel<NB>))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(fc_dw_parts_kernel<NB>, dim3((unsigned)min(units, 256)), dim3(512), lds, s, a, cols, dw, p.N, p.In, p.Out, units);
    auto kern = p.In % 2 == 0 ? fc_da_parts_kernel<NB, true> : fc_da_parts_kernel<NB, false>;
    if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_i * splits)), dim3(512), lds, s, p, rows);
    return launch_status();
}

template <int NB>
static void launch_fc_da(const FcDaArgs &p, int splits, hipStream_t s)
{
    if (p.nb != NB) {
        if constexpr (NB > 1) launch_fc_da<NB - 1>(p, splits, s);
        return;
    }
    const dim3 grid((unsigned)(p.tiles_i * p.tiles_m * splits));
    if (p.In % 4 == 0) hipLaunchKernelGGL((fc_da_kernel<NB, true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((fc_da_kernel<NB, false>), grid, dim3(256), 0, s, p);
}

int fc_backward(int N, int In, int Out, const float *a, const float *w, const float *dz, float *dw, float *db, float *da,
                int relu_mask, void *ws, size_t ws_bytes, hipStream_t s)
{
    const dim3 grid((unsigned)(((In + 127) / 128) * ((Out + 127) / 128)));
    // (the parts of dz lie in the workspace, which is there where da is asked for, behind its partial sums if it holds both)
    const bool staged = da && fc_bwd_staged(N, In, Out) && ws_bytes >= fc_bwd_workspace(N, In, Out, false), parts = N > 40;
    if (!staged) {
        auto dw_kernel = parts ? (In % 4 == 0 ? fc_dw_f32x3_kernel<true> : fc_dw_f32x3_kernel<false>) : (In % 4 == 0 ? fc_dw_kernel<true> : fc_dw_kernel<false>);
        hipLaunchKernelGGL(dw_kernel, grid, dim3(256), 0, s, a, dz, dw, N, In, Out);
        if (db) hipLaunchKernelGGL(fc_db_kernel, dim3((Out + 63) / 64), dim3(256), 0, s, dz, db, N, Out);
    }
    if (da) {
        FcDaArgs p;
        if (parts) fc_da_parts_plan(N, In, Out, p);
        else fc_da_plan(N, In, Out, p, true);
        const int splits = fc_da_splits(p);
        p.dz = dz; p.w = w; p.part = static_cast<float *>(ws);
        if (parts) {
            const int rc = staged ? launch_fc_bwd_parts<8>(p, splits, a, dw, db, s) : launch_fc_da_f32x3<8>(p, splits, s);
            if (rc) return rc;
        } else launch_fc_da<3>(p, splits, s);   // (up to 40 rows: three blocks of sixteen)
        const size_t n = (size_t)N * In;
        if (In % 4 == 0)
            hipLaunchKernelGGL(fc_da_finish_kernel<4>, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, s, p.part, a, da, n, splits, relu_mask);
        else
            hipLaunchKernelGGL(fc_da_finish_kernel<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p.part, a, da, n, splits, relu_mask);
    }
    return launch_status();
}

// =========================================================================
// bf16 operands (activations and weights bf16, dz rounded to bf16, fp32 sums and fp32 results): the
// matrix-unit numerics of the paper's accelerator applied to the dense layers' backward products.
//
// Both products contract over an index that is NOT the contiguous one of its operands in memory
// (dW: the batch index of dz[n][o] and a[n][i]; dA: the output index of W[o][i]), while
// v_mfma_f32_32x32x16_bf16 wants eight consecutive contraction indices per lane.  The tiles are staged
// in LDS as they lie in memory and the fragments are fetched with the LDS transpose read
// ds_read_b64_tr_b16 (within 16 lanes, lane i receives element i%4 of the 8-byte chunks that lanes
// i/4, i/4+4, i/4+8, i/4+12 point at: lane s points at contraction index s/4 and channel chunk s%4, so
// lane i ends up with four consecutive contraction indices of channel i).  LDS rows are 288 bytes
// (128 channels + 32 bytes of padding): four consecutive rows start 32 bytes apart in the banks.
// =========================================================================
namespace {

constexpr int kTrRow = 288;

__device__ __forceinline__ bf16x8 fc_tr_fragment(const char *lds_lo, const char *lds_hi)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4 *lp;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)lds_lo);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)lds_hi);
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// byte offset of this lane's chunk inside a 16-row x 32-channel block of a staged tile
__device__ __forceinline__ int fc_tr_lane_offset()
{
    const int lane = threadIdx.x & 63, G = lane >> 4, i = lane & 15;
    return (8 * (G >> 1) + (i >> 2)) * kTrRow + (G & 1) * 32 + (i & 3) * 8;
}

constexpr int kDwRows = 64;   // batch rows per pass of the dW kernel: four MFMA steps, 2 x 64 x 288 bytes of LDS (four workgroups per CU)

// dW = dz^T * a.  Workgroup: 128 (o) x 128 (i) block of dW; wave (wo, wi) owns a 64 x 64 sub-block = 2 x 2 MFMA
// tiles; input 2 r + y of its 64 lies in column r of tile y, so that a lane stores two neighbouring inputs.  dzb: dz rounded to
// bf16, rows of OutP >= Out + 7 elements (a multiple of 8), zeros beyond Out.
// UPDATE: instead of dW, the weights' step: the fp32 master values, requested before anything else so that the contraction
// hides their latency, take theta - lr dW, the bf16 copy is refreshed; the gradient is never in memory (10 bytes per weight
// instead of 18: bf16 training step of 32 images 4537 -> 4355 us, of two at 160x160 1360 -> 1251; with the master values requested in
// the epilogue every short workgroup waited for them and the update apart was faster).
template <bool UPDATE>
__global__ __launch_bounds__(256) void fc_dw_bf16_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ dzb,
                                                            float *__restrict__ dw, int N, int In, int Out, int OutP, float lr,
                                                            bf16_t *__restrict__ copy)
{
    __shared__ __align__(16) char Ds[kDwRows * kTrRow];
    __shared__ __align__(16) char As[kDwRows * kTrRow];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    const int wo = wv & 1, wi = wv >> 1;
    const int tiles_i = (In + 127) / 128;
    const int i0 = (blockIdx.x % tiles_i) * 128, o0 = (blockIdx.x / tiles_i) * 128;
    const int loff = fc_tr_lane_offset();

    f32x16 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const int ic = i0 + wi * 64 + 2 * r;                  // (In is even: the pair is inside or outside as one)
    auto out_row = [&](int x, int e) __attribute__((always_inline)) { return o0 + wo * 64 + x * 32 + (e >> 2) * 8 + kp * 4 + (e & 3); };
    f32x2_t theta[UPDATE ? 2 : 1][16];
    if constexpr (UPDATE) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                theta[x][e] = __builtin_nontemporal_load(reinterpret_cast<const f32x2_t *>(dw + (size_t)min(out_row(x, e), Out - 1) * In + min(ic, In - 2)));
    }

    for (int n0 = 0; n0 < N; n0 += kDwRows) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (not the loads in flight)
        // sixteen segments of eight outputs or inputs per row, all of a pass requested before the first is stored and without
        // conditions; past the ends the last ones again: rows become zeros, the others are not stored (In is a multiple of 8)
        const int seg = tid & 15, row_t = tid >> 4;
        fc_u32x4 vd[kDwRows / 16], va[kDwRows / 16];
#pragma unroll
        for (int q = 0; q < kDwRows / 16; ++q) {
            const size_t n = min(n0 + row_t + 16 * q, N - 1);
            vd[q] = *reinterpret_cast<const fc_u32x4 *>(dzb + n * OutP + min(o0 + seg * 8, OutP - 8));
            va[q] = *reinterpret_cast<const fc_u32x4 *>(a + n * In + min(i0 + seg * 8, In - 8));
        }
#pragma unroll
        for (int q = 0; q < kDwRows / 16; ++q) {
            const int row = row_t + 16 * q;
            const bool in = n0 + row < N;
            *reinterpret_cast<fc_u32x4 *>(Ds + row * kTrRow + seg * 16) = in ? vd[q] : fc_u32x4{0, 0, 0, 0};
            const fc_u32x4 x = in ? va[q] : fc_u32x4{0, 0, 0, 0};
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            char *dst = As + row * kTrRow + (seg >> 3) * 128 + (seg & 7) * 8;   // inputs 0, 2, 4, 6 of the segment; 1, 3, 5, 7 64 bytes on
            *reinterpret_cast<u32x2 *>(dst) = u32x2{__builtin_amdgcn_perm(x[1], x[0], 0x05040100u), __builtin_amdgcn_perm(x[3], x[2], 0x05040100u)};
            *reinterpret_cast<u32x2 *>(dst + 64) = u32x2{__builtin_amdgcn_perm(x[1], x[0], 0x07060302u), __builtin_amdgcn_perm(x[3], x[2], 0x07060302u)};
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int steps = min(kDwRows, N - n0 + 15) / 16;
        for (int s = 0; s < steps; ++s) {
            bf16x8 df[2], af[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const char *q = Ds + loff + (2 * wo + x) * 64 + 16 * s * kTrRow;
                df[x] = fc_tr_fragment(q, q + 4 * kTrRow);
            }
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const char *q = As + loff + (2 * wi + y) * 64 + 16 * s * kTrRow;
                af[y] = fc_tr_fragment(q, q + 4 * kTrRow);
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df[x], af[y], acc[x][y], 0, 0, 0);
        }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int o = out_row(x, e);
            if (o >= Out || ic >= In) continue;
            f32x2_t v = {acc[x][0][e], acc[x][1][e]};
            f32x2_t *dst = reinterpret_cast<f32x2_t *>(dw + (size_t)o * In + ic);
            if constexpr (UPDATE) {
                v = f32x2_t{sgd_step(theta[x][e][0], v[0], lr), sgd_step(theta[x][e][1], v[1], lr)};
                typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
                *reinterpret_cast<unsigned *>(copy + (size_t)o * In + ic) = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
            }
            __builtin_nontemporal_store(v, dst);
        }
}

// dz fp32 [N][Out] -> bf16 [N][OutP] with zeros in the padding columns, and its column sums db (if wanted), as fc_db_kernel
// forms them; one launch for both.
__global__ __launch_bounds__(256) void fc_dz_to_bf16_kernel(const float *__restrict__ dz, bf16_t *__restrict__ out, float *__restrict__ db,
                                                            int N, int Out, int OutP)
{
    __shared__ float part[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int o = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (o < OutP) {
#pragma unroll 16
        for (int n = wv; n < N; n += 4) {
            const float v = o < Out ? dz[(size_t)n * Out + o] : 0.f;
            s += v;
            out[(size_t)n * OutP + o] = f32_to_bf16(v);
        }
    }
    part[wv][lane] = s;
    __syncthreads();
    if (db && wv == 0 && o < Out) db[o] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

struct FcDaBf16Args {
    const bf16_t *dzb;  // [N][OutP], zeros beyond Out
    const bf16_t *w;    // [Out][In]
    float *part;        // [splits][N][In]
    int N, In, Out, OutP;
    int tiles_i, tiles_m, o_per_split;
};

// dA = dz * W.  Workgroup: 32 MB batch rows x 128 inputs x a range of outputs (the contraction index), 64 at a time; bound by
// streaming W.  Wave w owns inputs [32w, 32w+32) and all row blocks.  Weights and dz (rows of 64 outputs = 128 bytes and 16 of
// padding) of the next step are requested while the current one is multiplied, without conditions (a load under one is waited
// for where it ends); dz goes through LDS, as all four waves need it (fetched by each from L2 it was four times the weights'
// bytes).  Whole backward calls, 25088 -> 4096: batch 32 160 -> 139 us, batch 100 218 -> 172; 4096 -> 4096, batch 32 43 -> 31.5; 180
// sizes up to 128 rows 0.73 (one row) to 0.91 (128) on average.
template <int MB>
__global__ __launch_bounds__(256) void fc_da_bf16_kernel(FcDaBf16Args p)
{
    constexpr int kDzRow = 128 + 16;
    __shared__ __align__(16) char Ws[64 * kTrRow];
    __shared__ __align__(16) char Ds[MB * 32 * kDzRow];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 31, kp = lane >> 5;
    int b = blockIdx.x;
    const int ti = b % p.tiles_i; b /= p.tiles_i;
    const int tm = b % p.tiles_m; b /= p.tiles_m;
    const int split = b;
    const int row0 = tm * MB * 32, i0 = ti * 128;
    const int o_begin = split * p.o_per_split, o_end = min(o_begin + p.o_per_split, p.Out);
    const int loff = fc_tr_lane_offset() + wv * 64;

    f32x16 acc[MB];
#pragma unroll
    for (int x = 0; x < MB; ++x)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[x][e] = 0.f;

    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // weights: eight inputs of rows tid / 16 + 16 q; dz: eight outputs of batch rows tid / 8 + 32 q.  (Inputs, outputs and batch
    // rows past the ends: the last ones again; weight rows past the range become zeros, dz is zero there, the rest is not stored.)
    const int wseg = tid & 15, wrow = tid >> 4, dseg = tid & 7, drow = tid >> 3;
    const bf16_t *const wcol = p.w + min(i0 + wseg * 8, p.In - 8);
    fc_u32x4 vw[4], vd[MB];
    auto request = [&](int o) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) vw[q] = *reinterpret_cast<const fc_u32x4 *>(wcol + (size_t)min(o + wrow + 16 * q, p.Out - 1) * p.In);
#pragma unroll
        for (int q = 0; q < MB; ++q)
            vd[q] = *reinterpret_cast<const fc_u32x4 *>(p.dzb + (size_t)min(row0 + drow + 32 * q, p.N - 1) * p.OutP + min(o + dseg * 8, p.OutP - 8));
    };
    if (o_begin < o_end) request(o_begin);
    for (int o = o_begin; o < o_end; o += 64) {
        barrier();  // the previous step's fragment reads are done
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<fc_u32x4 *>(Ws + (wrow + 16 * q) * kTrRow + wseg * 16) = o + wrow + 16 * q < o_end ? vw[q] : fc_u32x4{0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < MB; ++q) *reinterpret_cast<fc_u32x4 *>(Ds + (drow + 32 * q) * kDzRow + dseg * 16) = vd[q];
        barrier();  // the staged rows are visible
        request(o + 64);   // (past the range: not used)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const char *q = Ws + loff + 16 * ks * kTrRow;
            const bf16x8 wf = fc_tr_fragment(q, q + 4 * kTrRow);
#pragma unroll
            for (int x = 0; x < MB; ++x) {
                const bf16x8 df = __builtin_bit_cast(bf16x8, *reinterpret_cast<const fc_u32x4 *>(Ds + (x * 32 + r) * kDzRow + ks * 32 + kp * 16));
                acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df, wf, acc[x], 0, 0, 0);
            }
        }
    }
    const int i = i0 + wv * 32 + r;
    if (i < p.In) {
#pragma unroll
        for (int x = 0; x < MB; ++x)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int n = row0 + x * 32 + (e >> 2) * 8 + kp * 4 + (e & 3);
                if (n < p.N) p.part[((size_t)split * p.N + n) * p.In + i] = acc[x][e];
            }
    }
}

// da = (sum over splits) [* (a > 0)], a in bf16
__global__ void fc_da_bf16_finish_kernel(const float *__restrict__ part, const bf16_t *__restrict__ a, float *__restrict__ da,
                                         size_t n, int splits, int relu_mask)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < splits; ++k) s += part[(size_t)k * n + i];
    if (relu_mask && !(bf16_to_f32(a[i]) > 0.f)) s = 0.f;
    da[i] = s;
}

void fc_da_bf16_plan(int N, int In, int Out, FcDaBf16Args &a)
{
    a.N = N; a.In = In; a.Out = Out;
    a.OutP = (Out + 31) / 32 * 32 + 32;   // a fragment load may start up to 24 columns before the end of the last chunk
    a.tiles_i = (In + 127) / 128;
    a.tiles_m = (N + 127) / 128;
    const int tiles = a.tiles_i * a.tiles_m;
    int splits = (768 + tiles - 1) / tiles;
    const int max_splits = (Out + 63) / 64;
    if (splits > max_splits) splits = max_splits;
    if (splits < 1) splits = 1;
    a.o_per_split = ((Out + splits - 1) / splits + 63) / 64 * 64;
}
int fc_da_bf16_splits(const FcDaBf16Args &a) { return (a.Out + a.o_per_split - 1) / a.o_per_split; }

}  // namespace

size_t fc_bwd_bf16_workspace(int N, int In, int Out)
{
    FcDaBf16Args a;
    fc_da_bf16_plan(N, In, Out, a);
    return round_up((size_t)N * a.OutP * 2, 256) + round_up((size_t)fc_da_bf16_splits(a) * N * In * 4, 256);
}

// a [N][In] bf16, w [Out][In] bf16, dz [N][Out] fp32 -> dw [Out][In] fp32, db [Out] fp32 (may be null),
// da [N][In] fp32 (may be null; optionally masked by a > 0).  In must be a multiple of 8.
// copy (optional, with lr): dw holds the fp32 master weights, which take the step theta - lr * gradient in place of receiving
// the gradient, and copy, [Out][In] bf16, is rounded from them; it may be w, which the data gradient has read by then.
int fc_backward_bf16(int N, int In, int Out, const bf16_t *a, const bf16_t *w, const float *dz, float *dw, float *db, float *da,
                     int relu_mask, void *ws, hipStream_t s, float lr, bf16_t *copy)
{
    FcDaBf16Args p;
    fc_da_bf16_plan(N, In, Out, p);
    bf16_t *dzb = static_cast<bf16_t *>(ws);
    const size_t nd = (size_t)N * p.OutP;
    hipLaunchKernelGGL(fc_dz_to_bf16_kernel, dim3((unsigned)((p.OutP + 63) / 64)), dim3(256), 0, s, dz, dzb, db, N, Out, p.OutP);
    if (da) {
        const int splits = fc_da_bf16_splits(p);
        p.dzb = dzb; p.w = w;
        p.part = reinterpret_cast<float *>(static_cast<char *>(ws) + round_up(nd * 2, 256));
        const int mb = N > 96 ? 4 : (N + 31) / 32;
        auto da_kernel = mb == 1 ? fc_da_bf16_kernel<1> : mb == 2 ? fc_da_bf16_kernel<2> : mb == 3 ? fc_da_bf16_kernel<3> : fc_da_bf16_kernel<4>;
        hipLaunchKernelGGL(da_kernel, dim3((unsigned)(p.tiles_i * p.tiles_m * splits)), dim3(256), 0, s, p);
        const size_t n = (size_t)N * In;
        hipLaunchKernelGGL(fc_da_bf16_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p.part, a, da, n,
                           splits, relu_mask);
    }
    const dim3 grid((unsigned)(((In + 127) / 128) * ((Out + 127) / 128)));
    if (copy) hipLaunchKernelGGL(fc_dw_bf16_kernel<true>, grid, dim3(256), 0, s, a, dzb, dw, N, In, Out, p.OutP, lr, copy);
    else hipLaunchKernelGGL(fc_dw_bf16_kernel<false>, grid, dim3(256), 0, s, a, dzb, dw, N, In, Out, p.OutP, 0.f, nullptr);
    return launch_status();
}

}  // namespace vgg
