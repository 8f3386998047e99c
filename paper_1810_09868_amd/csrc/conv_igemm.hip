// Implicit-GEMM 3x3 stride-1 pad-1 convolution on MFMA for gfx950, NHWC.
//
// GEMM view: rows = output pixels m = (n,h,w) flattened, columns = output
// channels, contraction index = (tap, input channel).  The forward
// convolution (appendix table row "convolution") and the data-gradient
// convolution (rows "reverse" + "convolution" of the backward column) both run
// through this kernel; they differ only in how the weights were packed.
//
// Staging.  A workgroup owns one tile of BM output pixels (see TileGeom:
// either BM consecutive pixels or a 16x16 patch) and BN output channels.  The
// tile's input halo is staged in LDS once per channel chunk, with zeros where
// the halo leaves the image, and is then read by all nine taps, so zero
// padding and image boundaries inside a tile need no masks.
//
// Every LDS row holds 64 bytes of one pixel's channels (16 fp32 or 32 bf16).
// Two row layouts keep the 16-byte fragment reads of consecutive rows on
// distinct banks: rows padded to 80 bytes (the register-staged kernel below,
// and the halo of the 8-wave direct-to-LDS kernel with up to 384 halo rows),
// or unpadded 64-byte rows whose 16-byte segments are XOR-swizzled with the
// row number (all weight rows of the direct-to-LDS kernels, and the halo of
// their other variants).  A lane reads 16 bytes of A and of B at the same
// (k-group, k-half) position: for bf16 that is the 8-element operand of one
// v_mfma_f32_32x32x16_bf16; for fp32 the four elements feed four
// v_mfma_f32_32x32x2_f32 (any fixed pairing of k indices between A and B is a
// valid contraction order).
#include "conv_tile.h"

namespace vgg {

template <typename T, int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(WM *WN * 64, WM *WN == 8 ? 4 : 2) void conv3x3_igemm_kernel(ConvArgs p)
{
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM / 32;  // 32x32 MFMA tiles per wave along pixels
    constexpr int TN = BN / WN / 32;  // and along channels
    constexpr int KC = kDataBytes / (int)sizeof(T);

    extern __shared__ __align__(16) char smem[];
    const int S = p.g.S;
    const int SA = p.rowsA;                     // rows reserved for the halo (>= S)
    int *pix = reinterpret_cast<int *>(smem);   // [SA] halo row -> input pixel or -1
    char *As = smem + round_up16(SA * 4);              // [SA][80]
    char *Bs = As + (size_t)SA * kRowBytes;            // [3][BN][80]

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int wm = wv % WM, wn = wv / WM;
    const int r = lane & 31, khalf = lane >> 5;

    const int tile_n = blockIdx.x % p.tiles_n;
    const int tile_m = blockIdx.x / p.tiles_n;
    const int n0 = tile_n * BN;
    const TileOrigin org = tile_origin(p.g, tile_m);
    const int pitch = p.g.pitch;

    for (int i = tid; i < SA; i += NT) pix[i] = i < S ? halo_pixel(p.g, org, i) : -1;

    // LDS byte offset (for tap (0,0)) of each of this lane's pixel rows
    int abase[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int m, hrow;
        tile_row(p.g, org, wm * (BM / WM) + i * 32 + r, m, hrow);
        abase[i] = hrow * kRowBytes + khalf * 16;
    }
    int bbase[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bbase[j] = (wn * (BN / WN) + j * 32 + r) * kRowBytes + khalf * 16;

    f32x16 acc[TM][TN];
    init_acc<BN, WN>(acc, p, n0, wn, khalf);

    const size_t xrow = (size_t)p.CinP * sizeof(T);
    const int nA = S * 4;  // 16-byte segments of the halo per chunk
    constexpr int NB = 3 * BN * 4 / NT;  // 16-byte weight segments per thread and stage
    constexpr int MAXA = kMaxAHaloSegsPerBlock / NT;  // halo segments per thread prefetched through registers
    const bool a_regs = nA <= MAXA * NT; // then SA == MAXA*NT/4: every thread copies exactly MAXA segments
    const int nstages = (p.CinP / KC) * 3;

    // Global -> register halves of the staging copies.  A stage is (channel chunk, kernel row): it
    // needs the three taps' weights of that row and, when the chunk changes, a new halo.
    // (branch-free: a pad row reads from a block of zeros instead of the tensor)
    auto load_a = [&](int c0, u32x4(&areg)[MAXA]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MAXA; ++j) {
            const int idx = tid + j * NT;
            const int off = pix[idx >> 2];
            const char *src = off < 0 ? reinterpret_cast<const char *>(kZeroRow)
                                      : p.x + (size_t)off * xrow + (size_t)c0 * sizeof(T);
            areg[j] = *reinterpret_cast<const u32x4 *>(src + (idx & 3) * 16);
        }
    };
    auto store_a = [&](const u32x4(&areg)[MAXA], char *As) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MAXA; ++j) {
            const int idx = tid + j * NT;
            *reinterpret_cast<u32x4 *>(As + (idx >> 2) * kRowBytes + (idx & 3) * 16) = areg[j];
        }
    };
    auto copy_a_direct = [&](int c0, char *As) __attribute__((always_inline)) {  // halo too large for the register path
        for (int idx = tid; idx < nA; idx += NT) {
            const int off = pix[idx >> 2];
            u32x4 v = {0u, 0u, 0u, 0u};
            if (off >= 0)
                v = *reinterpret_cast<const u32x4 *>(p.x + (size_t)off * xrow + (size_t)c0 * sizeof(T) + (idx & 3) * 16);
            *reinterpret_cast<u32x4 *>(As + (idx >> 2) * kRowBytes + (idx & 3) * 16) = v;
        }
    };
    auto load_b = [&](int c0, int kh, u32x4(&breg)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int idx = tid + j * NT;
            const int row = idx >> 2;  // kw*BN + n
            const int kw = row / BN;
            const int n = min(n0 + row - kw * BN, p.Cout - 1);  // columns past Cout are never stored
            breg[j] = *reinterpret_cast<const u32x4 *>(p.w + packed_w_segment<T>(kh * 3 + kw, n, c0, idx & 3, p.Cout, p.CinP));
        }
    };
    auto store_b = [&](const u32x4(&breg)[NB], char *Bs) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int idx = tid + j * NT;
            *reinterpret_cast<u32x4 *>(Bs + (idx >> 2) * kRowBytes + (idx & 3) * 16) = breg[j];
        }
    };

    u32x4 areg[MAXA], breg[NB];
    __syncthreads();  // halo table ready
    if (a_regs) { load_a(0, areg); store_a(areg, As); } else copy_a_direct(0, As);
    load_b(0, 0, breg);
    store_b(breg, Bs);
    __syncthreads();
    spread_acc(acc);

    auto compute = [&](int kh, const char *As, const char *Bs) __attribute__((always_inline)) {
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
            const int toff = (kh * pitch + kw) * kRowBytes;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                uint4 af[TM], bf[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    af[i] = *reinterpret_cast<const uint4 *>(As + abase[i] + toff + g * 32);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    bf[j] = *reinterpret_cast<const uint4 *>(Bs + kw * BN * kRowBytes + bbase[j] + g * 32);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) Mma<T>::run(acc[i][j], bf[j], af[i]);
            }
        }
    };

    // Software pipeline: the global loads of stage s+1 are issued before the MFMAs of stage s and
    // land in LDS after them (two barriers per stage), so their latency is covered by the arithmetic.
    int kh = 0, c0 = 0;
    for (int s = 0; s + 1 < nstages; ++s) {
        int nkh = kh + 1, nc0 = c0;
        if (nkh == 3) { nkh = 0; nc0 += KC; }
        const bool new_chunk = nkh == 0;
        load_b(nc0, nkh, breg);
        if (new_chunk && a_regs) load_a(nc0, areg);
        compute(kh, As, Bs);
        __syncthreads();  // every wave is done reading this stage's LDS data
        store_b(breg, Bs);
        if (new_chunk) {
            if (a_regs) store_a(areg, As); else copy_a_direct(nc0, As);
        }
        __syncthreads();
        kh = nkh; c0 = nc0;
    }
    compute(kh, As, Bs);

    conv_epilogue<T, BM, BN, WM, WN>(acc, p, org, smem, n0);
}

// ---------------------------------------------------------------------------
// Variant with direct-to-LDS weight loads.  Weight rows in LDS are 64 bytes
// without padding; the 16-byte segment s of row q lives at segment
// s ^ ((q >> 2) & 3), which keeps the fragment reads of 16 consecutive rows on
// distinct banks (halo rows likewise, or padded to 80 bytes where LDS allows).
// The weights of a stage are copied by global_load_lds_dwordx4 (lane l of a
// wave writes bytes [16 l, 16 l + 16) of a 1 KB block, so each lane fetches the
// segment that belongs at its position) into one of two buffers while the
// MFMAs of the previous stage run: no registers, no ds_write, one barrier per
// stage.  The kernel waits for these loads itself (s_waitcnt vmcnt(0) before
// the barrier that publishes a buffer).  The halo still goes through registers once per channel chunk.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int swz(int row) { return (row >> 2) & 3; }

template <typename T, int BM, int BN, int WM, int WN, int SA>
// (the second launch bound is the minimum number of waves per SIMD: two 8-wave or three 4-wave workgroups per CU)
__global__ __launch_bounds__(WM *WN * 64, WM *WN == 8 ? 4 : 3) void conv3x3_igemm_dma_kernel(ConvArgs p)
{
    constexpr int NT = WM * WN * 64, NW = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int KC = kDataBytes / (int)sizeof(T);
    // SA: halo rows reserved in LDS (host guarantees S <= SA)
    constexpr int SEGS = SA * 4;                    // 16-byte halo segments per chunk
    constexpr int MAXA = (SEGS + NT - 1) / NT;      // of which each thread copies at most MAXA
    constexpr int b_bytes = 3 * BN * kDataBytes;
    // Halo rows of the 8-wave kernel with the smaller halo are padded to 80 bytes instead of swizzled:
    // conflict-free as well, and linear, so every tap of a fragment read is the same per-lane
    // address plus an immediate offset (the other variants have no LDS left for the padding).
    constexpr bool APAD = SA == kDmaHaloRows && NW == 8;
    constexpr int AROW = APAD ? kRowBytes : kDataBytes;
    constexpr int NB = 3 * BN / 16 / NW;            // 1 KB blocks of a weight stage per wave
    static_assert(3 * BN % (16 * NW) == 0 && BN % 16 == 0, "weight stage must split into whole 1 KB blocks");

    extern __shared__ __align__(16) char smem[];
    const int S = p.g.S;
    int *pix = reinterpret_cast<int *>(smem);       // [SA]
    char *As = smem + SA * 4;                        // [SA][64]
    char *Bs = As + SA * AROW;                       // [2][3*BN][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int wm = wv % WM, wn = wv / WM;
    const int r = lane & 31, khalf = lane >> 5;
    // Workgroup b runs on XCD b % 8 and every XCD has its own L2.  Renumber so that each XCD works
    // through one contiguous range of (pixel tile, column tile) pairs: the column tiles of a pixel
    // tile then share the halo, and neighbouring pixel tiles their overlap, in one L2.
    const int nblk = gridDim.x, xcd = blockIdx.x & 7;
    const int bid = xcd * (nblk >> 3) + min(xcd, nblk & 7) + (blockIdx.x >> 3);
    // (split contraction: the ksplit workgroups of a tile are neighbours)
    const int split = bid % p.ksplit, tile = bid / p.ksplit;
    const int tile_n = tile % p.tiles_n;
    const int tile_m = tile / p.tiles_n;
    const int c_first = split * p.kchunks * KC;                    // this workgroup's channel range
    const int c_end = min(c_first + p.kchunks * KC, p.CinP);
    const int n0 = tile_n * BN;
    const TileOrigin org = tile_origin(p.g, tile_m);
    const int pitch = p.g.pitch;

    // This lane's part of the weight stage (c0, kh): NB blocks of 16 rows x 64 bytes.  The per-lane
    // byte offsets inside a kernel row's weights never change; the stage only moves a scalar base.
    unsigned woff[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int row = (wv * NB + q) * 16 + (lane >> 2);   // kw*BN + n
        const int kw = row / BN;
        const int n = min(n0 + row - kw * BN, p.Cout - 1);  // columns past Cout are never stored
        // (offset of this lane's source segment from that of tap (kh, 0), row 0, column c0, segment 0)
        woff[q] = (unsigned)(packed_w_segment<T>(kw, n, 0, (lane & 3) ^ swz(row), p.Cout, p.CinP));
    }
    const unsigned bs_lds = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)(Bs + wv * NB * 1024));
    auto dma_b = [&](int c0, int kh, int buf) __attribute__((always_inline)) {
        const char *base = p.w + packed_w_segment<T>(kh * 3, 0, c0, 0, p.Cout, p.CinP);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            // Issued as inline assembly on purpose: the compiler cannot tell that this write and the
            // fragment reads of the other buffer never overlap and would wait for it before every read.
            const unsigned dst = bs_lds + buf * b_bytes + q * 1024;
            asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(woff[q]), "s"(base) : "m0", "memory");
        }
    };
    dma_b(c_first, 0, 0);  // first: its latency covers the index arithmetic below

    for (int i = tid; i < SA; i += NT) pix[i] = i < S ? halo_pixel(p.g, org, i) : -1;

    int arow[TM];   // halo row of tap (0,0) of this lane's pixels; padded layout: its byte address
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int m;
        tile_row(p.g, org, wm * (BM / WM) + i * 32 + r, m, arow[i]);
        if (APAD) arow[i] = arow[i] * AROW + khalf * 16;
    }
    int baddr[2][TN];  // per k-group; tap kw adds kw*BN*64
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int row = wn * (BN / WN) + j * 32 + r;
        baddr[0][j] = row * kDataBytes + ((khalf ^ swz(row)) << 4);
        baddr[1][j] = baddr[0][j] ^ 32;
    }

    f32x16 acc[TM][TN];
    init_acc<BN, WN>(acc, p, n0, wn, khalf);

    const size_t xrow = (size_t)p.CinP * sizeof(T);
    // Input pixel (or -1 for a pad row) behind each of this thread's halo segments; global, not
    // generic, loads so that they neither touch the LDS counters nor look like LDS accesses.
    typedef const __attribute__((address_space(1))) u32x4 *gvec_t;
    __syncthreads();  // halo table ready
    auto load_a = [&](int c0, u32x4(&areg)[MAXA]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MAXA; ++j) {
            const int idx = min(tid + j * NT, SEGS - 1);
            const int px = pix[idx >> 2];  // read again for every chunk: cheaper than MAXA registers held across the loop
            const gvec_t src = px < 0 ? (gvec_t)kZeroRow : (gvec_t)(p.x + (size_t)px * xrow + (size_t)c0 * sizeof(T));
            areg[j] = src[idx & 3];
        }
    };
    auto store_a = [&](const u32x4(&areg)[MAXA]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MAXA; ++j) {
            const int idx = tid + j * NT;
            const int row = idx >> 2;
            if ((j + 1) * NT <= SEGS || idx < SEGS)
                *reinterpret_cast<u32x4 *>(As + row * AROW + (APAD ? (idx & 3) << 4 : ((idx & 3) ^ swz(row)) << 4)) = areg[j];
        }
    };
    auto compute = [&](int kh, const char *Bt) __attribute__((always_inline)) {
        const char *arow_kh[TM];  // padded layout: this stage's kernel row, once per stage
        if (APAD) {
#pragma unroll
            for (int i = 0; i < TM; ++i) arow_kh[i] = As + arow[i] + kh * pitch * AROW;
        }
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
            int aaddr[TM];
            if (!APAD) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int row = arow[i] + kh * pitch + kw;
                    aaddr[i] = row * kDataBytes + ((khalf ^ swz(row)) << 4);
                }
            }
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                uint4 af[TM], bf[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    af[i] = APAD ? *reinterpret_cast<const uint4 *>(arow_kh[i] + kw * AROW + g * 32)
                                 : *reinterpret_cast<const uint4 *>(As + (aaddr[i] ^ (g * 32)));
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    bf[j] = *reinterpret_cast<const uint4 *>(Bt + kw * BN * kDataBytes + baddr[g][j]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) Mma<T>::run(acc[i][j], bf[j], af[i]);
            }
        }
    };

    u32x4 areg[MAXA];
    load_a(c_first, areg);
    store_a(areg);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the direct-to-LDS loads have landed
    __syncthreads();
    spread_acc(acc);

    // Software pipeline over the stages.  Weight copies for the next stage go to the buffer that was
    // last read two stages ago; the next chunk's halo is requested at the first stage of a chunk and
    // stored to LDS after its last.
    const int nstages = ((c_end - c_first) / KC) * 3;
    int kh = 0, c0 = c_first, bb = 0;
    for (int s = 0; s + 1 < nstages; ++s) {
        int nkh = kh + 1, nc0 = c0;
        if (nkh == 3) { nkh = 0; nc0 += KC; }
        dma_b(nc0, nkh, bb ^ 1);
        if (kh == 0 && c0 + KC < c_end) load_a(c0 + KC, areg);
        compute(kh, Bs + bb * b_bytes);
        if (nkh == 0) {
            __syncthreads();  // every wave is done reading the halo of this chunk
            store_a(areg);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the weight copies have landed
        __syncthreads();
        kh = nkh; c0 = nc0; bb ^= 1;
    }
    compute(kh, Bs + bb * b_bytes);

    if (p.part) conv_partial_epilogue<BM, BN, WM, WN>(acc, p, org, n0, split);
    else conv_epilogue<T, BM, BN, WM, WN>(acc, p, org, smem, n0);
}

// ---------------------------------------------------------------------------
// bf16 variant with the weight fragments in registers.  The blocked weight layout (packed_w_index)
// keeps the 16 contraction indices of a block contiguous per output channel (32 bytes), so a wave loads
// its weight fragments straight from global memory (L2), two taps ahead, into a small ring of
// registers; LDS holds only the input halo.  Compared with the kernel above this removes the weights
// from LDS traffic (half the fragment reads), the per-stage weight copies and their barrier: one
// barrier per 32-channel chunk, i.e. per 288 MFMAs of a wave.
//
// MFMA shape: v_mfma_f32_16x16x32_bf16, each contracting all 32 channels of a chunk.  It does half the
// accumulator traffic per multiply-add of the 32x32x16 shape, and under the power that the operand values
// of this workload draw the chip sustains it at a higher rate (bare loops on random operands: 2.0 against
// 1.87 PFLOP/s; this kernel: +4.5 % over the same schedule on 32x32x16).
// Lane 16 g + q of a wave holds, of a pixel-block fragment, channels 8 g .. 8 g + 7 of pixel q (16 bytes of
// the pixel's 64-byte LDS row); of a weight fragment, the same contraction indices of output channel q (16
// bytes of the blocked layout: block 2 chunk + g / 2, half g % 2); of a 16x16 accumulator, channels
// 4 g .. 4 g + 3 of pixel q.
//
// Workgroup: WM x WN waves, each a (32 TM)-pixel x 64-channel sub-tile, i.e. 2 TM pixel blocks x 4 channel
// blocks of 16: TM = 4 (128 accumulator registers) with two workgroups per CU, or TM = 5 with one
// workgroup per CU and twice the registers per wave, for launches whose 256-pixel tiles would number
// between one and two per CU (then the CUs with two need twice as long as those with one: 320-pixel
// tiles give every CU at most one).
// A chunk is nine steps, one per tap; a step is 2 TM halo-fragment reads and 8 TM MFMAs.  The four weight
// fragments of a tap are requested two taps ahead into a ring of three taps; halo fragments one per pixel
// block, LA blocks ahead into a ring of LA + 1.  The halo of a chunk is copied by global_load_lds_dwordx4
// into one of two buffers a whole chunk ahead; rows are 80 bytes (64 data + 16 pad, conflict-free fragment
// reads at addresses that are a per-lane base plus an offset per tap); the copy treats a buffer as
// consecutive 16-byte slots, slot s = row s / 5, segment s % 5, every lane supplying the 32-bit offset of its
// slot from a scalar base that moves on by a chunk (slots outside the image are zeroed once and their lanes sit
// out: half the address registers of per-lane pointers, which is what lets every epilogue live in registers).
// Once the last halo fragment of a
// chunk has been requested (LA blocks before the chunk ends) the workgroup synchronises, reads on from the
// other buffer and copies the halo of the chunk after next into the one it has left.
// Every other instruction of a step is issued right after an MFMA, in its shadow: a wave issues in order,
// and issued as a block before the MFMAs they would leave the matrix pipe idle whenever the SIMD's other
// wave is not multiplying.
// All vector-memory waits are written by hand (the loads are inline assembly), counting the loads and
// copies issued since the one waited for; the schedule is static, so the counts are constants.  A variant must
// not spill: a load in flight over a spilled register would be lost (the build refuses one that does).
// The result leaves from registers, also pooled or masked: 128 -> 128 at 112x112, batch 32, masked 139 -> 130 us
// against the transposing pass through LDS.
// ---------------------------------------------------------------------------
constexpr int kWregHaloRows = 384;      // halo rows of the weights-in-registers kernel (64 KB of LDS) ...
constexpr int kWregHaloRowsHalf = 224; // ... of its 128-pixel tiles (40 KB)
constexpr int kWregHaloRowsBig = 448;   // ... and of its variant for tiles that straddle images (72 KB)

// EPI: how the tile leaves, a kernel of its own each (the main loop has no register to spare for what the others
// would keep alive across it).
enum ConvEpilogue { kEpiPlain, kEpiMasked, kEpiPooled, kEpiGeneral };

// FOLD: the sums of every p.kchunks chunks are formed from zero and then added to the total (which starts at the bias),
// as workgroups that share a contraction would add theirs.
template <int WM, int WN, int SA, int TM, int OCC, int RB, int EPI, bool FOLD>
__global__ __launch_bounds__(WM *WN * 64, OCC) void conv3x3_igemm_wreg_kernel(ConvArgs p)
{
    typedef bf16_t T;
    constexpr int NW = WM * WN, NT = NW * 64, BM = WM * TM * 32, BN = WN * 64;
    constexpr int NI = 2 * TM, NJ = 4;           // 16-pixel and 16-channel blocks per wave
    constexpr int KC = 32;                       // channels per chunk (one 64-byte LDS row)
    constexpr int NQ = (SA * 5 + NT - 1) / NT;   // halo copies per thread and chunk
    constexpr int ABUF = NQ * NT * 16;           // bytes per halo buffer (>= SA * 80)
    constexpr int TAPS = 9;                      // RB: taps of weight fragments in registers, requested RB - 1 taps ahead
    constexpr int LA = NI % 4 == 0 ? 3 : NI == 6 ? 5 : 4, RA = LA + 1;
    static_assert(TAPS % RB == 0 && (TAPS * NI) % RA == 0, "ring positions must repeat every chunk");
    static_assert(NJ <= NI && NQ <= 3 * LA, "weight loads and halo copies share the slots after the MFMAs");
    // halo copies (three per pixel block, from block NI - LA of the last tap on) issued before that tap's last weight load
    constexpr int early = NJ - 1 > NI - LA ? 3 * (NJ - 1 - (NI - LA)) : 0, NQ_EARLY = early < NQ ? early : NQ;
    static_assert(RB >= 2 && (RB - 1) * NJ + NQ <= 63, "wait counts fit the counter");

    extern __shared__ __align__(16) char smem[];   // [2][ABUF]
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv % WM, wn = wv / WM;
    const int q = lane & 15, g = lane >> 4;
    // (XCD-aware numbering as in the kernels above)
    const int nblk = gridDim.x, xcd = blockIdx.x & 7;
    const int bid = xcd * (nblk >> 3) + min(xcd, nblk & 7) + (blockIdx.x >> 3);
    const int tile_n = bid % p.tiles_n, tile_m = bid / p.tiles_n;
    const int n0 = tile_n * BN;
    const TileOrigin org = tile_origin(p.g, tile_m);
    const int pitch = p.g.pitch;
    const int nchunks = p.CinP / KC;
    const size_t xrow = (size_t)p.CinP * sizeof(T);

    // Halo copies: 32-bit offset of each of this lane's slots from the tile's first halo pixel (a scalar base that
    // moves on by a chunk), and the lanes that copy.  Slots of pixels outside the image are zeroed here, once, in
    // both buffers, and their lanes sit the copies out; the lanes of pad slots, which nobody reads, copy from the base, so that no copy
    // is ever without a lane (the waits below count copies).
    const int px0 = halo_first_pixel(p.g, org);
    unsigned aoff[NQ];
    unsigned long long alanes[NQ];
    {
        // The 64 slots of a copy lie in at most 14 rows.  Which pixel a row is takes some forty instructions, so it is
        // found once, by one lane (lane 16 j + r: row r of copies j, j + 4, ...), and handed to the slots' lanes.
        constexpr int NP = (NQ + 3) / 4;
        int px[NP];
#pragma unroll
        for (int h = 0; h < NP; ++h) {
            const int row = ((4 * h + (lane >> 4)) * NW + wv) * 64 / 5 + (lane & 15);
            px[h] = row < p.g.S ? halo_pixel(p.g, org, row) : -1;
        }
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            const int first = (k * NW + wv) * 64, slot = first + lane;
            const int row = slot / 5, seg = slot - row * 5;
            const int pk = __shfl(px[k >> 2], (k & 3) * 16 + row - first / 5, kWave);
            const bool in = pk >= 0 && seg < 4;
            aoff[k] = in ? (unsigned)(pk - px0) * (unsigned)xrow + seg * 16 : 0u;
            alanes[k] = __ballot(in || seg == 4);
            if (!in && seg < 4) {
                *reinterpret_cast<u32x4 *>(smem + slot * 16) = u32x4{0u, 0u, 0u, 0u};
                *reinterpret_cast<u32x4 *>(smem + ABUF + slot * 16) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    }
    unsigned long long abase;
    {
        const unsigned long long v = (unsigned long long)(uintptr_t)(p.x + (size_t)px0 * xrow);
        abase = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(v >> 32)) << 32) | (unsigned)__builtin_amdgcn_readfirstlane((unsigned)v);
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    auto copy_slot = [&](int buf, int k) __attribute__((always_inline)) {
        const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + buf * ABUF + (k * NW + wv) * 1024);
        // (every lane of the wave is active where this is called)
        asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
                     : : "s"(dst), "v"(aoff[k]), "s"(abase), "s"(alanes[k]) : "m0", "memory");
    };
    auto next_chunk = [&]() __attribute__((always_inline)) { abase += KC * sizeof(T); };

    // byte address (inside a buffer) of tap (0,0) of this lane's pixels, its 16 bytes of the row included (likewise:
    // lane l finds the halo rows of tile rows l, l + 64, ... of the wave)
    int arow[NI];
    {
        constexpr int NR = (NI + 3) / 4;
        int hr[NR];
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            int m;
            tile_row(p.g, org, wm * (TM * 32) + min(h * 64 + lane, TM * 32 - 1), m, hr[h]);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) arow[i] = __shfl(hr[i >> 2], (i & 3) * 16 + q, kWave) * kRowBytes + g * 16;
    }

    // weight fragment (tap t, chunk c, channels ch .. ch + 15): lane's 16 bytes at
    // ((t * KB + 2 c + g / 2) * Cout + ch + q) * 32 + (g % 2) * 16
    const int KB = p.CinP / 16;
    unsigned voff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)   // channels past Cout are never stored
        voff[j] = (unsigned)min(n0 + wn * 64 + j * 16 + q, p.Cout - 1) * 32u + (g & 1) * 16 + (unsigned)(g >> 1) * p.Cout * 32u;
    u32x4 bq[RB][NJ];
    auto load_w = [&](const char *sb, u32x4(&dst)[NJ]) __attribute__((always_inline)) {
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)sb);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uintptr_t)sb >> 32));
        const unsigned long long sbase = ((unsigned long long)hi << 32) | lo;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst[j]) : "v"(voff[j]), "s"(sbase) : "memory");
    };

    // Accumulators start at the bias (requested here into the first pixel block, copied to the others once
    // the loads have had time to land).
    f32x4v acc[NI][NJ];
    {
        const int c0 = n0 + wn * 64 + g * 4;
        if (!p.bias) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[0][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
        } else if ((p.Cout & 3) == 0) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[0][j] = *reinterpret_cast<const f32x4v *>(p.bias + min(c0 + j * 16, p.Cout - 4));
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[0][j][e] = p.bias[min(c0 + j * 16 + e, p.Cout - 1)];
        }
    }

    // prologue: the first two halo chunks and the weights of the first two taps
#pragma unroll
    for (int k = 0; k < NQ; ++k) copy_slot(0, k);
    if (nchunks > 1) {
        next_chunk();
#pragma unroll
        for (int k = 0; k < NQ; ++k) copy_slot(1, k);
    }
    const long long w_tap = (long long)KB * p.Cout * 32;            // next tap of the same chunk
    const long long w_c = 2ll * p.Cout * 32 - 8 * w_tap;            // last tap -> first tap of the next chunk
    const long long w_same = -8 * w_tap;                            // ... of the same chunk again (past the end)
#pragma unroll
    for (int t = 0; t + 1 < RB; ++t) load_w(p.w + t * w_tap, bq[t]);
    const char *wnext = p.w + (RB - 1) * w_tap;                     // the fragments requested next: tap RB - 1 of chunk 0
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int i = 1; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = acc[0][j];
    f32x4v total[FOLD ? NI : 1][NJ];
    auto fold = [&](bool first) __attribute__((always_inline)) {
        if constexpr (FOLD) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    total[i][j] = first ? acc[i][j] : total[i][j] + acc[i][j];
                    acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    fold(true);

    u32x4 af[RA];
#pragma unroll
    for (int f = 0; f < LA; ++f) af[f] = *reinterpret_cast<const u32x4 *>(smem + arow[f]);   // tap 0, pixel blocks 0 .. LA - 1

    for (int c = 0; c < nchunks; ++c) {
        const int ab = c & 1;
        const long long w_wrap = c + 1 < nchunks ? w_c : w_same;
        for_each_step([&](auto ic) {
            constexpr int t = decltype(ic)::value;
            // This tap's four weight fragments were requested during tap t - (RB - 1); since then came those of
            // the RB - 2 taps in between and, when the end of a chunk lies there too, its NQ halo copies (when the
            // request was made in the chunk's last tap: those of them issued after the last of the four).
            constexpr int younger = (RB - 2) * NJ + (t < RB - 2 ? NQ : t == RB - 2 ? NQ - NQ_EARLY : 0);
            u32x4 b0 = bq[t % RB][0], b1 = bq[t % RB][1], b2 = bq[t % RB][2], b3 = bq[t % RB][3];
            asm volatile("s_waitcnt vmcnt(%4)" : "+v"(b0), "+v"(b1), "+v"(b2), "+v"(b3) : "n"(younger));
            const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)wnext);
            const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uintptr_t)wnext >> 32));
            const unsigned long long sbase = ((unsigned long long)hi << 32) | lo;
            wnext += (t + RB - 1) % TAPS == TAPS - 1 ? w_wrap : w_tap;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                constexpr int first_next = NI - LA;   // the pixel block during which the first fragment of the next chunk is requested
                if (t == TAPS - 1 && i == first_next) {
                    // Every halo read of this chunk has been issued; the waits at the taps so far have covered
                    // the next chunk's copies, issued a whole chunk ago.  After the barrier the other buffer is
                    // published and this one is free for the chunk after next.
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    if (c + 2 < nchunks) next_chunk();   // (past the end: the last chunk again, never read; keeps the wait counts static)
                }
                const int f = t * NI + i;             // position in the chunk's sequence of halo fragments
                const int fr = (f + LA) % (TAPS * NI), nt = fr / NI, ni = fr % NI;
                const int nbuf = f + LA < TAPS * NI ? ab : ab ^ 1;
                const char *abase = smem + nbuf * ABUF + ((nt / 3) * pitch + nt % 3) * kRowBytes;
                const bf16x8 a = __builtin_bit_cast(bf16x8, af[f % RA]);
                const bool copying = t == TAPS - 1 && i >= first_next;
                acc[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b0), a, acc[i][0], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                af[(f + LA) % RA] = *reinterpret_cast<const u32x4 *>(abase + arow[ni]);
                __builtin_amdgcn_sched_barrier(0);
                acc[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b1), a, acc[i][1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (i < NJ)
                    asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(bq[(t + RB - 1) % RB][i]) : "v"(voff[i]), "s"(sbase) : "memory");
                if (copying && (i - first_next) * 3 < NQ) copy_slot(ab, (i - first_next) * 3);
                __builtin_amdgcn_sched_barrier(0);
                acc[i][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b2), a, acc[i][2], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (copying && (i - first_next) * 3 + 1 < NQ) copy_slot(ab, (i - first_next) * 3 + 1);
                __builtin_amdgcn_sched_barrier(0);
                acc[i][3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b3), a, acc[i][3], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (copying && (i - first_next) * 3 + 2 < NQ) copy_slot(ab, (i - first_next) * 3 + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }, std::make_integer_sequence<int, TAPS>{});
        if (FOLD && ((c + 1) % p.kchunks == 0 || c + 1 == nchunks)) fold(false);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the weight loads and halo copies issued past the end
    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = total[i][j];
    }

    const int wrow0 = wm * (TM * 32);
    if (EPI == kEpiGeneral || (p.Cout & 7)) {   // pooled and un-pooled result, or a channel count that 16-byte stores do not divide
        conv_epilogue_impl<T, BM, BN, WM, WN>(
            [&](int i, int j0, char *epi, float lo) __attribute__((always_inline)) {
                // (bf16: a pass is all 64 columns of the wave; pixel block i of 32 rows = 16-pixel blocks 2 i, 2 i + 1)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const f32x4v &t = acc[2 * i + h][j];
                        store4(reinterpret_cast<T *>(epi + (h * 16 + q) * kEpiRow) + j * 16 + g * 4, fmaxf(t[0], lo), fmaxf(t[1], lo),
                               fmaxf(t[2], lo), fmaxf(t[3], lo));
                    }
            },
            [&](auto fn) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) fn(wrow0 + i * 16 + q, j * 16 + g * 4 + e, acc[i][j][e]);
            },
            p, org, smem, n0);
        return;
    }
    // Straight from registers, without LDS or a barrier.  A lane holds four consecutive channels of a pixel per
    // accumulator; lanes 16 apart (the next four channels of the same pixel) swap the values of one of two
    // accumulators (v_permlane16_swap: the even row of 16 lanes ends up with eight channels of the first, the odd
    // row with eight channels of the second) and store 16 bytes each.
    // (the lane number is taken afresh, so that no address of the epilogue is formed before the main loop and held
    // across it)
    int le;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(le));
    const int qe = le & 15, ge = le >> 4;
    const float lo = p.relu ? 0.f : -__builtin_inff();
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    auto pack = [&](const f32x4v &t, unsigned(&x)[2]) __attribute__((always_inline)) {   // ReLU, round
        const f32x2_t v0 = {fmaxf(t[0], lo), fmaxf(t[1], lo)}, v1 = {fmaxf(t[2], lo), fmaxf(t[3], lo)};
        x[0] = __builtin_bit_cast(unsigned, __builtin_convertvector(v0, bf16x2_t));
        x[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(v1, bf16x2_t));
    };
    auto swap16 = [](unsigned(&x0)[2], unsigned(&x1)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const auto sw = __builtin_amdgcn_permlane16_swap(x0[k], x1[k], false, false);
            x0[k] = sw[0];
            x1[k] = sw[1];
        }
        return u32x4{x0[0], x0[1], x1[0], x1[1]};
    };
    if (EPI == kEpiPlain || EPI == kEpiMasked) {
        // (mask > 0) factor: the 16 bytes of the mask behind each store, all of them requested at once into the registers that
        // the main loop has left, and without conditions (pixels and channels past the ends: the first and the last ones, not
        // used): a load under a condition is waited for where it ends, four memory latencies a tile.  128 -> 128 at 112x112,
        // batch 32: 129.5 -> 129.1 us (bound by the burst itself), 512 -> 512 at 14x14, batch 100, 75.0 -> 71.8, 200 -> 96 at 45x60, batch 7,
        // 18.4 -> 16.4.
        T *y = reinterpret_cast<T *>(p.y);
        const T *mask = reinterpret_cast<const T *>(p.mask);
        const int col0 = n0 + wn * 64 + (ge >> 1) * 8;
        u32x4 mk[EPI == kEpiMasked ? NI / 2 : 1][NJ];
        int mrow[NI / 2];
#pragma unroll
        for (int ip = 0; ip < NI / 2; ++ip) {
            mrow[ip] = tile_pixel(p.g, org, wrow0 + (2 * ip + (ge & 1)) * 16 + qe);
            if (EPI == kEpiMasked) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    mk[ip][j] = *reinterpret_cast<const u32x4 *>(mask + (size_t)max(mrow[ip], 0) * p.Cout + min(col0 + j * 16, p.Cout - 8));
            }
        }
#pragma unroll
        for (int ip = 0; ip < NI / 2; ++ip) {
            const int m = mrow[ip];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                unsigned x0[2], x1[2];
                pack(acc[2 * ip][j], x0);
                pack(acc[2 * ip + 1][j], x1);
                u32x4 v = swap16(x0, x1);
                if (EPI == kEpiMasked) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const unsigned w = mk[ip][j][k];
                        const unsigned keep = (__uint_as_float(w << 16) > 0.f ? 0xffffu : 0u) |
                                              (__uint_as_float(w & 0xffff0000u) > 0.f ? 0xffff0000u : 0u);
                        v[k] &= keep;
                    }
                }
                if (m >= 0 && col0 + j * 16 < p.Cout) *reinterpret_cast<u32x4 *>(y + (size_t)m * p.Cout + col0 + j * 16) = v;
            }
        }
        return;
    }
    // 2x2 maximum of the rounded values (patch tiles: a 16-pixel block is one patch row, so a window is two blocks
    // of the wave and two neighbouring lanes).  Even lanes serve the windows of rows 4 b, 4 b + 1, odd lanes those
    // of rows 4 b + 2, 4 b + 3; the four values in window order, a later one only when strictly greater.
    {
        T *pool = reinterpret_cast<T *>(p.pool);
        const bool odd = qe & 1;
        auto xchg = [](float v) __attribute__((always_inline)) {   // the neighbouring lane's value (DPP quad permute 1, 0, 3, 2)
            return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
        };
#pragma unroll
        for (int b = 0; b < NI / 4; ++b) {
            const int ph = (org.h0 + wrow0 / kTileW + 4 * b) / 2 + (odd ? 1 : 0), pw = (org.w0 >> 1) + (qe >> 1);
            const bool in = 2 * ph < p.g.H && 2 * pw < p.g.W;
            const size_t at = (((size_t)org.n * (p.g.H >> 1) + ph) * (p.g.W >> 1) + pw) * p.Cout;
#pragma unroll
            for (int j = 0; j < NJ; j += 2) {
                unsigned best[2][2], which[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    unsigned x[4][2];
#pragma unroll
                    for (int r = 0; r < 4; ++r) pack(acc[4 * b + r][j + h], x[r]);
                    which[h] = 0;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        unsigned out = 0;
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            float v[4];   // rows 4 b .. 4 b + 3 of this lane's pixel column
#pragma unroll
                            for (int r = 0; r < 4; ++r) v[r] = __uint_as_float(e ? x[r][k] & 0xffff0000u : x[r][k] << 16);
                            // what the neighbour serves of mine goes to it, what I serve of its comes here
                            const float own0 = odd ? v[2] : v[0], own1 = odd ? v[3] : v[1];
                            const float got0 = xchg(odd ? v[0] : v[2]), got1 = xchg(odd ? v[1] : v[3]);
                            const float w0 = odd ? got0 : own0, w1 = odd ? own0 : got0, w2 = odd ? got1 : own1, w3 = odd ? own1 : got1;
                            float m = w0;
                            unsigned a = 0;
                            if (w1 > m) { m = w1; a = 1; }
                            if (w2 > m) { m = w2; a = 2; }
                            if (w3 > m) { m = w3; a = 3; }
                            out |= e ? __float_as_uint(m) : __float_as_uint(m) >> 16;
                            which[h] |= a << (8 * (2 * k + e));
                        }
                        best[h][k] = out;
                    }
                }
                const u32x4 v = swap16(best[0], best[1]);
                const auto sw = __builtin_amdgcn_permlane16_swap(which[0], which[1], false, false);
                const int col = n0 + wn * 64 + (j + (ge & 1)) * 16 + (ge >> 1) * 8;
                if (in && col < p.Cout) {
                    *reinterpret_cast<u32x4 *>(pool + at + col) = v;
                    if (p.argmax) {   // (bytes, of any alignment)
                        const unsigned pos[2] = {sw[0], sw[1]};
                        __builtin_memcpy(p.argmax + at + col, pos, 8);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// bf16, launches with fewer tiles than the chip has SIMDs to fill (small batches): a workgroup of G waves owns
// 64 pixels x 16 NJ channels, and its waves share the contraction: p.ksplit ranges of p.kchunks channel chunks, taken
// by the waves in turn (wave w: w and w + G), each with all nine taps.  What bounds such a launch is not the matrix pipe but
// the chain launch -> first loads -> multiply -> combine and the instructions along it, so the kernel has one of each: a wave copies its own chunk's halo
// into its own LDS region and requests all nine taps' weights at once (9 NJ fragments in registers, plain loads; a tap's
// registers are refilled for the wave's next chunk as soon as its MFMAs are issued), no barrier between the shared table and the end,
// and the waves' sums meet in LDS instead of in a partial-sum buffer that a second launch has to read.
// LDS rows are 64 bytes, segment s of row q at s ^ ((q >> 1) & 3): conflict-free for the fragment reads of
// v_mfma_f32_16x16x32_bf16 (lane 16 g + q reads segment g of pixel q).
// ---------------------------------------------------------------------------
constexpr int kSmallPx = 64;         // pixels per tile
constexpr int kSmallHaloRows = 256;  // most halo rows of a tile (the launch picks patches where consecutive pixels need more)

constexpr int kSmallRanges = 8;      // most ranges of the contraction

template <int NJ, int G, bool TWO>   // TWO: waves may have two ranges
__global__ __launch_bounds__(G * 64, 2) void conv3x3_small_bf16_kernel(ConvArgs p)
{
    typedef bf16_t T;
    constexpr int NI = 4, BN = NJ * 16, KC = 32, TAPS = 9;
    constexpr int RP = BN + 4;                    // floats per row of the combine buffer
    static_assert(kSmallHaloRows <= G * 64, "a thread per halo row");
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane & 15, g = lane >> 4;
    // (each XCD takes a contiguous range of tiles, pixel tiles fastest: the weights, the larger operand here, are
    // then read into one L2 only)
    const int nblk = gridDim.x, xcd = blockIdx.x & 7;
    const int bid = xcd * (nblk >> 3) + min(xcd, nblk & 7) + (blockIdx.x >> 3);
    const int tile_n = fast_div(bid, p.dTiles), tile_m = bid - tile_n * p.g.ntiles;
    const int n0 = tile_n * BN;
    const TileOrigin org = tile_origin(p.g, tile_m);
    const int pitch = p.g.pitch, nchunks = p.CinP / KC;
    // the chunk after c of this wave's ranges (nchunks: none)
    auto next_of = [&](int c) __attribute__((always_inline)) {
        const int n = c + 1, skip = n % p.kchunks == 0 ? (G - 1) * p.kchunks : 0;
        return min(n + skip, nchunks);
    };
    const int c_first = min(wv * p.kchunks, nchunks);
    const size_t xrow = (size_t)p.CinP * sizeof(T);

    // weight fragment (tap t, chunk c, channels ch .. ch + 15): see conv3x3_igemm_wreg_kernel
    const int KB = p.CinP / 16;
    const size_t w_tap = (size_t)KB * p.Cout * 32;
    unsigned voff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)   // channels past Cout are never stored
        voff[j] = (unsigned)min(n0 + j * 16 + q, p.Cout - 1) * 32u + (g & 1) * 16 + (unsigned)(g >> 1) * p.Cout * 32u;
    u32x4 bw[TAPS][NJ];
    auto load_w = [&](int c, int t) __attribute__((always_inline)) {
        const char *sb = p.w + t * w_tap + (size_t)c * 2 * p.Cout * 32;
#pragma unroll
        for (int j = 0; j < NJ; ++j) bw[t][j] = *reinterpret_cast<const u32x4 *>(sb + voff[j]);
    };
#pragma unroll
    for (int t = 0; t < TAPS; ++t) load_w(min(c_first, nchunks - 1), t);

    // What bounds the front of such a launch is the instructions issued before the first multiplication (2.8 of 9 us at one
    // image's 14x14 and 28x28 layers when every wave found its own pixels), so that is done once per workgroup: thread t finds the
    // pixel behind halo row t, the last wave the halo rows of the tile's 64 pixels, and the table is shared through LDS.
    // [rowsA] byte offsets from the halo's first pixel, [64] halo rows of tap (0,0)
    int *const table = reinterpret_cast<int *>(smem + p.tableA);
    const int px0 = halo_first_pixel(p.g, org);
    if (tid < p.rowsA) {
        const int px = tid < p.g.S ? halo_pixel(p.g, org, tid) : -1;
        table[tid] = px < 0 ? (int)0x80000000u : (px - px0) * (int)xrow;   // (outside the image: beyond the buffer, reads zeros)
    }
    if (wv == G - 1) {
        int m, h;
        tile_row(p.g, org, lane, m, h);
        table[p.rowsA + lane] = h;
    }
    // What a thread adds and stores after the multiplications: its four channels' bias and, without a pool, its pixels and mask.
    constexpr int C4 = BN / 4, OUT = (kSmallPx * C4 + G * 64 - 1) / (G * 64);   // (channel quads of a tile row; of the tile per thread)
    T *y = reinterpret_cast<T *>(p.y), *pool = reinterpret_cast<T *>(p.pool);
    const int col = n0 + (tid % C4) * 4;
    const f32x4v bias = *reinterpret_cast<const f32x4v *>(p.bias ? reinterpret_cast<const char *>(p.bias + min(col, p.Cout - 4))
                                                                 : reinterpret_cast<const char *>(kZeroRow));
    int pixel[OUT];
    u32x2 mk[OUT];
#pragma unroll
    for (int k = 0; k < OUT; ++k) {
        const int row = (k * G * 64 + tid) / C4;
        pixel[k] = row < kSmallPx ? tile_pixel(p.g, org, row) : -1;   // (16-wide columns: more threads than quads)
        mk[k] = *reinterpret_cast<const u32x2 *>(p.mask ? p.mask + ((size_t)max(pixel[k], 0) * p.Cout + min(col, p.Cout - 4)) * sizeof(T)
                                                        : reinterpret_cast<const char *>(kZeroRow));
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // (not __syncthreads(), which would wait for the loads above)

    const int bufs = p.rowsA * kDataBytes;                            // bytes of a halo buffer (rowsA a multiple of 16)
    char *As = smem + wv * bufs;                                      // this wave's buffer
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)As);
    // A copy moves 16 rows x 64 bytes; segment s of row q lies at s ^ ((q >> 1) & 3).
    constexpr int COPIES = kSmallHaloRows / 16;
    unsigned from[COPIES];
#pragma unroll
    for (int k = 0; k < COPIES; ++k)
        if (k * 16 < p.rowsA) from[k] = (unsigned)table[k * 16 + (lane >> 2)] + (((lane & 3) ^ ((lane >> 3) & 3)) << 4);
    int hrow[NI];   // halo row of tap (0,0) of this lane's pixels
#pragma unroll
    for (int i = 0; i < NI; ++i) hrow[i] = table[p.rowsA + i * 16 + q];
    // (from the halo's first pixel; offsets of pixels are below 2^31, the one that stands for "outside the image" is beyond)
    const uintptr_t x0 = (uintptr_t)p.x + (size_t)px0 * xrow;
    const u32x4 xbuf = {(unsigned)__builtin_amdgcn_readfirstlane((unsigned)x0), (unsigned)__builtin_amdgcn_readfirstlane((unsigned)(x0 >> 32)),
                        0x80000000u, 0x00020000u};
    auto copy = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < COPIES; ++k) {
            if (k * 16 < p.rowsA) {
                const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + k * 1024);
                asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                             : : "s"(dst), "v"(from[k]), "s"(xbuf), "s"(c * kDataBytes) : "m0", "memory");
            }
        }
    };
    if (c_first < nchunks) copy(c_first);
    f32x4v acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};

    // At most two ranges per wave (w and w + G): the first one's sums wait in registers.
    f32x4v first[TWO ? NI : 1][NJ];
    auto take = [&]() __attribute__((always_inline)) {
        if constexpr (TWO) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    first[i][j] = acc[i][j];
                    acc[i][j] = f32x4v{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    take();
    for (int c = c_first; c < nchunks;) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this chunk's halo has landed (and its weights)
        const int cn = next_of(c);
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            bf16x8 a[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int row = hrow[i] + (t / 3) * pitch + t % 3;
                a[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(As + row * kDataBytes + ((g ^ (row >> 1)) & 3) * 16));
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bw[t][j]), a[i], acc[i][j], 0, 0, 0);
            if (cn < nchunks) load_w(cn, t);
        }
        if (cn < nchunks) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // (this chunk's reads are done)
            copy(cn);
        }
        if (c + 1 == c_first + p.kchunks && wv + G < p.ksplit) take();
        c = cn;
    }

    // Combine: the ranges' sums go to LDS, [range][pixel][channel], in place of the halos; then each thread adds those
    // of its four channels in a fixed order (bias first), applies ReLU / mask, and stores; with a pool, of the four
    // pixels of a window.
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem);
    auto park = [&](const f32x4v(&v)[NI][NJ], int range) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                *reinterpret_cast<f32x4v *>(red + (size_t)(range * kSmallPx + i * 16 + q) * RP + j * 16 + g * 4) = v[i][j];
    };
    if constexpr (TWO) {
        const bool two = wv + G < p.ksplit;
        if (two) park(first, wv);
        if (wv < p.ksplit) park(acc, two ? wv + G : wv);
    } else if (wv < p.ksplit) park(acc, wv);
    __syncthreads();
    const float lo = p.relu ? 0.f : -__builtin_inff();
    auto value = [&](int row, T(&out)[4]) __attribute__((always_inline)) {   // this thread's four channels of tile row `row`
        f32x4v s = bias;
        for (int w = 0; w < p.ksplit; ++w) s += *reinterpret_cast<const f32x4v *>(red + (size_t)(w * kSmallPx + row) * RP + (tid % C4) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = f32_to_bf16(fmaxf(s[e], lo));
    };
    if (col >= p.Cout) return;
    if (!pool) {
#pragma unroll
        for (int k = 0; k < OUT; ++k) {
            if (pixel[k] < 0) continue;
            T out[4], m[4];
            value((k * G * 64 + tid) / C4, out);
            __builtin_memcpy(m, &mk[k], 8);
            if (p.mask) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!(bf16_to_f32(m[e]) > 0.f)) out[e] = (T)0;
            }
            __builtin_memcpy(y + (size_t)pixel[k] * p.Cout + col, out, 8);
        }
        return;
    }
    // (patch tiles of 4 x 16 pixels: sixteen windows)
    for (int u = tid; u < kSmallPx / 4 * C4; u += G * 64) {
        const int win = u / C4, dy = win >> 3, dx = win & 7;
        const int ph = (org.h0 >> 1) + dy, pw = (org.w0 >> 1) + dx;
        if (2 * ph >= p.g.H || 2 * pw >= p.g.W) continue;
        T best[4];
        unsigned char which[4] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            T v[4];
            const int row = (2 * dy + (k >> 1)) * kTileW + 2 * dx + (k & 1);
            value(row, v);
            const int m = tile_pixel(p.g, org, row);
            if (m >= 0 && y) __builtin_memcpy(y + (size_t)m * p.Cout + col, v, 8);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k == 0 || bf16_to_f32(v[e]) > bf16_to_f32(best[e])) { best[e] = v[e]; which[e] = (unsigned char)k; }
        }
        const size_t at = (((size_t)org.n * (p.g.H >> 1) + ph) * (p.g.W >> 1) + pw) * p.Cout + col;
        __builtin_memcpy(pool + at, best, 8);
        if (p.argmax) __builtin_memcpy(p.argmax + at, which, 4);
    }
}

// LDS bytes of a launch.  One halo buffer per wave: a second one, copied a chunk ahead, never gained (5174 launches: 1.00
// to 1.05 times the time) and cost up to 1.8 times where it left a CU one workgroup instead of two.
static size_t conv_small_lds(int G, int S, int ksplit)
{
    const size_t halo = (size_t)G * round_up16(S) * kDataBytes, red = (size_t)ksplit * kSmallPx * (2 * 16 + 4) * 4;
    return (halo > red ? halo : red) + (round_up16(S) + kSmallPx) * sizeof(int);   // (the table behind either)
}
template <int NJ, int G>
static int launch_conv_small(const ConvArgs &a0, const TileGeom &g, hipStream_t stream)
{
    ConvArgs a = a0;
    a.g = g;
    a.tiles_n = (a.Cout + NJ * 16 - 1) / (NJ * 16);
    a.rowsA = round_up16(g.S);
    a.dTiles = make_fast_div(g.ntiles);
    auto kern = conv3x3_small_bf16_kernel<NJ, G, false>;
    if constexpr (G == 4 && NJ == 2)   // (where columns are 16 wide every wave has one range)
        if (a.ksplit > G) kern = conv3x3_small_bf16_kernel<NJ, G, true>;
    if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    const size_t lds = conv_small_lds(G, g.S, a.ksplit);
    a.tableA = (int)(lds - (a.rowsA + kSmallPx) * sizeof(int));
    hipLaunchKernelGGL(kern, dim3((unsigned)(g.ntiles * a.tiles_n)), dim3(G * 64), lds, stream, a);
    return launch_status();
}

template <int WM, int WN, int SA, int TM = 4, int OCC = 2, int RB = 3, bool FOLD = false>
static int launch_conv_wreg(const ConvArgs &a0, const TileGeom &g, hipStream_t stream)
{
    ConvArgs a = a0;
    constexpr int NT = WM * WN * 64, BN = WN * 64;
    constexpr int NQ = (SA * 5 + NT - 1) / NT;
    a.g = g;
    a.tiles_n = (a.Cout + BN - 1) / BN;
    a.rowsA = SA;
    const size_t lds = (size_t)2 * NQ * NT * 16;   // (more than the epilogue's staging blocks)
    auto launch = [&](auto kern) {
        if (!raise_lds_limit(reinterpret_cast<const void *>(kern))) return (int)VGG_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3((unsigned)(a.g.ntiles * a.tiles_n)), dim3(NT), lds, stream, a);
        return launch_status();
    };
    if ((a.pool && a.y) || (a.Cout & 7)) return launch(conv3x3_igemm_wreg_kernel<WM, WN, SA, TM, OCC, RB, kEpiGeneral, FOLD>);
    if constexpr (TM % 2 == 0 && !FOLD)   // (a pool is planned neither on 192- and 320-pixel tiles nor where sums are folded)
        if (a.pool) return launch(conv3x3_igemm_wreg_kernel<WM, WN, SA, TM, OCC, RB, kEpiPooled, FOLD>);
    if (a.mask) return launch(conv3x3_igemm_wreg_kernel<WM, WN, SA, TM, OCC, RB, kEpiMasked, FOLD>);
    return launch(conv3x3_igemm_wreg_kernel<WM, WN, SA, TM, OCC, RB, kEpiPlain, FOLD>);
}

template <typename T, int BM, int BN, int WM, int WN, int SA>
static int launch_conv_dma(const ConvArgs &a0, const TileGeom &g, hipStream_t stream)
{
    ConvArgs a = a0;
    a.g = g;
    a.tiles_n = (a.Cout + BN - 1) / BN;
    a.rowsA = SA;
    const size_t arow_bytes = (SA == kDmaHaloRows && WM * WN == 8) ? kRowBytes : kDataBytes;   // as in the kernel
    size_t lds = (size_t)a.rowsA * 4 + (size_t)a.rowsA * arow_bytes + (size_t)2 * 3 * BN * kDataBytes;
    if (lds < (size_t)WM * WN * kEpiBytes) lds = (size_t)WM * WN * kEpiBytes;
    auto kern = conv3x3_igemm_dma_kernel<T, BM, BN, WM, WN, SA>;
    if (lds > 64 * 1024 && !raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.g.ntiles * a.tiles_n * a.ksplit)), dim3(WM * WN * 64), lds, stream, a);
    return launch_status();
}

template <typename T, int BM, int BN, int WM, int WN>
static int launch_conv(const ConvArgs &a0, int N, int H, int W, hipStream_t stream)
{
    ConvArgs a = a0;
    a.g = make_tile_geom(N, H, W, BM);
    a.tiles_n = (a.Cout + BN - 1) / BN;
    constexpr int NT = WM * WN * 64;
    a.rowsA = a.g.S * 4 <= kMaxAHaloSegsPerBlock ? kMaxAHaloSegsPerBlock / 4 : a.g.S;
    size_t lds = round_up((size_t)a.rowsA * 4, 16) + (size_t)a.rowsA * kRowBytes + (size_t)3 * BN * kRowBytes;
    if (lds < (size_t)WM * WN * kEpiBytes) lds = (size_t)WM * WN * kEpiBytes;
    if (lds > 160 * 1024) return VGG_ERR_UNSUPPORTED;
    auto kern = conv3x3_igemm_kernel<T, BM, BN, WM, WN>;
    if (lds > 64 * 1024 && !raise_lds_limit(reinterpret_cast<const void *>(kern))) return VGG_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.g.ntiles * a.tiles_n)), dim3(WM * WN * 64), lds, stream, a);
    return launch_status();
}

// Sums the partial results of a split contraction: y = f(bias + sum over splits), f = ReLU and/or the
// (mask > 0) factor, converted to T.  One thread per four channels.
template <typename T>
__global__ __launch_bounds__(256) void conv_split_finish_kernel(const float *__restrict__ part, const float *__restrict__ bias,
                                                                const T *__restrict__ mask, T *__restrict__ y, size_t quads,
                                                                int Cout, int ksplit, int relu)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= quads) return;
    const int col = (int)((i * 4) % (size_t)Cout);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (bias) s = *reinterpret_cast<const f32x4 *>(bias + col);
    for (int k = 0; k < ksplit; ++k) s += *reinterpret_cast<const f32x4 *>(part + ((size_t)k * quads + i) * 4);
    const float lo = relu ? 0.f : -__builtin_inff();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        s[e] = fmaxf(s[e], lo);
        if (mask && !(Elem<T>::load(mask + i * 4 + e) > 0.f)) s[e] = 0.f;
    }
    store4(y + i * 4, s[0], s[1], s[2], s[3]);
}

// Which kernel a shape gets (the codes vgg_conv3x3_plan reports), and whether its contraction is split over
// several workgroups per tile.
enum ConvKernel {
    kStaged = 0, kDma, kDmaBig, kDmaHalf,       // register-staged; direct-to-LDS with 384 / 448 / 192 halo rows
    kWreg, kWregBig, kWregTall, kWregTallBig,   // weights in registers: 256- and 320-pixel tiles, 384 / 448 halo rows
    kWregHalf, kWregHalfBig,                    // ... 128-pixel tiles, 224 / 384 halo rows (the sums folded per range
                                                //     where the contraction is split)
    kWregDeep, kWregDeepBig,                    // ... with nine taps of weights in flight
    kSmall4, kSmall8,                           // 64 x 32 or 64 x 16 tiles, the contraction split over four / eight waves
    kF32x3, kF32x3Big, kF32x3Half,              // fp32 in three bf16 parts: 256-pixel tiles, 384 / 448 halo rows; 128-pixel tiles
    kWregMid, kWregMidDeep                      // weights in registers, 192-pixel tiles, 384 halo rows; nine taps of weights in flight
};
// the kernels whose workgroups may share a tile's contraction through memory
static bool over_workgroups(int kernel) { return kernel == kDma || kernel == kDmaBig || kernel == kF32x3 || kernel == kF32x3Big || kernel == kF32x3Half; }
struct ConvPlan {
    TileGeom g;
    int kernel;
    int bn;              // channels per tile
    int ksplit, kchunks;
};

// Split of the contraction, decided on tiles of 256 pixels.  Small batches: fewer tiles than CUs, each walking the whole
// contraction alone.  Then the contraction is summed in ranges of (at least two) channel chunks, by a workgroup each,
// whose partial sums a second kernel adds, or (bf16, where that is faster) inside one workgroup in the same order.
static void conv_split(int dtype, const TileGeom &g, int CinP, int Cout, int &ksplit, int &kchunks)
{
    const int chunks = CinP * dtype_size(dtype) / kDataBytes;
    const bool narrow = Cout <= 64 || g.ntiles * ((Cout + 127) / 128) < 512;
    const int total = g.ntiles * ((Cout + (narrow ? 63 : 127)) / (narrow ? 64 : 128));
    ksplit = 1; kchunks = chunks;
    // Measured: pays when at most half the CUs would have a workgroup and a tile's contraction is
    // long enough (a bf16 chunk takes a quarter of the time of an fp32 one).
    if (g.S <= kDmaHaloRowsBig && Cout % 4 == 0 && total <= 128 && chunks >= (dtype == VGG_BF16 ? 8 : 4)) {
        int want = (512 + total - 1) / total;   // two workgroups per CU
        if (want > chunks / 2) want = chunks / 2;
        kchunks = (chunks + want - 1) / want;
        ksplit = (chunks + kchunks - 1) / kchunks;
    }
}
// The only place that says whether workgroups may share a tile through memory: the launch (conv_plan) and the query that
// sizes the buffer of partial sums (conv3x3_igemm_workspace) both ask it.  Images whose consecutive pixels have a halo
// beyond kDmaHaloRowsBig are never split that way, on whatever tiles they then run.
static void conv_split_in_memory(int dtype, int N, int H, int W, int CinP, int Cout, int &ksplit, int &kchunks)
{
    conv_split(dtype, make_tile_geom(N, H, W, 256), CinP, Cout, ksplit, kchunks);
}

// Tiles of the small-problem kernel: consecutive pixels, or patches where their halo is the smaller one (56 wide:
// 240 halo rows against 108) or a pool is to be fused, and they stick out of the image by at most a quarter.
static TileGeom conv_small_geom(int N, int H, int W, bool pool)
{
    const TileGeom lin = make_tile_geom(N, H, W, kSmallPx), patch = make_patch_geom(N, H, W, kSmallPx);
    const bool fits = patch.ntiles * 4 <= lin.ntiles * 5, cheaper = (long)patch.ntiles * patch.S < (long)lin.ntiles * lin.S;
    return lin.mode == 0 && ((fits && (cheaper || pool)) || lin.S > kSmallHaloRows) ? patch : lin;
}

bool conv3x3_pool_fusable(int dtype, int H, int W, int Cout);

static ConvPlan conv_plan(int dtype, int N, int H, int W, int CinP, int Cout, bool pool)
{
    ConvPlan c;
    c.g = make_tile_geom(N, H, W, 256);
    const bool wide = c.g.S > kDmaHaloRowsBig;
    if (wide) {
        // wide images (from about 60 pixels): the halo of consecutive pixels does not fit the direct-to-LDS kernels;
        // patches do, unless more than a third of their pixels would lie outside the image (bf16 128 -> 128 at 64x70,
        // batch 10: 30 -> 19 us).
        // bf16: at most 32 input channels leave little to win on a padded pixel where it also costs several column
        // tiles or element-wise stores (66x66 batch 9, 32 -> 1024 36 us, 42 on patches that pad by 1.47; batch 30, 32 -> 36 22 /
        // 26): at most 1.4 of the image then, except beyond 640 halo rows, which the staged kernel is slow to fetch (24x200
        // batch 43, 32 -> 8 42 us, 17 on patches that pad by 1.39; 81x81 batch 20, 64 -> 64 26 / 17 at 1.40).
        // fp32 multiplies at a sixteenth of the rate and pays for every padded pixel, so only 64-wide tiles of which no CU
        // gets more than before: 322 of 505 shapes, 0.86 of the staged kernel's time on average, 0.99 at most (the others
        // 1.2 on average; 66x66 batch 9, 384 -> 64 backwards 175 us, 280 on patches).
        const TileGeom patch = make_patch_geom(N, H, W, 256);
        const int cols64 = (Cout + 63) / 64;
        const bool little = CinP <= 32 && (Cout >= 128 || Cout % 8) && c.g.S <= 640;
        const bool pays = dtype == VGG_BF16 || ((Cout <= 64 || patch.ntiles * ((Cout + 127) / 128) < 512) &&
                                                (patch.ntiles * cols64 + 255) / 256 <= (c.g.ntiles * cols64 + 255) / 256);
        if (pays && (long)patch.ntiles * 256 * 10 <= (long)c.g.M * (dtype == VGG_BF16 && little ? 14 : 15)) c.g = patch;
    }
    const bool dma = c.g.S <= kDmaHaloRows, dma_big = !dma && c.g.S <= kDmaHaloRowsBig;
    const int cols = (Cout + 127) / 128, wide_tiles = c.g.ntiles * cols;
    const int chunks = CinP * dtype_size(dtype) / kDataBytes;
    // Too few 256x128 tiles to give every CU two workgroups (the 14x14 layers): 64-wide column tiles
    // double the workgroup count and three of them fit on a CU.
    const bool narrow = Cout <= 64 || wide_tiles < 512;
    c.ksplit = 1; c.kchunks = chunks;
    c.kernel = dma ? kDma : (dma_big ? kDmaBig : kStaged);
    c.bn = narrow ? 64 : 128;
    if (dtype == VGG_F32) {
        if (!pool) conv_split_in_memory(dtype, N, H, W, CinP, Cout, c.ksplit, c.kchunks);
        // fp32, 64-wide tiles, a launch of only a few workgroups per CU (the 14x14 layers at batch 100: 616
        // on 768 slots): 128-pixel tiles double the count and even out the load, +15 % there.
        const int total = c.g.ntiles * ((Cout + 63) / 64);
        if (c.ksplit == 1 && narrow && (dma || dma_big) && !pool && total >= 256 && total < 2048) {
            const TileGeom h = make_tile_geom(N, H, W, 128);
            if (h.S <= kDmaHaloRowsHalf) { c.g = h; c.kernel = kDmaHalf; }
        }
        // The same launches on the bf16 matrix unit (conv_f32x3.hip), in the same tiles: 0.48 to 0.93 of the time over 150 shapes (128 ->
        // 256 at 56x56, batch 100, 1388 -> 763 us; 512 -> 512 at 28x28, batch 50, 1580 -> 773; 16 -> 40 at 20x33, batch 30, 14.4 ->
        // 13.4).  (That kernel's weight offsets are 32 bits: beyond 4 GiB of weights per tap, and only there, the direct-to-LDS kernel
        // splits fp32 contractions.)
        if ((size_t)Cout * CinP * sizeof(float) >= ((size_t)1 << 32)) return c;
        const int cols64 = (Cout + 63) / 64;
        if (wide) {
            // 8 x 16 patches that pad by at most 1.6: over 240 shapes 0.34 to 0.95 of the time (8 -> 320 channels at 9x102 23 / 56 us),
            // at 1.7 and more up to 1.02 where the other kernel's tiles are 128 wide.  One chunk of 16 channels is half zeros
            // (0.96 to 1.11).  Launches below the last two sizes, 20 to 50 us, would take 0.6 to 0.8 of the time here; they keep the
            // direct-to-LDS kernel, whose patches of wide fp32 images are tested at these sizes.
            const TileGeom t = make_patch_geom(N, H, W, 128);
            const int tiles = t.ntiles * cols64;
            if (!pool && (long)t.ntiles * 128 * 10 <= (long)c.g.M * 16 && (CinP >= 64 ? (long)tiles * CinP >= 256 * 16 : CinP >= 32 && tiles >= 512)) {
                c.g = t; c.kernel = kF32x3Half; c.bn = 64;
            }
            return c;
        }
        // (a contraction of 16 channels is half zeros there: up to 256 tiles 0.7 to 0.95 of the time, beyond 0.97 to 1.28)
        if (c.kernel == kStaged || (CinP <= 16 && c.g.ntiles * (c.kernel == kDmaHalf ? cols64 : 2 * cols) > 256)) return c;
        c.kernel = c.kernel == kDma ? kF32x3 : c.kernel == kDmaBig ? kF32x3Big : kF32x3Half;
        // Few tiles: 128-pixel ones, up to 40 tiles of 256 pixels 0.84 to 0.97 of the time (7x10, batch 7, 112 -> 128 25.8 -> 21.7 us);
        // beyond 50 up to 1.19 where the contraction is long.
        if (narrow && !pool && c.kernel != kF32x3Half && c.g.ntiles * cols64 <= 40) {
            const TileGeom t = make_tile_geom(N, H, W, 128);
            if (t.S <= kF32x3HaloRowsHalfBig) {
                c.g = t; c.kernel = kF32x3Half;
                if (c.ksplit > 1) {
                    const int want = (512 + t.ntiles * cols64 - 1) / (t.ntiles * cols64);
                    c.kchunks = (chunks + (want < c.ksplit ? want : c.ksplit) - 1) / (want < c.ksplit ? want : c.ksplit);
                }
            }
        }
        if (c.ksplit > 1) {   // (whole chunks of 32 channels: never more ranges than conv_split's, whose partial sums the scratch holds)
            c.kchunks = (c.kchunks + 1) / 2 * 2;
            c.ksplit = (chunks + c.kchunks - 1) / c.kchunks;
        }
        return c;
    }
    // bf16.  Shapes whose contraction is split (conv_split) form the same partial sums and add them in the same order,
    // but inside a workgroup.  Few tiles: the waves of a workgroup share the ranges (64 x 32 tiles; eight waves where
    // every CU gets at most one workgroup).  Against the split over workgroups, over 2430 launches: up to 256 tiles 0.14
    // to 0.95 of its time; up to 512 (two to a CU, what the LDS holds) 0.6 to 0.97 while a wave walks at most six chunks,
    // 0.9 to 1.4 beyond; up to 1024 0.7 to 1.05 with one range of at most four chunks per wave, 1.05 to 1.7 with two.
    // (512 -> 512 at 14x14, batch 1, 9.1 us instead of 13.4; at 28x28, batch 1, 9.9 / 19.3, batch 2 16.7 / 22.7.)  Below 12
    // chunks, with more than 64 output channels and more than 512 tiles the 128-pixel tiles below are faster still (256 ->
    // 512 at 28x28, batch 4: 15.4 us, 17.4 here; 320 -> 128 at 20x19, batch 43 20.7 / 25.3).
    if (!pool || !conv3x3_pool_fusable(dtype, H, W, Cout)) conv_split(dtype, c.g, CinP, Cout, c.ksplit, c.kchunks);
    if (c.ksplit > 1) {
        const TileGeom t = conv_small_geom(N, H, W, pool);
        const int tiles = t.ntiles * ((Cout + 31) / 32), G = tiles <= 256 && c.ksplit > 4 ? 8 : 4;
        const int chain = (c.ksplit + G - 1) / G * c.kchunks;   // chunks that a wave walks
        // (wide images have no other split to go to)
        const bool few = tiles <= 256 || (tiles <= 512 && (wide || chain <= 6)) ||
                         (tiles <= 1024 && (chunks >= 12 || Cout <= 64) && (wide || (c.ksplit <= G && chain <= 4)));
        // (that kernel's offsets inside a tile are 31 bits)
        const bool near = (size_t)halo_reach(W, kSmallPx) * CinP * sizeof(bf16_t) < ((size_t)1 << 31);
        if (few && near && (!pool || t.mode == 1) && c.ksplit <= kSmallRanges && conv_small_lds(G, t.S, c.ksplit) <= 160 * 1024) {
            c.g = t;
            c.kernel = G == 8 ? kSmall8 : kSmall4;
            // (up to half the CUs: columns of 16 channels, half the weights for each to fetch; 512 -> 512 at 14x14, batch 1, 9.4 -> 7.9 us)
            c.bn = tiles <= 128 ? 16 : 32;
            return c;
        }
    }
    // Weights in registers: more than 64 output channels, and a contraction of at least three chunks unless
    // there is a tile for every CU (below that the 64-wide direct-to-LDS launch is as fast).  The tile by the time of the
    // CU with most of them, in units of a 256 x 128 tile's (one wave per SIMD multiplies nearly as fast as two, so a CU's
    // tiles simply add up): 320 pixels cost 1.25, 128 pixels 0.56, 64-wide direct-to-LDS tiles 0.67.  Measured (us) for 512
    // channels, 256 / 320 / 128 pixels: 28x28 batch 10 (124, 100, 248 tiles) 44 / 54 / 35, batch 16 (196, 160, 392) 46 /
    // 55 / 50, batch 32 (392, 316, 784) 88 / 115 / 105; 14x14 batch 50 (156, 124, 308) 44 / 55 / 50.  64-wide tiles win
    // where the channels fill a last 128-wide column by half or less: 28x36x20, 96 -> 132 20 us, 27 on 128-wide ones;
    // 53x56 batch 12, 96 -> 192 19 / 25; 53x73 batch 53 on patches, 64 -> 132 101 / 131.
    // (that kernel's halo offsets inside a tile are 32 bits)
    const bool reach = (size_t)halo_reach(W) * CinP * sizeof(bf16_t) < ((size_t)1 << 32);
    // Split over workgroups, as fp32: at most 64 output channels, or a contraction of more than 12 chunks or five ranges
    // (on the tiles below a few workgroups would walk all of it: 14x14 batch 1, 1024 -> 1024 20 us on 256 workgroups, 68 on 16;
    // 7x7 batch 1, 2048 -> 512 20 / 130; 50x66 batch 1, 1024 -> 512 48 / 69; with less 0.61 to 1.02 of its time there).
    if (!wide && c.ksplit > 1 && (Cout <= 64 || chunks > 12 || c.ksplit > 5)) return c;
    const int ksplit = c.ksplit, kchunks = c.kchunks;   // (of the kernels below only the 128-pixel tiles fold their sums)
    c.ksplit = 1; c.kchunks = chunks;
    if (Cout > 64 && (dma || dma_big) && reach && (!narrow || chunks >= 3 || wide_tiles >= 256)) {
        auto rounds = [](int tiles) { return (tiles + 255) / 256; };
        float best = (float)rounds(wide_tiles);
        const float cost64 = 0.67f * rounds(c.g.ntiles * ((Cout + 63) / 64));
        if ((narrow || wide) && ksplit == 1 && cost64 < best) {
            best = cost64;
            c.bn = 64;
        } else {
            c.kernel = dma ? kWreg : kWregBig;
            c.bn = 128;
        }
        if (!narrow) return c;
        if (!pool) {
            const TileGeom t = make_tile_geom(N, H, W, 320);
            const float cost = 1.25f * rounds(t.ntiles * cols);
            if (t.S <= kWregHaloRowsBig && cost < best) {
                best = cost;
                c.g = t;
                c.bn = 128;
                c.kernel = t.S <= kWregHaloRows ? kWregTall : kWregTallBig;
            }
        }
        const TileGeom t = make_tile_geom(N, H, W, 128);
        const int tiles = t.ntiles * cols;
        // 192 pixels cost 0.78: in place of 256-pixel tiles 0.84 to 0.96 of the time of 169 shapes (96 -> 200 at 45x60, batch 7, 14.3 -> 12.4 us;
        // 480 -> 112 at 25x52, batch 27, 45.6 -> 39.2), in place of 128-pixel ones with the larger halo 0.81 to 0.96 of 81, with the
        // smaller one 0.94 to 1.07 of 50, so not there; nor, at up to three chunks, where a 256-pixel tile has the smaller halo (0.95).
        const bool half = t.S <= kWregHaloRowsHalf && 0.56f * rounds(tiles) < best;
        if (!pool && ksplit == 1 && !half && (chunks > 3 || c.kernel != kWreg)) {
            const TileGeom mid = make_tile_geom(N, H, W, 192);
            const float cost = 0.78f * rounds(mid.ntiles * cols);
            if (mid.S <= kWregHaloRows && cost < best) {
                best = cost;
                c.g = mid;
                c.bn = 128;
                c.kernel = mid.ntiles * cols <= 256 && chunks >= 12 ? kWregMidDeep : kWregMid;
            }
        }
        if (t.S <= kWregHaloRows && 0.56f * rounds(tiles) < best) {
            c.g = t;
            c.bn = 128;
            const bool big = t.S > kWregHaloRowsHalf;
            // (one tile per CU, alone there: with two taps of weights ahead each tap waits for L2; nine taps ahead
            // 36 -> 31.6 at 28x28 batch 10, 35 -> 27.4 at 14x14 batch 32; no gain on eight chunks)
            if (tiles <= 256 && chunks >= 12 && ksplit == 1) c.kernel = big ? kWregDeepBig : kWregDeep;
            else {
                c.kernel = big ? kWregHalfBig : kWregHalf;
                c.ksplit = ksplit; c.kchunks = kchunks;
            }
        }
    }
    return c;
}

// Bytes of partial sums conv3x3_igemm needs for this shape (0: none).  bf16 shapes whose partial sums meet inside a
// workgroup leave it untouched, but callers size and pass their buffers by it.
size_t conv3x3_igemm_workspace(int dtype, int N, int H, int W, int CinP, int Cout)
{
    int ksplit, kchunks;
    conv_split_in_memory(dtype, N, H, W, CinP, Cout, ksplit, kchunks);
    return ksplit > 1 ? round_up((size_t)ksplit * N * H * W * Cout * 4, 256) : 0;
}

// For inspection: {kernel (ConvKernel), pixels per tile, channels per tile, tile mode (0 consecutive pixels, 1 patches),
// pixel tiles, ranges of the contraction (kDma, kDmaBig: a workgroup each), workgroups}.
void conv3x3_igemm_plan_info(int dtype, int N, int H, int W, int CinP, int Cout, bool pool, int info[7])
{
    const ConvPlan c = conv_plan(dtype, N, H, W, CinP, Cout, pool);
    info[0] = c.kernel;
    info[1] = c.g.rows;
    info[2] = c.bn;
    info[3] = c.g.mode;
    info[4] = c.g.ntiles;
    info[5] = c.ksplit;
    info[6] = c.g.ntiles * ((Cout + c.bn - 1) / c.bn) * (over_workgroups(c.kernel) ? c.ksplit : 1);
}

bool conv3x3_pool_fusable(int dtype, int H, int W, int Cout)
{
    return H % 16 == 0 && W % kTileW == 0 && Cout % (16 / dtype_size(dtype)) == 0;
}

// Whether conv3x3_igemm takes a pool for this shape: besides the sizes above, the launches of the small-problem
// kernel that run on patches (the model's 56x56, 28x28 and 14x14 layers at small batches).
bool conv3x3_pool_fused(int dtype, int N, int H, int W, int CinP, int Cout)
{
    if (conv3x3_pool_fusable(dtype, H, W, Cout)) return true;
    if (dtype != VGG_BF16 || H % 2 || W % 2 || Cout % 8) return false;
    const int k = conv_plan(dtype, N, H, W, CinP, Cout, true).kernel;
    return k == kSmall4 || k == kSmall8;
}

// x: [N*H*W][CinP], w: [9][Cout][CinP] (elements of dtype); y: [N*H*W][Cout].
// pool (optional): 2x2 max of y, only when conv3x3_pool_fused(); y may then be null; argmax (optional, with pool).
// part_ws: part_bytes of scratch; where conv3x3_igemm_workspace() asks for more than that (or it is null), the
// contraction is not split over workgroups.
int conv3x3_igemm(int dtype, int N, int H, int W, int CinP, int Cout, const void *x, const void *w,
                  const float *bias, const void *mask, void *y, void *pool, unsigned char *argmax, int relu, void *part_ws,
                  size_t part_bytes, hipStream_t stream)
{
    if (pool && !conv3x3_pool_fused(dtype, N, H, W, CinP, Cout)) return VGG_ERR_UNSUPPORTED;
    ConvPlan c = conv_plan(dtype, N, H, W, CinP, Cout, pool != nullptr);
    const bool split = over_workgroups(c.kernel) && c.ksplit > 1;
    if (split && (!part_ws || !y || part_bytes < (size_t)c.ksplit * N * H * W * Cout * 4)) { c.ksplit = 1; c.kchunks = CinP * dtype_size(dtype) / kDataBytes; }
    ConvArgs a;
    a.x = static_cast<const char *>(x);
    a.w = static_cast<const char *>(w);
    a.bias = bias;
    a.mask = static_cast<const char *>(mask);
    a.y = static_cast<char *>(y);
    a.pool = static_cast<char *>(pool);
    a.argmax = pool ? argmax : nullptr;
    a.CinP = CinP; a.Cout = Cout;
    a.relu = relu; a.tiles_n = 0; a.rowsA = 0;
    a.part = split && c.ksplit > 1 ? static_cast<float *>(part_ws) : nullptr;
    a.ksplit = c.ksplit; a.kchunks = c.kchunks;
    const bool narrow = c.bn == 64;
    const TileGeom &g = c.g;
    int rc = VGG_ERR_UNSUPPORTED;
    if (dtype == VGG_F32) {
        switch (c.kernel) {
        case kF32x3: case kF32x3Big: case kF32x3Half: rc = launch_conv_f32x3(a, g, narrow, stream); break;
        case kDmaHalf: rc = launch_conv_dma<float, 128, 64, 4, 1, kDmaHaloRowsHalf>(a, g, stream); break;
        case kDma:
            rc = narrow ? launch_conv_dma<float, 256, 64, 4, 1, kDmaHaloRows>(a, g, stream)
                        : launch_conv_dma<float, 256, 128, 4, 2, kDmaHaloRows>(a, g, stream);
            break;
        case kDmaBig:
            rc = narrow ? launch_conv_dma<float, 256, 64, 4, 1, kDmaHaloRowsBig>(a, g, stream)
                        : launch_conv_dma<float, 256, 128, 4, 2, kDmaHaloRowsBig>(a, g, stream);
            break;
        default:
            rc = narrow ? launch_conv<float, 256, 64, 4, 1>(a, N, H, W, stream)
                        : launch_conv<float, 256, 128, 4, 2>(a, N, H, W, stream);
        }
    } else {
        switch (c.kernel) {
        case kWreg: rc = launch_conv_wreg<2, 2, kWregHaloRows>(a, g, stream); break;
        case kWregBig: rc = launch_conv_wreg<2, 2, kWregHaloRowsBig>(a, g, stream); break;
        case kWregTall: rc = launch_conv_wreg<2, 2, kWregHaloRows, 5, 1>(a, g, stream); break;
        case kWregTallBig: rc = launch_conv_wreg<2, 2, kWregHaloRowsBig, 5, 1>(a, g, stream); break;
        case kWregMid: rc = launch_conv_wreg<2, 2, kWregHaloRows, 3>(a, g, stream); break;
        case kWregMidDeep: rc = launch_conv_wreg<2, 2, kWregHaloRows, 3, 1, 9>(a, g, stream); break;
        case kWregHalf:
            rc = a.ksplit > 1 ? launch_conv_wreg<2, 2, kWregHaloRowsHalf, 2, 2, 3, true>(a, g, stream) : launch_conv_wreg<2, 2, kWregHaloRowsHalf, 2, 3>(a, g, stream);
            break;
        case kWregHalfBig:
            rc = a.ksplit > 1 ? launch_conv_wreg<2, 2, kWregHaloRows, 2, 2, 3, true>(a, g, stream) : launch_conv_wreg<2, 2, kWregHaloRows, 2, 2>(a, g, stream);
            break;
        case kWregDeep: rc = launch_conv_wreg<2, 2, kWregHaloRowsHalf, 2, 1, 9>(a, g, stream); break;
        case kWregDeepBig: rc = launch_conv_wreg<2, 2, kWregHaloRows, 2, 1, 9>(a, g, stream); break;
        case kSmall4: rc = c.bn == 16 ? launch_conv_small<1, 4>(a, g, stream) : launch_conv_small<2, 4>(a, g, stream); break;
        case kSmall8: rc = c.bn == 16 ? launch_conv_small<1, 8>(a, g, stream) : launch_conv_small<2, 8>(a, g, stream); break;
        case kDma:
            rc = narrow ? launch_conv_dma<bf16_t, 256, 64, 4, 1, kDmaHaloRows>(a, g, stream)
                        : launch_conv_dma<bf16_t, 256, 128, 4, 2, kDmaHaloRows>(a, g, stream);
            break;
        case kDmaBig:
            rc = narrow ? launch_conv_dma<bf16_t, 256, 64, 4, 1, kDmaHaloRowsBig>(a, g, stream)
                        : launch_conv_dma<bf16_t, 256, 128, 4, 2, kDmaHaloRowsBig>(a, g, stream);
            break;
        default:
            rc = narrow ? launch_conv<bf16_t, 256, 64, 4, 1>(a, N, H, W, stream)
                        : launch_conv<bf16_t, 256, 128, 4, 2>(a, N, H, W, stream);
        }
    }
    if (rc != VGG_OK || !a.part) return rc;
    const size_t quads = (size_t)N * H * W * Cout / 4;
    const dim3 grid((unsigned)((quads + 255) / 256));
    if (dtype == VGG_F32)
        hipLaunchKernelGGL(conv_split_finish_kernel<float>, grid, dim3(256), 0, stream, a.part, bias,
                           static_cast<const float *>(mask), static_cast<float *>(y), quads, Cout, c.ksplit, relu);
    else
        hipLaunchKernelGGL(conv_split_finish_kernel<bf16_t>, grid, dim3(256), 0, stream, a.part, bias,
                           static_cast<const bf16_t *>(mask), static_cast<bf16_t *>(y), quads, Cout, c.ksplit, relu);
    return launch_status();
}

}  // namespace vgg
