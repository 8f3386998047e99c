// Host-side brute-force check of the tile geometry used by the convolution kernels
// (paper_1810_09868_amd/csrc/common.h): for every tile of every listed shape, every tile row
// must be a distinct output pixel, every pixel must be covered exactly once, and the halo row
// that each of the nine taps reads must hold exactly the neighbouring input pixel, or be a
// zero row when the neighbour lies outside the image.  Prints "ok <count>" or the first error.
#include <cstdio>
#include <vector>

#include "../../paper_1810_09868_amd/csrc/common.h"

using namespace vgg;

// patch: patches whether or not they divide the image
static long check(int N, int H, int W, int rows, bool patch = false)
{
    const TileGeom g = patch ? make_patch_geom(N, H, W, rows) : make_tile_geom(N, H, W, rows);
    std::vector<int> seen((size_t)g.M, 0);
    long taps = 0;
    for (int t = 0; t < g.ntiles; ++t) {
        const TileOrigin o = tile_origin(g, t);
        // what the 32-bit offsets of the halo copies count from and how far they go
        const int first = halo_first_pixel(g, o);
        for (int i = 0; i < g.S; ++i) {
            const int px = halo_pixel(g, o, i);
            if (px >= 0 && (px < first || px - first >= halo_reach(W, rows))) { printf("halo pixel %d is out of reach of %d N%d H%d W%d rows%d\n", px, first, N, H, W, rows); return -1; }
        }
        for (int j = 0; j < rows; ++j) {
            int m, hrow;
            tile_row(g, o, j, m, hrow);
            if (m != tile_pixel(g, o, j)) { printf("tile_pixel mismatch N%d H%d W%d rows%d tile%d j%d\n", N, H, W, rows, t, j); return -1; }
            if (m < 0) continue;
            if (m >= g.M || seen[m]++) { printf("pixel %d bad/duplicate N%d H%d W%d rows%d\n", m, N, H, W, rows); return -1; }
            const int n = m / (H * W), h = (m / W) % H, w = m % W;
            for (int kh = 0; kh < 3; ++kh)
                for (int kw = 0; kw < 3; ++kw) {
                    const int i = hrow + kh * g.pitch + kw;
                    if (i < 0 || i >= g.S) { printf("halo row %d outside [0,%d) N%d H%d W%d rows%d tile%d j%d\n", i, g.S, N, H, W, rows, t, j); return -1; }
                    const int hh = h + kh - 1, ww = w + kw - 1;
                    const int want = (hh < 0 || hh >= H || ww < 0 || ww >= W) ? -1 : (n * H + hh) * W + ww;
                    const int got = halo_pixel(g, o, i);
                    if (got != want) { printf("tap (%d,%d) of pixel %d reads %d, wants %d (N%d H%d W%d rows%d)\n", kh, kw, m, got, want, N, H, W, rows); return -1; }
                    ++taps;
                }
        }
    }
    for (int m = 0; m < g.M; ++m)
        if (!seen[m]) { printf("pixel %d not covered N%d H%d W%d rows%d\n", m, N, H, W, rows); return -1; }
    return taps;
}

// The halo size is found on one period of tiles: against all of them, on sizes drawn at random.
static bool check_period()
{
    unsigned long long seed = 88172645463325252ull;
    auto draw = [&](int n) { seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17; return (int)(seed % (unsigned)n) + 1; };
    for (int k = 0; k < 40000; ++k) {
        const int rows = (const int[]){64, 128, 192, 256, 320}[draw(5) - 1], N = draw(40), H = draw(k % 3 ? 40 : 200), W = draw(k % 5 ? 70 : 300);
        const TileGeom g = make_tile_geom(N, H, W, rows);
        if (g.mode) continue;
        auto q = [&](int m) { return ((long)(m / (H * W)) * (H + 1) + m % (H * W) / W) * (W + 1) + m % W; };
        long best = 0;
        for (int m0 = 0; m0 < g.M; m0 += rows) {
            const long span = q(m0 + rows < g.M ? m0 + rows - 1 : g.M - 1) - q(m0);
            if (span > best) best = span;
        }
        if (g.S != best + 2 * (W + 2) + 1) { printf("halo of N%d H%d W%d rows%d: %d rows, needs %ld\n", N, H, W, rows, g.S, best + 2 * (W + 2) + 1); return false; }
    }
    return true;
}

// fast_div against the division it replaces: every small divisor, a few large ones, numerators
// around every multiple of the divisor they can reach plus the top of the 31-bit range.
static bool check_fast_div()
{
    std::vector<int> ds;
    for (int d = 1; d <= 3000; ++d) ds.push_back(d);
    for (int d : {50176, 50177, 65535, 65536, 65537, 1000003, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, 2147483647}) ds.push_back(d);
    for (int d : ds) {
        const FastDiv f = make_fast_div(d);
        auto ok = [&](long long n) {
            if (n < 0 || n > 2147483647ll) return true;
            if (fast_div((int)n, f) != (int)(n / d)) { printf("fast_div(%lld, %d) = %d\n", n, d, fast_div((int)n, f)); return false; }
            return true;
        };
        for (long long n = 0; n < 4096; ++n) if (!ok(n)) return false;
        for (long long k = 1; k <= 2147483647ll / d; k += 1 + k / 7)
            for (int e = -1; e <= 1; ++e) if (!ok(k * d + e)) return false;
        const long long top = 2147483647ll / d * d;
        for (int e = -2; e <= 2; ++e) if (!ok(top + e)) return false;
        for (long long n = 2147483647ll - 64; n <= 2147483647ll; ++n) if (!ok(n)) return false;
    }
    return true;
}

int main()
{
    if (!check_fast_div() || !check_period()) return 1;
    const int shapes[][3] = {{2, 224, 224}, {3, 112, 112}, {5, 56, 56}, {7, 28, 28}, {100, 14, 14}, {9, 14, 14}, {3, 5, 7},
                             {1, 2, 2}, {4, 1, 1}, {2, 3, 300}, {2, 300, 3}, {5, 16, 48}, {1, 32, 32}, {2, 17, 16}, {1, 8, 16},
                             {3, 24, 16}, {2, 40, 48}, {3, 50, 66}, {1, 24, 200}, {2, 31, 33}};
    long total = 0;
    for (auto &s : shapes)
        for (int rows : {64, 128, 192, 256, 320})
            for (bool patch : {false, true}) {
                const long c = check(s[0], s[1], s[2], rows, patch);
                if (c < 0) return 1;
                total += c;
            }
    printf("ok %ld\n", total);
    return 0;
}
