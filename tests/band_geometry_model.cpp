// The work items that csrc/conv_band.hpp and csrc/conv_band_grads.hpp cut maps into, over maps of every proportion the library
// accepts: they cover the map, fit the kernels' LDS and registers, and a staging unit's place survives being packed.  Host side
// of the headers only, no GPU.  Built and run by tests/test_host_path_cpu.py.
#include <cstdio>
#include <type_traits>

#include "../paper_1611_06256_amd/csrc/conv_band_grads.hpp"

using namespace ga3c;

extern "C" {      // what the headers' kernels register themselves with
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}

static int problems = 0, maps = 0, most_rows = 0;
#define PROBLEM(...) do { if (++problems <= 20) { printf("problem: " __VA_ARGS__); printf("\n"); } } while (0)

// rows of the map 0 .. rows - 1 in items of R rows, nb of them per frame
static void covered(const char *what, int rows, int R, int nb, int H, int W, int n) {
    if (R < 1 || nb < 1 || (long)R * nb < rows || (long)R * (nb - 1) >= rows) PROBLEM("%s of %d frames of %dx%d: %d items of %d rows for %d", what, n, H, W, nb, R, rows);
}

template <int OC, bool ONE>
static void dgrad(int n, int H, int W) {
    BandGeom b = band_geom(H, W);
    if (!band_dgrad_geom<OC, ONE>(b, n)) { PROBLEM("input gradient of %dx%d, %d filters: no geometry", H, W, OC); return; }
    covered("input gradient", (H + 1) / 2, b.R, b.nb, H, W, n);
    if (b.F > 1 && b.nb > 1) PROBLEM("several frames and bands of one in an item");
    const int PW = b.cols + 1, RL = b.R + 1, PIT = band_dgrad_pitch<OC, ONE>(), lds = b.F * RL * PW * PIT;
    if (lds > (OC == 32 ? BAND_HALF_LDS : BAND_LDS - 2048)) PROBLEM("input gradient of %dx%d, %d filters: %d bytes of LDS", H, W, OC, lds);
    if (b.F * RL * b.OW * (OC / 8) > 256 * band_dgrad_maxu<OC>()) PROBLEM("input gradient of %dx%d, %d filters: too many units", H, W, OC);
    most_rows = b.R > most_rows ? b.R : most_rows;
    if (BandDgradUnit::none().any()) PROBLEM("no unit is one");
    for (int f = 0; f < b.F; f += b.F > 1 ? b.F - 1 : 1)
        for (int r = 0; r <= b.R; ++r)
            for (int xc : {0, b.OW - 1})
                for (int cg : {0, OC / 8 - 1}) {
                    const uint32_t byte = ((uint32_t)(f * RL + r) * PW + xc + 1) * PIT + 16 * cg;
                    const BandDgradUnit u = BandDgradUnit::at(byte, r);
                    if (!u.any() || u.byte() != (int)byte || u.row() != r) {
                        PROBLEM("input gradient of %d frames of %dx%d, %d filters, %s: row %d at byte %u comes back as row %d at byte %d", n, H, W, OC,
                                ONE ? "one term" : "three terms", r, byte, u.row(), u.byte());
                        return;
                    }
                }
}

template <int OC, bool ONE>
static void wgrad(int n, int H, int W) {
    BandWgradGeom b{};
    if (!band_wgrad_geom<OC, ONE>(b, n, H, W)) { PROBLEM("weight gradient of %dx%d, %d filters: no geometry", H, W, OC); return; }
    covered("weight gradient", b.OH, b.R, b.nb, H, W, n);
    if (band_wgrad_lds(b, b.R, ONE) > BAND_LDS - 2048) PROBLEM("weight gradient of %dx%d: %d bytes of LDS", H, W, band_wgrad_lds(b, b.R, ONE));
    if ((2 * b.R + 2) * 16 * b.nx > 256 * BAND_WGRAD_MAXX || 32 * b.R * b.NO > 256 * BAND_WGRAD_MAXD) PROBLEM("weight gradient of %dx%d: too many units", H, W);
    if (b.nbx > 8192 / OC || b.nbx > b.items) PROBLEM("weight gradient of %dx%d: %d partial gradients", H, W, b.nbx);
}

static void map(int n, int H, int W) {
    if (!band_ok<32>(H, W) || !band_grads_ok(H, W)) return;      // as the library decides
    ++maps;
    BandGeom b = band_geom(H, W);
    if (!band_fwd_geom<32>(b, n)) { PROBLEM("forward pass of %dx%d: no geometry", H, W); return; }
    covered("forward pass", b.OH, b.R, b.nb, H, W, n);
    dgrad<32, false>(n, H, W); dgrad<32, true>(n, H, W); dgrad<64, false>(n, H, W); dgrad<64, true>(n, H, W);
    wgrad<32, false>(n, H, W); wgrad<32, true>(n, H, W); wgrad<64, false>(n, H, W); wgrad<64, true>(n, H, W);
}

int main() {
    for (int n : {1, 3, 40, 255, 256, 257, 511, 512, 640, 2560, 100000})
        for (int W : {4, 5, 6, 7, 8, 9, 12, 16, 26, 37, 50, 77, 84, 120, 160})
            for (int H = 4; H <= 1400; H += H < 90 || (H >= 497 && H < 700) ? 1 : 37) map(n, H, W);
    printf("%d maps, at most %d rows an item, %d problems\n", maps, most_rows, problems);
    return problems || maps < 1000 || most_rows != BAND_DGRAD_MAXR ? 1 : 0;
}
