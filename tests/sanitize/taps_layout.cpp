// The staged layout of the tap-staged bf16 kernel, on the CPU: every strip read of every output pixel and tap finds in
// the stage what the convolution needs there (the channels of one input pixel, or zeros outside the image), for odd
// images, kernels, dilations and tiles, and stays inside the stage; and in the first, middle and last tiles of layers next to
// what the library lets through (pixels and padded rows below 2^24, rows of 3000 pixels, padded granules below 2^31).
#include <cstdio>
#include <vector>

#include "nm_internal.h"

using namespace nm;

static void magic(unsigned d, unsigned* mul, unsigned* shift)
{
    unsigned s = 0;
    while ((1ull << s) < d) ++s;
    *mul = (unsigned)(((1ull << (31 + s)) / d) + 1);
    *shift = s;
}

static long checked = 0;

static bool layer(int B, int H, int W, int kh, int kw, int dh, int dw, int BP, bool sampled = false)
{
    const int ph = dh * (kh - 1) / 2, pw = dw * (kw - 1) / 2;
    const long line = taps_line(W, pw), Hp = H + ph, P = (long)B * H * W;
    unsigned lm, ls, im, is;
    magic((unsigned)line, &lm, &ls);
    magic((unsigned)Hp, &im, &is);
    auto place = [&](long p) { return (p / (H * W) * Hp + p % (H * W) / W) * line + p % W * 9; };
    const long n = (long)taps_loads(taps_granules(BP, H, W, ph, pw)) * 64, tiles = (P + BP - 1) / BP;
    if (sampled && ((B + 2.0) * Hp >= 16777216.0 || (B + 2.0) * Hp * line >= 2147483648.0 || P >= 16777216 || n > 10240)) return false;
    for (long p0 = 0; p0 < P; p0 += BP) {
        const long tile = p0 / BP;
        if (sampled && tile > 2 && tile + 3 < tiles && tile != tiles / 2) continue;
        const long t0 = place(p0) - (ph * line + pw * 9) + Hp * line;
        if (t0 < 0) return false;
        std::vector<TapsSource> stage;
        for (long g = 0; g < n; ++g) {
            stage.push_back(taps_source((unsigned)(t0 + g), (unsigned)line, lm, ls, im, is, B, H, W, ph));
            if (stage.back().pixel >= P) return false;
        }
        for (int l = 0; l < BP; ++l) {
            const long p = p0 + l < P ? p0 + l : P - 1, base = place(p) - place(p0);
            const int b = (int)(p / (H * W)), ho = (int)(p % (H * W) / W), wo = (int)(p % W);
            for (int a = 0; a < kh; ++a)
                for (int c = 0; c < kw; ++c) {
                    const int hi = ho + a * dh - ph, wi = wo + c * dw - pw;
                    const bool in = hi >= 0 && hi < H && wi >= 0 && wi < W;
                    for (unsigned o = 0; o < 8; ++o) {
                        const long at = base + a * dh * line + c * dw * 9 + o;
                        if (at < 0 || at >= n) return false;
                        const TapsSource& s = stage[at];
                        if (in ? s.pixel != (b * H + hi) * W + wi || s.oct != o : s.pixel != -1) return false;
                        ++checked;
                    }
                }
        }
    }
    return true;
}

int main()
{
    for (int B : {1, 3})
        for (int H : {1, 2, 7, 9})
            for (int W : {1, 5, 8, 14, 33})
                for (int k : {1, 2, 3, 4, 5})    // 3x1, 1x3, 3x3, 5x3, 3x3 dilated by 2 and 1
                    for (int BP : {64, 160, 224, 448}) {
                        const int kh = k == 2 ? 1 : k == 4 ? 5 : 3, kw = k == 1 ? 1 : 3, dh = k == 5 ? 2 : 1;
                        if (!layer(B, H, W, kh, kw, dh, 1, BP) || !layer(B, H, W, kh, kw, dh, 2, BP)) {
                            printf("wrong: B %d H %d W %d kernel %dx%d dilation %d tile %d\n", B, H, W, kh, kw, dh, BP);
                            return 1;
                        }
                    }
    struct Far { int B, H, W, kh, kw, dh, dw; };
    for (const Far& f : {Far{8388605, 1, 1, 3, 3, 1, 1}, Far{1, 5592300, 3, 3, 1, 1, 1}, Far{1, 5592, 3000, 1, 3, 1, 1}, Far{3976818, 1, 4, 1, 3, 1, 56},
                         Far{2, 1398000, 6, 3, 3, 1, 1}, Far{1, 5592400, 1, 1, 5, 1, 1}, Far{239, 26000, 2, 5, 1, 2, 1}})
        for (int BP : {64, 128})
            if (!(BP == 128 && f.dw > 2) && !layer(f.B, f.H, f.W, f.kh, f.kw, f.dh, f.dw, BP, true)) {
                printf("wrong: B %d H %d W %d kernel %dx%d dilation %d %d tile %d\n", f.B, f.H, f.W, f.kh, f.kw, f.dh, f.dw, BP);
                return 1;
            }
    printf("taps layout: ok, %ld reads\n", checked);
    return 0;
}
