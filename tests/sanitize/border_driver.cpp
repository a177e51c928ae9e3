// The units of the adjoint's mirror pass, on the host with the kernel's own
// index code: for frames of every border mode and padding, the units visit each
// pixel that padded rows or columns fold onto exactly once in every channel,
// no pixel twice and none outside the frame.  "ok" on the last line.
#include "dppix_internal.h"

#include <stdio.h>

#include <vector>

using namespace dppix;

static long frames = 0, bad = 0;

static void check(int H, int W, int C, int b, int pad)
{
    ++frames;
    FrameRec F{};
    F.H = H;
    F.W = W;
    F.C = C;
    F.b = b;
    F.pad = pad;
    F.GR = (H + b - 1) / b;
    F.GC = (W + b - 1) / b;
    const BorderArea m = border_area(F);
    std::vector<int> seen((size_t)C * H * W, 0);
    const int64_t units = (int64_t)C * (border_parts(m.nA) + border_parts(m.nB));
    for (int64_t u = 0; u < units; ++u) {
        const BorderPart part(m, W, (int)u);
        for (int k = 0; k < part.n; ++k) {
            int y, x;
            part.pixel(m, k, [&](int v) { return v / (int)part.wide; }, y, x);
            if (part.ch < 0 || part.ch >= C || y < 0 || y >= H || x < 0 || x >= W || part.n > (int)kBorderPixels) {
                ++bad;
                continue;
            }
            ++seen[((size_t)part.ch * H + y) * W + x];
        }
    }
    std::vector<char> row(H, 0), col(W, 0);
    for (int y = H; y < F.GR * b; ++y)
        row[fold(y, H, pad)] = 1;
    for (int x = W; x < F.GC * b; ++x)
        col[fold(x, W, pad)] = 1;
    for (int c = 0; c < C; ++c)
        for (int y = 0; y < H; ++y)
            for (int x = 0; x < W; ++x) {
                const int n = seen[((size_t)c * H + y) * W + x];
                if (n > 1 || (n == 0 && (row[y] || col[x]))) {
                    if (++bad < 20)
                        printf("%d visits of (%d, %d, %d): H %d W %d b %d pad %d\n", n, c, y, x, H, W, b, pad);
                }
            }
}

int main()
{
    static const int bs[] = {1, 2, 3, 4, 8, 16, 24, 64, 100, 256};
    static const int sides[] = {1, 2, 3, 5, 8, 15, 16, 17, 31, 33, 64, 65, 127, 128, 129, 200, 257, 300};
    for (int pad = 0; pad < 2; ++pad)
        for (int b : bs)
            for (int H : sides)
                for (int W : sides)
                    check(H, W, 1 + (H + W) % 3, b, pad);
    check(1030, 2050, 3, 256, 0);
    check(2050, 1030, 2, 256, 1);
    printf("%ld frames, %ld wrong\n", frames, bad);
    printf(bad ? "failed\n" : "ok\n");
    return bad != 0;
}
