// Stages one block of label rows on the host, with the index code of the
// label kernels (LabPlace), for every walk that frames of the given widths
// have: every write stays in its own row, every column that the stencil reads
// holds the sum of the pixel that it mirrors, and every source vector lies in
// the frame.  Built with AddressSanitizer; "ok" on the last line.
#include "dppix_internal.h"

#include <stdio.h>

#include <algorithm>
#include <vector>

using namespace dppix;

static long walks = 0, bad = 0;

static uint16_t sum_of(int column) { return (uint16_t)(1 + column % 60000); }

static void fail(const char* what, int W, int b, int K, int pad, int px0, int cols)
{
    if (++bad <= 20)
        printf("%s: W %d b %d K %d pad %d px0 %d cols %d\n", what, W, b, K, pad, px0, cols);
}

// threads: of the workgroup
static void walk(int W, int b, int K, int pad, int px0, int cols, int threads)
{
    ++walks;
    const int stride = label_stride(4 * threads), G = label_groups(cols);
    if (G * kLabBlock > threads || (cols + 3) / 4 > threads)
        fail("lanes", W, b, K, pad, px0, cols);
    for (int row = 0; row < 2; ++row) {
        // row 0 is the first of the allocation, row 1 lies between two others
        std::vector<uint16_t> rows((size_t)stride * (row ? 3 : 1) + 8, 0);
        uint16_t* base = rows.data() + (8 - ((uintptr_t)rows.data() >> 1) % 8) % 8;     // 16-byte aligned, as LDS is
        rows.assign(rows.size(), 0);
        uint16_t* S = base + (size_t)row * stride;
        for (int g = 0; g < G; ++g) {
            LabPlace p;
            p.setup(g, px0, cols, W, pad);
            if (p.kind == kLabNone)
                continue;
            if (p.kind == kLabSingle) {
                for (int c = p.pa; c < p.pb; ++c) {
                    const int at = kLabLeft + c - px0;
                    if (at < 0 || at >= stride)
                        fail("single write outside its row", W, b, K, pad, px0, cols);
                    else
                        S[at] = sum_of(edge_fold(c, W, pad));
                }
                continue;
            }
            if (p.from < 0 || p.from + 16 > W)
                fail("source outside the frame", W, b, K, pad, px0, cols);
            v4u lo, hi;
            for (int i = 0; i < 4; ++i) {
                lo[i] = sum_of(p.from + 2 * i) | (uint32_t)sum_of(p.from + 2 * i + 1) << 16;
                hi[i] = sum_of(p.from + 8 + 2 * i) | (uint32_t)sum_of(p.from + 9 + 2 * i) << 16;
            }
            p.put(lo, hi, S, px0, W, pad);
        }
        for (int c = px0 - 1; c <= px0 + cols; ++c)
            if (S[kLabLeft + c - px0] != sum_of(edge_fold(c, W, pad))) {
                fail("staged column", W, b, K, pad, px0, cols);
                break;
            }
        for (uint16_t* q = rows.data(); q < rows.data() + rows.size(); ++q)
            if (*q != 0 && (q < S || q >= S + stride)) {
                fail("write outside its row", W, b, K, pad, px0, cols);
                break;
            }
    }
}

// The walks of the plan from labels, as k_plan_labels cuts a tile of K cells.
static void plan_walks(int W, int b, int K, int pad)
{
    const int GC = (W + b - 1) / b;
    const int threads = label_threads(std::min(K * b, kLabCols));
    const int TX = (GC + K - 1) / K;
    for (int ct = 0; ct < TX; ++ct) {
        if (ct >= 2 && ct + 2 < TX)
            continue;   // (inside the frame they are all alike)
        const int c0 = ct * K, KC = std::min(K, GC - c0), X0 = c0 * b, XW = KC * b;
        const int xend = pad == kPadNone ? std::min(XW, W - X0) : XW;
        for (int cx = 0; cx < xend; cx += kLabCols)
            walk(W, b, K, pad, X0 + cx, std::min(kLabCols, xend - cx), threads);
    }
}

int main()
{
    static const int sides[] = {1, 2, 3, 4, 5, 7, 8, 12, 16, 20, 24, 31, 32, 48, 64, 100, 128, 200, 255, 256};
    for (int pad = 0; pad < 3; ++pad) {
        // label masks: equal chunks of real columns
        for (int W = 1; W <= 4100; W += W < 1030 ? 1 : 11) {
            const int width = label_chunk(W), threads = label_threads(std::min(width, W));
            for (int px0 = 0; px0 < W; px0 += width)
                walk(W, 0, 0, pad, px0, std::min(width, W - px0), threads);
        }
        // plans from labels: tiles of one or a few cells, and as wide as rows of up to 2048 bytes make them
        for (int b : sides)
            for (int W = 1; W <= 2100; W += (W < 40 || (W > 900 && W < 1030) || (W > 1950 && W < 2010)) ? 1 : 23) {
                const int GC = (W + b - 1) / b;
                for (int K : {1, 3, 1000 / b, 1008 / b, 2048 / b, GC})
                    if (K >= 1 && K <= GC)
                        plan_walks(W, b, K, pad);
            }
    }
    printf("%ld walks, %ld wrong\n", walks, bad);
    printf(bad ? "failed\n" : "ok\n");
    return bad != 0;
}
