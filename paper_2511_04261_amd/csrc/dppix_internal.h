// dppix_internal.h — device-side records and launch interfaces of libdppix.
//
// Layout of the work: every frame is cut into bands of b_bg padded rows (one
// row of grid cells) and each band into tiles of K grid cells.  A tile is the
// unit a workgroup processes (Thm. 3 of the paper: cells are independent, so
// any distribution of cells over processing units is valid).  Tiles are
// numbered frame-major, band-major, left to right — which is also row-major
// cell order, the order of the compact store (Table IV).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dppix {

constexpr int kStrip = 16;             // bytes one lane moves per row (dwordx4)
constexpr int kMaxThreads = 512;
constexpr int kMaxB = 256;             // 255 * 256 rows fits a 16-bit lane sum
constexpr int kMaxGroups = 24;         // launch groups: layout x channels x workgroup size
constexpr int kTicketWords = 2 * kMaxGroups;      // two per launch group (resident-grid tickets)

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Unpadded border mode (Algorithm 1): positions past the frame are absent —
// they add nothing to sums or mask counts, and each (sub)cell's mean divides
// by its real pixel count.
constexpr int kPadNone = 2;

// Mirror index of padded coordinate x >= 0 into [0, L).
__host__ __device__ __forceinline__ int fold(int x, int L, int mode)
{
    if (x < L)
        return x;
    if (mode == 0) {
        if (x < 2 * L)          // first mirror image, the common case
            return 2 * L - 1 - x;
        const int p = 2 * L;
        const int y = x % p;
        return y < L ? y : p - 1 - y;
    }
    if (L == 1)
        return 0;
    if (x < 2 * L - 1)
        return 2 * L - 2 - x;
    const int p = 2 * L - 2;
    const int y = x % p;
    return y < L ? y : p - y;
}

// Mirror index of a coordinate in [-1, 2L) for the Sobel stencil: -1 mirrors
// like the frame's own padding, the unpadded mode mirrors like the symmetric one.
__host__ __device__ __forceinline__ int edge_fold(int x, int L, int mode)
{
    if (mode == kPadNone)   // the Sobel stencil mirrors like the symmetric mode
        mode = 0;
    if (x < 0)
        return (mode == 0 || L == 1) ? 0 : 1;
    return fold(x, L, mode);
}

// One frame as the kernels see it (host computes everything derivable).
struct FrameRec {
    int32_t H, W, C, layout;
    int64_t pitch;            // U8: bytes per row; F32: floats per row
    int32_t b, s, n, pad;     // b_bg, b_fg, n = b/s, pad mode
    int32_t GR, GC, K, TX;    // grid rows/cols, cells per tile, tiles per band
    int32_t tau, noise_bg, noise_fg, off32;    // off32: (b + 1) rows of the frame span < 2^31 bytes
    int32_t cnb, ctx, cunits, lnb;            // plan units: bands, tiles per band, units of the frame; bands per unit
                                              // of the plan from labels
    int64_t cell_base;        // first cell of the frame in batch-wide cell arrays
    int64_t fine_base;        // first subcell in dense fine arrays
    int64_t tile_base;        // first tile
    double sigma_bg, sigma_fg;
    uint32_t key0, key1, fi0, fi1;
};

// Units of a batch by frame: entry k says that the k-th frame with units of a
// kind is `frame` and its first unit `first`; the entry after the last holds the
// number of units.  A kernel finds its unit's frame by a search that a wave
// does together, one load for 64 frames, so the table grows with the frames
// alone.  (Maps with an entry per unit were written and uploaded with every
// plan.  dp_pix_plan_create on the host, with them and now: 256 frames of 576 x
// 768 to 4000 x 6000: 6.6 -> 0.41 ms, workspace 6.1 -> 1.5 MB; 64 of 1300 x
// 2050, b 256: 5.7 ms -> 16 us; 16 fp32 of 2161 x 3841, b 256: 451 -> 5 us.)
struct UnitSpan {
    int64_t first;
    int32_t frame, pad_;
};

// The pixels that padded rows or columns fold onto: all columns of rows [ra,
// re) (nA of them), and columns [ca, ce) of the other rows (nB).  A padding
// that folds more than once may reach any row (column).
struct BorderArea {
    int ra, re, ca, ce;
    uint32_t nA, nB;          // (fewer than 256 padded rows or columns: below 2^32)
};

__host__ __device__ inline BorderArea border_area(const FrameRec& F)
{
    const int PR = F.GR * F.b - F.H, PC = F.GC * F.b - F.W;
    const int edge = F.pad == 1 ? 1 : 0;   // the reflected mode does not repeat the last row
    BorderArea m;
    m.ra = PR <= F.H - edge ? F.H - edge - PR : 0;
    m.re = PR <= F.H - edge ? F.H - edge : F.H;
    m.ca = PC <= F.W - edge ? F.W - edge - PC : 0;
    m.ce = PC <= F.W - edge ? F.W - edge : F.W;
    m.nA = (uint32_t)(m.re - m.ra) * (uint32_t)F.W;
    m.nB = (uint32_t)(F.H - (m.re - m.ra)) * (uint32_t)(m.ce - m.ca);
    return m;
}

// A unit of the mirror pass: up to kBorderPixels pixels of one channel and one
// of the two areas, row by row (a lane's loads are two levels deep, so they are
// shared out).
constexpr uint32_t kBorderPixels = 512;
__host__ __device__ inline uint32_t border_parts(uint32_t n) { return n / kBorderPixels + (n % kBorderPixels != 0); }

struct BorderPart {
    int ch, y0, x0;           // channel, and row and column of pixel p0 within the area
    bool rows;                // of the area of whole rows
    uint32_t wide;            // of the area
    int n;                    // pixels

    __host__ __device__ inline BorderPart(const BorderArea& m, int W, int unit)
    {
        const uint32_t parts_a = border_parts(m.nA), parts = parts_a + border_parts(m.nB);
        ch = (int)((uint32_t)unit / parts);
        const uint32_t part = (uint32_t)unit - (uint32_t)ch * parts;
        rows = part < parts_a;
        wide = rows ? (uint32_t)W : (uint32_t)(m.ce - m.ca);
        const uint32_t p0 = (part - (rows ? 0u : parts_a)) * kBorderPixels, left = (rows ? m.nA : m.nB) - p0;
        n = (int)(left < kBorderPixels ? left : kBorderPixels);
        y0 = (int)(p0 / wide);
        x0 = (int)(p0 - (uint32_t)y0 * wide);
    }

    // The frame's row and column of pixel k; by_wide divides by `wide`.
    template <typename Div>
    __host__ __device__ inline void pixel(const BorderArea& m, int k, const Div& by_wide, int& y, int& x) const
    {
        const int q = by_wide(x0 + k);
        y = y0 + q;
        x = x0 + k - q * (int)wide;
        if (rows)
            y += m.ra;
        else {
            y += y < m.ra ? 0 : m.re - m.ra;
            x += m.ca;
        }
    }
};

// Workspace layout of a plan (byte offsets from the bound workspace base):
// tables written once by dp_pix_plan_bind and only read afterwards, so one
// bound plan serves any number of concurrent calls.
struct WsLayout {
    size_t frames;        // FrameRec[n_frames]
    size_t tile_map;      // int32[n_tiles][2]: (frame, tile within frame) per scheduling index
    size_t unit_map;      // int32[n_units][2]: (frame, plan unit within frame), frame-major
    size_t border_spans;  // UnitSpan[fp32 frames + 1]: units of the adjoint's mirror pass
    size_t lab_spans;     // UnitSpan[u8 frames + 1], by channel count: units of the plan from labels
    size_t edge_spans;    // the same of the label masks
    size_t met_spans;     // the same of the metrics
    size_t simple_counts; // uint64[n_frames][4]: store counts of a call without masks (every cell simple)
    size_t total;
};

// Per-call state that travels with a store (byte offsets from store->state):
// what dp_pix_plan (or dp_pix_store_index) derives from the flags beside the
// store's counts, and the ticket words of that call sequence's launches.
struct StateLayout {
    size_t tile_cnt;      // uint32[n_tiles]: complex cells per tile
    size_t tile_fg;       // uint32[n_tiles]: complex cells of the frame before the tile
    size_t counters;      // uint32[kTicketWords]: tickets of persistent launches (two per group)
    size_t total;
};

struct TileArgs {
    const FrameRec* frames;
    const int32_t* tile_map;
    const int32_t* unit_map;
    int32_t n_frames;
    int64_t sched_offset;     // first scheduling index of this launch
    int64_t n_tiles;          // tiles of this launch
    uint32_t* ticket;         // [0]: next tile, [1]: finished workgroups
    int32_t persistent;
    // per-frame pointer tables (device arrays of device pointers)
    const uint8_t* const* masks;
    const uint64_t* simple_counts;   // store counts when no frame has a mask (geometry only)
    int64_t total_cells;             // cells of the whole batch (store flags)
    const void* const* images;
    void* const* outs;
    // products of the plan, held by the caller's store
    uint8_t* flags;           // store flags, 1 = complex cell
    uint64_t* counts;         // store counts: per frame n_bg, n_fg, bg offset, fg offset
    uint32_t* tile_cnt;       // store state: complex cells per tile
    uint32_t* tile_fg;        // store state: complex cells of the frame before the tile
    // per-frame Philox (key, counter) of this call: noise[2f] = seed,
    // noise[2f + 1] = frame_index; NULL: the frame records' own
    const uint64_t* noise;
    // store statistics
    float* bg;
    float* fg;
    uint8_t* clip_bg;
    uint8_t* clip_fg;
    // diagnostics
    uint32_t* dbg_coarse;
    uint32_t* dbg_fine;
    // backward
    const float* const* grad_out;
    float* const* grad_in;
    float* g_bg;              // per-statistic gradient, store layout
    float* g_fg;
    uint32_t* cell_index;     // frame-local store index of every cell
    // complexity label
    uint8_t* const* masks_out;
    int32_t edge_threshold;
    int32_t edge_rows;        // rows of a label mask unit
    // units of the label kernels, the metrics and the mirror pass: the spans
    // of this launch's frames (one more entry than frames)
    const UnitSpan* spans;
    int32_t n_spans;
    int32_t span_units;       // units of each frame if all have as many, else 0
    // utility metrics: per unit (SSIM partial sum, squared-error sum)
    double* met_partial;
    int32_t met_rows;         // rows of a metrics unit
};

// The label kernels stage rows of channel sums in blocks of kLabBlock, a lane
// per 16-pixel group of a block (with a halo group on each side) and a lane
// per four columns: 992 columns are what 256 lanes take.  label_chunk: the
// width of the equal chunks, whole groups, that the label masks cut W columns
// into; label_threads: lanes for walks of up to `cols` columns; label_stride:
// LDS columns of a staged row (the right edge's groups reach past the last).
constexpr int kLabBlock = 4;
constexpr int kLabCols = 992;
constexpr int kLabLeft = 16;                      // LDS columns before column 0
__host__ __device__ inline int label_chunk(int W)
{
    const int n = (W + kLabCols - 1) / kLabCols;
    return ((W + n - 1) / n + 15) & ~15;
}
__host__ __device__ inline int label_threads(int cols) { return (cols / 4 + 8 + 63) & ~63; }
__host__ __device__ inline int label_stride(int cols) { return cols + 64; }
__host__ __device__ inline int label_groups(int cols) { return (cols + 16) / 16 + 1; }   // of a staged row

// One 16-pixel group of the staged columns [px0 - 1, px0 + cols], as a lane
// keeps it from block to block: where its pixels come from and how their sums
// reach the row.  Column x of the frame is staged at kLabLeft + x - px0.
enum LabGroup : int {
    kLabNone,      // nothing of the group is needed
    kLabInside,    // sixteen pixels of the frame
    kLabMirror,    // all past the right edge: the sixteen pixels they mirror, reversed
    kLabCross,     // across the right edge: the frame's last sixteen pixels give both sides
    kLabSingle     // anything else (left halo, narrow frames): pixel by pixel
};

struct LabPlace {
    int kind, x, from;     // first column of the group, first pixel its vectors hold
    int pa, pb;            // columns [pa, pb) of the group that are needed

    __host__ __device__ __forceinline__ void setup(int g, int px0, int cols, int W, int pad)
    {
        x = px0 + 16 * (g - 1);
        pa = x > px0 - 1 ? x : px0 - 1;
        pb = x + 16 < px0 + cols + 1 ? x + 16 : px0 + cols + 1;
        const int mirrored = (pad == 1 ? 2 * W - 2 : 2 * W - 1) - (x + 15);
        from = x;
        if (pa >= pb || (x < 0 && px0 == 0 && W >= 16))
            kind = kLabNone;   // (column -1 is written by the group that holds its mirror image)
        else if (x >= 0 && x + 16 <= W)
            kind = kLabInside;
        else if (x >= W && mirrored >= 0 && mirrored + 16 <= W) {
            kind = kLabMirror;
            from = mirrored;
        } else if (x >= 0 && x < W && W >= 16) {
            kind = kLabCross;
            from = W - 16;
        } else
            kind = kLabSingle;
    }

    __host__ __device__ __forceinline__ bool vector() const { return kind != kLabNone && kind != kLabSingle; }

    // The sums of the sixteen pixels from `from` on (pairs, the first in the
    // low half) into the staged row S.
    __host__ __device__ __forceinline__ void put(v4u lo, v4u hi, uint16_t* S, int px0, int W, int pad) const
    {
        uint16_t* d = S + kLabLeft + x - px0;
        if (__builtin_expect(kind == kLabMirror, 0)) {
            asm volatile("");   // a branch of its own: few lanes reverse
            const v4u a = v4u{hi.w, hi.z, hi.y, hi.x}, b = v4u{lo.w, lo.z, lo.y, lo.x};
            lo = (a >> 16) | (a << 16);
            hi = (b >> 16) | (b << 16);
        }
        if (kind == kLabCross) {
            // sums of the frame's last sixteen columns at their places, and
            // reversed at the places that mirror them (what they overlap of
            // the groups beside them, they write alike).  Where the walk
            // itself starts past the edge, the former lie before the row and
            // no column needs them.
            const bool real = W > px0;
            uint16_t* e = S + kLabLeft + from - px0;
            uint16_t* m = S + kLabLeft + (pad == 1 ? W - 1 : W) - px0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t pr = i < 4 ? lo[i & 3] : hi[i & 3];
                m[15 - 2 * i] = (uint16_t)pr;
                m[14 - 2 * i] = (uint16_t)(pr >> 16);
                if (real) {
                    e[2 * i] = (uint16_t)pr;
                    e[2 * i + 1] = (uint16_t)(pr >> 16);
                }
            }
            return;
        }
        reinterpret_cast<v4u*>(d)[0] = lo;
        reinterpret_cast<v4u*>(d)[1] = hi;
        if (x == 0 && px0 == 0)   // (of a walk that starts further right, column -1 is no column)
            d[-1] = (uint16_t)(pad == 1 ? lo.x >> 16 : lo.x);
    }
};

// Host-side launchers (defined in dppix_kernels.hip).
// prefix_scan: every frame has the same C and n and the batch has at most
// kPrefixScanTiles tiles (each workgroup of the scan then re-reads the counts
// of all earlier frames instead of waiting for the others).
constexpr int64_t kPrefixScanTiles = 16384;
hipError_t launch_plan(const TileArgs& a, int64_t n_units, int threads, size_t lds, bool prefix_scan,
                       hipStream_t s);
// The scan of the tile counts alone.
hipError_t launch_scan(const TileArgs& a, bool prefix_scan, hipStream_t s);
// Tile counts from the frames' Sobel labels (edge_threshold, images): the units
// of the frames with C channels.  The scan follows.
hipError_t launch_plan_labels(const TileArgs& a, int C, int64_t n_units, int threads, size_t lds, hipStream_t s);
// Tile counts of complex cells from the store's flags alone, then the scan.
hipError_t launch_store_index(const TileArgs& a, bool prefix_scan, hipStream_t s);
hipError_t launch_forward(const TileArgs& a, int layout, int C, int threads, size_t lds, int grid, hipStream_t s);
// paced: RGB frames whose tiles write faster than the memory takes it (k_reconstruct_u8).
hipError_t launch_reconstruct(const TileArgs& a, int layout, int C, bool paced, int threads, size_t lds, int grid,
                              hipStream_t s);
hipError_t launch_backward_reduce(const TileArgs& a, int threads, size_t lds, int grid, hipStream_t s);
hipError_t launch_backward_mirror(const TileArgs& a, int64_t n_units, int threads, hipStream_t s);
hipError_t launch_philox(const uint32_t* in, uint32_t* out, int64_t n, hipStream_t s);
hipError_t launch_noise_advance(uint64_t* noise, int32_t n, uint64_t step, hipStream_t s);
hipError_t launch_edge_mask(const TileArgs& a, int C, int64_t n_units, int threads, size_t lds, hipStream_t s);
// Blocks of seven rows of a metrics unit at most: a lane adds the squared
// errors of one 16-pixel group of each in 32 bits.
constexpr int64_t kMetBlocksMax = 4096;
static_assert(kMetBlocksMax * 16 * 255 * 255 <= (int64_t)UINT32_MAX, "a lane's squared errors fit 32 bits");
hipError_t launch_metrics(const TileArgs& a, int C, bool narrow, int64_t n_units, hipStream_t s);
int metrics_unit_pixels(int C, bool narrow);   // pixels of a row one metrics unit covers
hipError_t launch_metrics_reduce(const TileArgs& a, double* out, hipStream_t s);
hipError_t occupancy_forward(int layout, int C, int threads, size_t lds, int* blocks_per_cu);

}  // namespace dppix
