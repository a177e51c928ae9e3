// dppix_api.hip — host side of the libdppix C ABI: argument validation, plan
// layout (geometry, tiles, workspace, store capacities) and kernel launches.
#include "dppix.h"
#include "dppix_internal.h"
#include "dppix_tiles.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <vector>

using namespace dppix;

namespace {

thread_local std::string g_err;

dppix_status_t fail(dppix_status_t st, const std::string& msg)
{
    g_err = msg;
    return st;
}

dppix_status_t dev_fail(hipError_t e, const char* what)
{
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return DPPIX_EDEVICE;
}

constexpr int kDefaultThreads = 256;
constexpr int64_t kTileBytesTarget = 2048;  // padded bytes per tile row (u8)
constexpr int64_t kPlanCellsMax = 2048;     // cells per band of one plan unit
constexpr int64_t kPlanLdsMax = 32 * 1024;  // LDS of one plan unit
constexpr int64_t kTileLdsTarget = 48 * 1024 + 16;
constexpr int64_t kTileLdsMax = 150 * 1024 + 16;
constexpr int kMaxDim = 1 << 24;

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
size_t grad_scratch_need(dppix_plan_t p);

}  // namespace

// Frames sharing layout, channel count and workgroup size, launched together.
struct LaunchGroup {
    int layout, C;
    int threads;          // workgroup size chosen for the group's tiles
    int rec_threads;      // the same for their reconstruction
    bool paced;           // reconstruction with paced stores: every frame's tiles ask for it
    int64_t lo, hi;       // scheduling-index range
    size_t lds_fwd, lds_rec;
};

struct dppix_plan {
    std::vector<dppix_frame_desc_t> desc;
    std::vector<FrameRec> frames;
    std::vector<int32_t> sched_frame;
    std::vector<int64_t> sched_base;
    int64_t n_tiles = 0;
    int64_t n_units = 0;
    // units of the metrics, the plan from labels and the label masks: those of
    // the frames with C channels are the spans [chan[C - 1], chan[C])
    int32_t met_rows = 0, edge_rows = 0;    // rows of a unit
    std::vector<UnitSpan> met, lab, edge, border;
    int32_t chan[5] = {0, 0, 0, 0, 0};
    bool met_narrow[4] = {false, false, false, false};   // narrow units of the metrics, by channel count
    int lab_threads = 64, edge_threads = 64;
    size_t lab_cells = 0;               // counters of the largest unit of the plan from labels
    bool prefix_scan = false;           // the plan's scan needs no hand-off between workgroups
    int64_t total_cells = 0;
    int64_t total_fine = 0;
    int64_t total_pixels = 0;
    size_t bg_cap = 0, fg_cap = 0;
    WsLayout ws{};
    StateLayout st{};
    size_t lds[6] = {0, 0, 0, 0, 0, 0};
    std::vector<LaunchGroup> groups;
    bool any_f32 = false, any_u8 = false;
    int threads = 0;                    // 0: per launch group (forward, reconstruct), else fixed
    int persistent = 0;
    int cus = 0;                        // compute units of the bound device
    uint8_t* bound = nullptr;
    size_t bound_bytes = 0;
    std::vector<uint8_t> host_tables;   // frame records and scheduling maps, as uploaded
};

struct dppix_graph {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

// Largest multiple of `unit` not above x (at least `unit` when x >= unit).
int64_t round_down(int64_t x, int64_t unit) { return (x / unit) * unit; }

dppix_status_t validate(const dppix_frame_desc_t& d, int32_t f)
{
    char buf[256];
    auto bad = [&](const char* what) {
        std::snprintf(buf, sizeof buf, "frame %d: %s", f, what);
        return fail(DPPIX_EINVAL, buf);
    };
    if (d.height < 1 || d.width < 1)
        return bad("height and width must be >= 1");
    if (d.height > kMaxDim || d.width > kMaxDim)
        return fail(DPPIX_ENOTSUP, "frame dimensions above 2^24");
    if (d.channels < 1 || d.channels > 4)
        return bad("channels must be in 1..4");
    if (d.layout != DPPIX_U8_HWC && d.layout != DPPIX_F32_CHW)
        return bad("unknown layout");
    if (d.layout == DPPIX_U8_HWC && d.pitch < (int64_t)d.width * d.channels)
        return bad("pitch must be >= width*channels bytes");
    if (d.layout == DPPIX_F32_CHW && d.pitch < (int64_t)d.width)
        return bad("pitch must be >= width floats");
    if (d.pad_mode != DPPIX_PAD_SYMMETRIC && d.pad_mode != DPPIX_PAD_REFLECT && d.pad_mode != DPPIX_PAD_NONE)
        return bad("unknown pad_mode");
    if (d.b_fg < 1 || d.b_bg < d.b_fg)
        return bad("need 1 <= b_fg <= b_bg");
    if (d.b_bg % d.b_fg != 0)
        return bad("b_bg must be a multiple of b_fg (b = n * s_b)");
    if (d.b_bg > kMaxB)
        return fail(DPPIX_ENOTSUP, "b_bg above 256");
    if (d.m < 1)
        return bad("m must be >= 1");
    if (!(d.eps_bg > 0.0) || !(d.eps_fg > 0.0))
        return bad("eps_bg and eps_fg must be > 0 (+inf disables noise)");
    if (d.fg_min_count < 0 || (int64_t)d.fg_min_count > (int64_t)d.b_bg * d.b_bg)
        return bad("fg_min_count must be in [0, b_bg^2]");
    if (d.tile_cells < 0)
        return bad("tile_cells must be >= 0");
    const int64_t n = d.b_bg / d.b_fg;
    const int64_t GR = (d.height + d.b_bg - 1) / d.b_bg, GC = (d.width + d.b_bg - 1) / d.b_bg;
    if ((GR * n) * (GC * n) > (int64_t)UINT32_MAX)
        return fail(DPPIX_ENOTSUP, "more than 2^32 subcells in one frame");
    return DPPIX_OK;
}

double sigma_of(int b, int m, double eps)
{
    // Eq. (11): Delta = 255 m / b^2; Eq. (8): sigma = Delta / eps
    const double delta = 255.0 * (double)m / ((double)b * (double)b);
    return delta / eps;
}

// Per-kind LDS bytes of one frame with K cells per tile.
size_t frame_lds(int kind, const FrameRec& F) { return lds_plan(kind, F.K, F.b, F.n, F.C).bytes; }

int kind_fwd(const FrameRec& F) { return F.layout == DPPIX_F32_CHW ? kFwdF32 : kFwdU8; }
int kind_rec(const FrameRec& F) { return F.layout == DPPIX_F32_CHW ? kRecF32 : kRecU8; }

// Tile width: about kTileBytesTarget padded bytes per row, tiles of one band
// balanced, u8 tiles starting on 16-byte boundaries when possible, LDS bounded.
void choose_tiles(FrameRec& F, int32_t requested)
{
    const int64_t unit_bytes = (F.layout == DPPIX_F32_CHW) ? 4 * (int64_t)F.b : (int64_t)F.b * F.C;
    int64_t align = 16 / std::gcd<int64_t>(16, unit_bytes);  // cells per 16-byte-aligned step
    int64_t K;
    if (requested > 0) {
        K = std::min<int64_t>(requested, F.GC);
    } else {
        // the band's padded row cut into the fewest tiles of at most about
        // kTileBytesTarget bytes (a batch of 768-pixel frames alone runs 7 %
        // faster with one 2304-byte tile per band, the mixed-resolution batch
        // 3.8 % slower; the autotuner can pick the former for such batches)
        int64_t kmax = std::max<int64_t>(1, kTileBytesTarget / unit_bytes);
        if (kmax >= align)
            kmax = round_down(kmax, align);
        const int64_t band = (int64_t)F.GC * unit_bytes;
        const int64_t tx = std::max<int64_t>(1, (band + kTileBytesTarget - 1) / kTileBytesTarget);
        K = (F.GC + tx - 1) / tx;
        if (K % align != 0 && ((K + align - 1) / align) * align <= std::max(kmax, K))
            K = ((K + align - 1) / align) * align;
        K = std::min<int64_t>(K, F.GC);
    }
    F.K = (int32_t)std::max<int64_t>(1, K);
    // keep every tile kind of this frame within the LDS target
    while (F.K > 1) {
        size_t need = std::max(frame_lds(kind_fwd(F), F), frame_lds(kind_rec(F), F));
        if (F.layout == DPPIX_F32_CHW)
            need = std::max(need, frame_lds(kBwd, F));
        if ((int64_t)need <= kTileLdsTarget)
            break;
        F.K = std::max(1, F.K / 2);
    }
    F.TX = (F.GC + F.K - 1) / F.K;
    // Plan units: whole tiles of a band (at most kPlanCellsMax cells), and as
    // many bands as keep about one 16-row strip item per lane of a 256-lane
    // workgroup (several bands' worth of rows per lane when b < 16).
    F.ctx = (int32_t)std::max<int64_t>(1, std::min<int64_t>(F.TX, kPlanCellsMax / F.K));
    const int64_t kc = std::min<int64_t>((int64_t)F.ctx * F.K, F.GC);
    const int64_t nstr = (kc * F.b + 15) / 16;
    const int64_t rows = std::min<int64_t>(F.b, 16);
    const int64_t items = nstr * ((F.b + rows - 1) / rows);
    int64_t cnb = (int64_t)kDefaultThreads * std::max<int64_t>(1, 16 / F.b) / items;
    cnb = std::max<int64_t>(1, std::min<int64_t>(cnb, F.GR));
    while (cnb > 1 && plan_lds((int)cnb, F.ctx, F.K) > kPlanLdsMax)
        --cnb;
    F.cnb = (int32_t)cnb;
    F.cunits = (int32_t)(((F.GR + cnb - 1) / cnb) * ((F.TX + F.ctx - 1) / F.ctx));
}

// XCD-aware tile order within one launch's scheduling range [lo, hi): the
// dispatcher hands workgroup i of a launch to XCD i mod kXcds, and each XCD
// has its own L2.  Neighbouring tiles of a band share the cache lines their
// rows are cut at (rows whose pitch or tile width is not a whole number of
// lines), so the map gives every XCD runs of kXcdRun consecutive tiles:
// within each chunk of kXcds * kXcdRun workgroups, workgroup i takes tile
// (i mod kXcds) * kXcdRun + i / kXcds of the chunk.  A shared line is then
// fetched once, by one L2, while both tiles are in flight.  The last partial
// chunk keeps the linear order.
constexpr int64_t kXcds = 8;
constexpr int64_t kXcdRun = 8;

void xcd_runs(int32_t* map, int64_t lo, int64_t hi)
{
    const int64_t n = hi - lo, chunk = kXcds * kXcdRun;
    const int64_t full = (n / chunk) * chunk;
    std::vector<int32_t> tmp(2 * (size_t)full);
    for (int64_t i = 0; i < full; ++i) {
        const int64_t c = i / chunk, w = i - c * chunk;
        const int64_t t = c * chunk + (w % kXcds) * kXcdRun + w / kXcds;
        tmp[2 * i] = map[2 * (lo + t)];
        tmp[2 * i + 1] = map[2 * (lo + t) + 1];
    }
    std::copy(tmp.begin(), tmp.end(), map + 2 * lo);
}

// Workgroup size of a frame's forward tiles.  A tile with few phase-1 items
// (strips x groups of subgrid rows, fp32: x channels; e.g. b = 16 or narrow
// frames) keeps more tiles in flight per CU with 128 lanes; larger tiles fill 256
// (measured on 64 x 1080p and 300 x 768x576 batches; fp32 forward of 64 x 3 x 218 x
// 178, b 8: 256 / 128 lanes 21.7 / 18.2 us, of 32 x 3 x 512 x 512, b 16: 35 / 38).  A u8
// batch of fewer tiles than there are CUs (`few`) is bound by each tile's own
// chain, which more lanes shorten: one 1080p frame 256 / 512 lanes 13.2 / 12.6 us,
// one 768 x 576 frame 128 / 256 / 512 lanes 13.2 / 12.2 / 11.8.
constexpr int64_t kFewTiles = 256;

int tile_threads(const FrameRec& F, int64_t tiles)
{
    const int64_t bytes = (int64_t)F.K * F.b * F.C;
    if (F.layout != DPPIX_U8_HWC)
        return F.C * std::min(F.n, kRowGroupF) * ((bytes / F.C + 3) / 4) <= 320 ? 128 : kDefaultThreads;
    const int q = F.s == 2 ? 4 : ((F.s == 3 || F.s == 4) ? 2 : 1);
    const int64_t items = (bytes + 15) / 16 * ((std::min(F.n, kRowGroup) + q - 1) / q);
    if (tiles < kFewTiles)
        return items > 256 ? 512 : (items > 128 ? kDefaultThreads : 128);
    return items <= 320 ? 128 : kDefaultThreads;
}

// Workgroup size of a frame's reconstruction tiles.  They only write, and where a
// tile has enough 16-byte stores more lanes cover the latency of its statistics:
// 64 x 1080p, b 32 (3840 stores a tile): 256 / 512 lanes 78.6 / 74.1 us; 4 frames of
// 4000 x 6000, b 16 (2000): 128 / 256 lanes 81 / 72; 100 x 576 x 768, b 16 (1152): 30.6 /
// 35.7.  With few tiles per CU, 512 lanes leave them uneven: 8 x 1080p, 816 tiles:
// 13.9 / 16.0.  fp32 tiles take 256 (64 x 3 x 218 x 178: 128 / 256 lanes 11.9 / 10.8).
int rec_threads(const FrameRec& F, int64_t tiles)
{
    const int base = tile_threads(F, tiles);
    if (F.layout != DPPIX_U8_HWC)
        return kDefaultThreads;
    const int64_t stores = ((int64_t)F.K * F.b * F.C + 15) / 16 * F.b;
    if (tiles < kFewTiles || stores < 1536)
        return base;
    return tiles >= 2048 && stores >= 3072 ? 512 : kDefaultThreads;
}

// Whether a frame's reconstruction tiles pace their stores (the sides of the
// line: k_reconstruct_u8's PACED).
bool rec_paced(const FrameRec& F)
{
    return F.layout == DPPIX_U8_HWC && F.C == 3 && F.n == 2 && (F.s == 5 || F.s == 6);
}

// Plan units of the batch.  Fewer than two a compute unit (kPlanUnits) leave
// some idle, so units of several bands are halved, down to kPlanItems strip
// items (a wave and a bit): 64 frames of 218 x 178, b 8: 64 units of 336 items
// 13.5 us, 256 of 84: 10.3, 1792 of 12: 14; 24 photos of odd sizes, b 16: 393 of up
// to 256 15.2, 729 of up to 160 14.1; 16 x 512 x 512 fp32, b 4: 10.8 whole, 7.9
// halved.  Up to kPlanUnitsFull more halving only pays while a unit still
// fills its 256 lanes: 16 x 1080p, b 4: 544 units of 960 items 17.2 us, 1088 of
// 480: 15.4; but 32 x 720 x 1280, b 12: 640 of 243 12.6, 1920 of 81 16.8; 100 x 480
// x 640, b 12: 700 of 246 12.7, 1400 of 123 15.4.
constexpr int64_t kPlanUnits = 512, kPlanUnitsFull = 1024;
constexpr int64_t kPlanItems = 72, kPlanItemsFull = 256;

void spread_units(dppix_plan& p)
{
    auto items = [](const FrameRec& F, int64_t bands) {
        const int64_t rows = std::min(F.b, 16);
        return bands * ((std::min<int64_t>((int64_t)F.ctx * F.K, F.GC) * F.b + 15) / 16) * ((F.b + rows - 1) / rows);
    };
    for (bool more = true; more;) {
        more = false;
        p.n_units = 0;
        for (const FrameRec& F : p.frames)
            p.n_units += F.cunits;
        if (p.n_units >= kPlanUnitsFull)
            break;
        const int64_t least = p.n_units < kPlanUnits ? kPlanItems : kPlanItemsFull;
        for (FrameRec& F : p.frames)
            if (F.cnb > 1 && items(F, (F.cnb + 1) / 2) >= least) {
                F.cnb = (F.cnb + 1) / 2;
                F.cunits = ((F.GR + F.cnb - 1) / F.cnb) * ((F.TX + F.ctx - 1) / F.ctx);
                more = true;
            }
    }
    for (const FrameRec& F : p.frames)
        p.lds[kPlan] = std::max<size_t>(p.lds[kPlan], plan_lds(F.cnb, F.ctx, F.K));
}

// Spans of the units of frames in the order given; units(F): a frame's.
template <typename Units>
std::vector<UnitSpan> span_units(const dppix_plan& p, const std::vector<int32_t>& order, Units units)
{
    std::vector<UnitSpan> out(order.size() + 1);
    int64_t at = 0;
    for (size_t k = 0; k < order.size(); ++k) {
        out[k] = UnitSpan{at, order[k], 0};
        at += units(p.frames[order[k]]);
    }
    out.back() = UnitSpan{at, 0, 0};
    return out;
}

int64_t span_total(const std::vector<UnitSpan>& spans) { return spans.empty() ? 0 : spans.back().first; }

// Units of each of the n frames from span lo on, if they have as many, else 0.
int32_t equal_units(const std::vector<UnitSpan>& spans, int32_t lo, int32_t n)
{
    const int64_t u = spans[lo + 1].first - spans[lo].first;
    for (int32_t k = lo; k < lo + n; ++k)
        if (spans[k + 1].first - spans[k].first != u)
            return 0;
    return (int32_t)u;
}

// Rows of a unit, step * m - over for the largest m up to `most` that gives
// the batch `wanted` units; units(F, rows) counts a frame's.  Huge batches:
// no more units than twice the tiles (a launch has at most 2^31).
template <typename Units>
int32_t unit_rows(const dppix_plan& p, Units units, int32_t step, int32_t over, int32_t most, int64_t wanted)
{
    auto total = [&](int32_t m) {
        int64_t t = 0;
        for (const FrameRec& F : p.frames)
            t += units(F, step * m - over);
        return t;
    };
    int32_t m = most;
    while (m > 2 && total(m) < wanted)
        --m;
    while (2 * m <= kMetBlocksMax && total(m) > 2 * p.n_tiles + (1 << 20))
        m *= 2;
    return step * m - over;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Units of the utility metrics: columns of metrics_unit_pixels pixels x
// segments of rows.  A unit reads six rows more than it has, and works in
// blocks of seven, so a segment is 7 m - 6 rows; wanted: four rounds of the
// 768 workgroups the GPU holds at once (16 x 1080p: m = 3 / 6 / 10: 196 / 170 /
// 164 us; one 6000 x 4000 frame: m = 3 / 6 / 8 / 10: 155 / 131 / 125 / 129 us).
// At most kMetBlocksMax blocks (a lane's squared errors).
constexpr int64_t kMetUnits = 3000;

int64_t metrics_units(const FrameRec& F, bool narrow, int32_t rows)
{
    return ceil_div(F.W, metrics_unit_pixels(F.C, narrow)) * ceil_div(F.H, rows);
}

// Whether the frames of C channels take narrow units: their windows fill less
// than 77 % of the wide units' lanes (narrow / wide units: RGB, 76 %, 64 and 256
// frames of 128 x 128: 15.6 / 15.2 and 38 / 45 us; 78 %, 32 of 256 x 256: 26 / 25;
// 54 %, 256 of 218 x 178: 92 / 108; 96 %, 128 of 160 x 160: 36 / 30).
bool metrics_narrow(const dppix_plan& p, int C)
{
    int64_t windows = 0, lanes = 0;
    const int64_t unit = metrics_unit_pixels(C, false);
    for (const FrameRec& F : p.frames)
        if (F.C == C) {
            windows += (int64_t)F.H * std::max(F.W - 6, 0);
            lanes += (int64_t)F.H * ceil_div(F.W, unit) * unit;
        }
    return (double)windows < 0.77 * (double)lanes;
}

// Units of the label masks: equal chunks of columns x segments of rows.  A
// unit stages two rows more than it labels, in blocks of four: 4 m - 2 rows, m
// at most 4 (64 x 1080p: m = 3 / 4 / 8 / 16: 92 / 95 / 101 / 114 us; 16 x 1080p: m
// = 2 / 3 / 4 / 8: 29 / 25 / 25 / 25 us).  Wanted: a workgroup of up to four
// waves for each SIMD, and two of the single waves that frames of up to 227
// columns take (256 RGB frames of 64 x 64: m = 1 / 2 / 3 / 4: 9.7 / 7.3 / 7.4 / 8.6 us;
// 512 of 32 x 32: 9.6 / 7.3 / 7.5 / 8.6; 64 of 218 x 178: 9.2 / 8.1 / 8.8 / 8.7).
constexpr int64_t kEdgeUnits = 1024;

// LDS of a walk's two blocks of staged rows.
size_t label_lds(int threads) { return 4 * (size_t)kLabBlock * (size_t)label_stride(4 * threads); }

int64_t edge_units(const FrameRec& F, int32_t rows) { return ceil_div(F.W, kLabCols) * ceil_div(F.H, rows); }

// Bands of a unit of the plan from labels (one tile's columns): about kLabRows
// rows, so that the two rows a unit stages beyond its own are few, and at
// most 2048 cell counters (16 x 1080p b 32: 32 / 64 rows: 34 / 36 us; 24 photos b
// 16: 16 / 32 / 64 rows: 32 / 31 / 38 us; 64 x 1080p: no difference).
constexpr int32_t kLabRows = 32;

int32_t label_bands(const FrameRec& F)
{
    const int32_t nb = std::max(1, std::min(kLabRows / F.b, 2048 / F.K));
    return std::min(nb, F.GR);
}

}  // namespace

extern "C" {

const char* dp_pix_version(void) { return "dppix 0.1 (gfx950)"; }

const char* dp_pix_status_string(dppix_status_t s)
{
    switch (s) {
    case DPPIX_OK: return "ok";
    case DPPIX_EINVAL: return "invalid argument";
    case DPPIX_ENOMEM: return "out of memory";
    case DPPIX_EDEVICE: return "device error";
    case DPPIX_ENOTSUP: return "not supported";
    }
    return "unknown status";
}

const char* dp_pix_last_error(void) { return g_err.c_str(); }

dppix_status_t dp_pix_plan_create(const dppix_frame_desc_t* descs, int32_t n_frames, dppix_plan_t* out)
{
    if (out == nullptr)
        return fail(DPPIX_EINVAL, "out is NULL");
    *out = nullptr;
    if (descs == nullptr || n_frames < 1)
        return fail(DPPIX_EINVAL, "need at least one frame descriptor");
    for (int32_t f = 0; f < n_frames; ++f) {
        dppix_status_t st = validate(descs[f], f);
        if (st != DPPIX_OK)
            return st;
    }
    dppix_plan* p = new (std::nothrow) dppix_plan;
    if (p == nullptr)
        return fail(DPPIX_ENOMEM, "host allocation failed");
    p->desc.assign(descs, descs + n_frames);
    p->frames.resize(n_frames);
    int64_t cell = 0, fine = 0, tile = 0;
    for (int32_t f = 0; f < n_frames; ++f) {
        const dppix_frame_desc_t& d = descs[f];
        FrameRec& F = p->frames[f];
        std::memset(&F, 0, sizeof F);
        F.H = d.height;
        F.W = d.width;
        F.C = d.channels;
        F.layout = d.layout;
        F.pitch = d.pitch;
        F.b = d.b_bg;
        F.s = d.b_fg;
        F.n = d.b_bg / d.b_fg;
        F.pad = d.pad_mode;
        F.GR = (d.height + d.b_bg - 1) / d.b_bg;   // G_R = ceil(M / b)
        F.GC = (d.width + d.b_bg - 1) / d.b_bg;    // G_C = ceil(N / b)
        // tau = 0 in the unpadded mode: majority of each cell's real pixels
        F.tau = d.fg_min_count > 0 ? d.fg_min_count
                                   : (d.pad_mode == DPPIX_PAD_NONE ? 0 : (d.b_bg * d.b_bg + 1) / 2);
        F.noise_bg = std::isinf(d.eps_bg) ? 0 : 1;
        F.noise_fg = std::isinf(d.eps_fg) ? 0 : 1;
        F.sigma_bg = F.noise_bg ? sigma_of(F.b, d.m, d.eps_bg) : 0.0;
        F.sigma_fg = F.noise_fg ? sigma_of(F.s, d.m, d.eps_fg) : 0.0;
        F.key0 = (uint32_t)(d.seed & 0xFFFFFFFFu);
        F.key1 = (uint32_t)(d.seed >> 32);
        F.fi0 = (uint32_t)(d.frame_index & 0xFFFFFFFFu);
        F.fi1 = (uint32_t)(d.frame_index >> 32);
        F.off32 = ((int64_t)d.b_bg + 1) * d.pitch * (d.layout == DPPIX_F32_CHW ? 4 : 1) < ((int64_t)1 << 31);
        choose_tiles(F, d.tile_cells);
        {
            size_t need = std::max(frame_lds(kind_fwd(F), F), frame_lds(kind_rec(F), F));
            if ((int64_t)need > kTileLdsMax) {
                delete p;
                return fail(DPPIX_ENOTSUP, "n*n*channels too large for one tile in LDS");
            }
        }
        F.lnb = label_bands(F);
        p->lab_cells = std::max<size_t>(p->lab_cells, (size_t)F.lnb * (size_t)(F.K + 1));
        p->lab_threads = std::max(p->lab_threads, label_threads((int)std::min<int64_t>((int64_t)F.K * F.b, kLabCols)));
        p->edge_threads = std::max(p->edge_threads, label_threads(std::min(label_chunk(F.W), F.W)));
        F.cell_base = cell;
        F.fine_base = fine;
        F.tile_base = tile;
        cell += (int64_t)F.GR * F.GC;
        fine += (int64_t)F.GR * F.n * F.GC * F.n;
        tile += (int64_t)F.GR * F.TX;
        p->bg_cap += (size_t)F.GR * F.GC * F.C;
        p->fg_cap += (size_t)F.GR * F.GC * F.n * F.n * F.C;
        p->total_pixels += (int64_t)F.H * F.W;
        if (F.layout == DPPIX_F32_CHW)
            p->any_f32 = true;
        else
            p->any_u8 = true;
        for (int k = 1; k < 6; ++k) {
            if (k == kBwd && F.layout != DPPIX_F32_CHW)
                continue;
            if ((k == kFwdU8 || k == kRecU8) && F.layout != DPPIX_U8_HWC)
                continue;
            if ((k == kFwdF32 || k == kRecF32) && F.layout != DPPIX_F32_CHW)
                continue;
            p->lds[k] = std::max(p->lds[k], frame_lds(k, F));
        }
    }
    spread_units(*p);
    p->total_cells = cell;
    p->total_fine = fine;
    p->n_tiles = tile;
    if (tile > (int64_t)INT32_MAX || p->n_units > (int64_t)INT32_MAX) {
        delete p;
        return fail(DPPIX_ENOTSUP, "more than 2^31 tiles");
    }
    p->prefix_scan = tile <= kPrefixScanTiles;
    for (const FrameRec& F : p->frames)
        p->prefix_scan = p->prefix_scan && F.C == p->frames[0].C && F.n == p->frames[0].n && F.K < 65536;
    // Scheduling order: frames with the heaviest tiles first (longest tiles
    // start early, the tail is made of light ones); ties keep batch order.
    std::vector<int32_t> order(n_frames);
    std::iota(order.begin(), order.end(), 0);
    auto tile_cost = [&](int32_t f) {
        const FrameRec& F = p->frames[f];
        const int64_t bpp = F.layout == DPPIX_F32_CHW ? 4 : 1;
        return (int64_t)F.b * F.K * F.b * F.C * bpp;
    };
    // group-major (one kernel instantiation per layout and channel count, one
    // launch per workgroup size)
    auto group_key = [&](int32_t f) {
        const FrameRec& F = p->frames[f];
        return (F.layout * 8 + F.C) * 4 + (512 / tile_threads(F, tile)) / 2;
    };
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        if (group_key(x) != group_key(y))
            return group_key(x) < group_key(y);
        return tile_cost(x) > tile_cost(y);
    });
    p->sched_frame = order;
    p->sched_base.resize(n_frames + 1);
    int64_t acc = 0;
    for (int32_t k = 0; k < n_frames; ++k) {
        p->sched_base[k] = acc;
        const FrameRec& F = p->frames[order[k]];
        acc += (int64_t)F.GR * F.TX;
    }
    p->sched_base[n_frames] = acc;
    for (int32_t k = 0; k < n_frames; ++k) {
        const FrameRec& F = p->frames[order[k]];
        const int th = tile_threads(F, tile);
        if (p->groups.empty() || p->groups.back().layout != F.layout || p->groups.back().C != F.C ||
            p->groups.back().threads != th)
            p->groups.push_back(LaunchGroup{F.layout, F.C, th, 0, true, p->sched_base[k], p->sched_base[k], 0, 0});
        LaunchGroup& g = p->groups.back();
        g.hi = p->sched_base[k + 1];
        g.rec_threads = std::max(g.rec_threads, rec_threads(F, tile));
        g.paced = g.paced && rec_paced(F);
        g.lds_fwd = std::max(g.lds_fwd, frame_lds(kind_fwd(F), F));
        g.lds_rec = std::max(g.lds_rec, frame_lds(kind_rec(F), F));
    }

    if (p->groups.size() > (size_t)kMaxGroups) {   // 2 layouts x 4 channel counts x 3 sizes at most
        delete p;
        return fail(DPPIX_ENOTSUP, "too many launch groups");
    }

    // Workspace layout.
    WsLayout& w = p->ws;
    size_t o = 0;
    w.frames = o;      o = align256(o + sizeof(FrameRec) * n_frames);
    w.tile_map = o;    o = align256(o + sizeof(int32_t) * 2 * (size_t)p->n_tiles);
    w.unit_map = o;    o = align256(o + sizeof(int32_t) * 2 * (size_t)p->n_units);
    w.simple_counts = o; o = align256(o + sizeof(uint64_t) * 4 * (size_t)n_frames);
    // Units of the kernels with units of their own, by frame: the metrics and
    // the labels take bytes, frames of one channel count after another (a
    // launch each), the adjoint floats.
    std::vector<int32_t> by_chan;
    if (p->any_f32) {
        for (int32_t f = 0; f < n_frames; ++f)
            if (p->frames[f].pad != DPPIX_PAD_NONE && !p->any_u8)
                by_chan.push_back(f);
        p->border = span_units(*p, by_chan, [](const FrameRec& F) {
            const BorderArea m = border_area(F);
            return (int64_t)F.C * (border_parts(m.nA) + border_parts(m.nB));
        });
    } else {
        for (int C = 1; C <= 4; ++C) {
            for (int32_t f = 0; f < n_frames; ++f)
                if (p->frames[f].C == C)
                    by_chan.push_back(f);
            p->chan[C] = (int32_t)by_chan.size();
        }
        for (int C = 1; C <= 4; ++C)
            p->met_narrow[C - 1] = metrics_narrow(*p, C);
        auto met_units = [&](const FrameRec& F, int32_t rows) { return metrics_units(F, p->met_narrow[F.C - 1], rows); };
        p->met_rows = unit_rows(*p, met_units, 7, 6, 10, kMetUnits);
        p->edge_rows = unit_rows(*p, edge_units, 4, 2, 4, p->edge_threads == 64 ? 2 * kEdgeUnits : kEdgeUnits);
        p->met = span_units(*p, by_chan, [&](const FrameRec& F) { return met_units(F, p->met_rows); });
        p->edge = span_units(*p, by_chan, [&](const FrameRec& F) { return edge_units(F, p->edge_rows); });
        p->lab = span_units(*p, by_chan, [](const FrameRec& F) { return F.TX * ceil_div(F.GR, F.lnb); });
    }
    auto place = [&](size_t& at, const std::vector<UnitSpan>& spans) {
        at = o;
        o = align256(o + sizeof(UnitSpan) * spans.size());
    };
    place(w.border_spans, p->border);
    place(w.lab_spans, p->lab);
    place(w.edge_spans, p->edge);
    place(w.met_spans, p->met);
    w.total = o;
    // Per-call state carried by each store.
    StateLayout& sl = p->st;
    o = 0;
    sl.tile_cnt = o;   o = align256(o + sizeof(uint32_t) * (size_t)p->n_tiles);
    sl.tile_fg = o;    o = align256(o + sizeof(uint32_t) * (size_t)p->n_tiles);
    sl.counters = o;   o = align256(o + sizeof(uint32_t) * kTicketWords);
    sl.total = o;

    // Host image of the tables: frame records, and per scheduling index the
    // frame and the tile within it.
    p->host_tables.assign(w.total, 0);
    std::memcpy(p->host_tables.data() + w.frames, p->frames.data(), sizeof(FrameRec) * n_frames);
    int32_t* map = reinterpret_cast<int32_t*>(p->host_tables.data() + w.tile_map);
    for (int32_t k = 0; k < n_frames; ++k)
        for (int64_t i = p->sched_base[k]; i < p->sched_base[k + 1]; ++i) {
            map[2 * i] = order[k];
            map[2 * i + 1] = (int32_t)(i - p->sched_base[k]);
        }
    for (const LaunchGroup& g : p->groups)
        xcd_runs(map, g.lo, g.hi);
    {
        // without masks every cell is simple: n_bg = cells, n_fg = 0, and the
        // frames' statistics packed back to back in batch order
        uint64_t* sc = reinterpret_cast<uint64_t*>(p->host_tables.data() + w.simple_counts);
        uint64_t bg_off = 0;
        for (int32_t f = 0; f < n_frames; ++f) {
            const FrameRec& F = p->frames[f];
            const uint64_t cells = (uint64_t)F.GR * (uint64_t)F.GC;
            sc[4 * f + 0] = cells;
            sc[4 * f + 1] = 0;
            sc[4 * f + 2] = bg_off;
            sc[4 * f + 3] = 0;
            bg_off += cells * (uint64_t)F.C;
        }
    }
    auto put = [&](size_t at, const std::vector<UnitSpan>& spans) {
        std::copy(spans.begin(), spans.end(), reinterpret_cast<UnitSpan*>(p->host_tables.data() + at));
    };
    put(w.border_spans, p->border);
    put(w.lab_spans, p->lab);
    put(w.edge_spans, p->edge);
    put(w.met_spans, p->met);
    int32_t* umap = reinterpret_cast<int32_t*>(p->host_tables.data() + w.unit_map);
    for (int32_t f = 0, u = 0; f < n_frames; ++f)
        for (int32_t i = 0; i < p->frames[f].cunits; ++i, ++u) {
            umap[2 * u] = f;
            umap[2 * u + 1] = i;
        }
    *out = p;
    return DPPIX_OK;
}

void dp_pix_plan_destroy(dppix_plan_t p) { delete p; }

dppix_status_t dp_pix_plan_sizes(dppix_plan_t p, dppix_sizes_t* out)
{
    if (p == nullptr || out == nullptr)
        return fail(DPPIX_EINVAL, "NULL plan or output");
    out->workspace_bytes = p->ws.total;
    out->store_state_bytes = p->st.total;
    out->bg_capacity = p->bg_cap;
    out->fg_capacity = p->fg_cap;
    out->flag_bytes = (size_t)p->total_cells;
    out->clip_bytes_bg = p->bg_cap;
    out->clip_bytes_fg = p->fg_cap;
    out->grad_scratch_bytes = grad_scratch_need(p);
    out->metrics_scratch_bytes = align256(16 * (size_t)std::max<int64_t>(1, span_total(p->met)));
    out->n_tiles = p->n_tiles;
    out->total_pixels = p->total_pixels;
    out->forward_launches = (int64_t)p->groups.size();
    return DPPIX_OK;
}

dppix_status_t dp_pix_plan_frame_info(dppix_plan_t p, int32_t f, dppix_frame_info_t* out)
{
    if (p == nullptr || out == nullptr)
        return fail(DPPIX_EINVAL, "NULL plan or output");
    if (f < 0 || f >= (int32_t)p->frames.size())
        return fail(DPPIX_EINVAL, "frame index out of range");
    const FrameRec& F = p->frames[f];
    out->grid_rows = F.GR;
    out->grid_cols = F.GC;
    out->n = F.n;
    out->pad_rows = F.GR * F.b - F.H;
    out->pad_cols = F.GC * F.b - F.W;
    out->tile_cells = F.K;
    out->tiles_per_band = F.TX;
    out->fg_min_count = F.tau;
    out->cell_offset = F.cell_base;
    out->fine_offset = F.fine_base;
    out->sigma_bg = F.sigma_bg;
    out->sigma_fg = F.sigma_fg;
    return DPPIX_OK;
}

dppix_status_t dp_pix_plan_set_launch(dppix_plan_t p, int32_t threads, int32_t persistent)
{
    if (p == nullptr)
        return fail(DPPIX_EINVAL, "NULL plan");
    if (threads != 0 && (threads < 64 || threads > kMaxThreads || threads % 64 != 0))
        return fail(DPPIX_EINVAL, "threads must be 0 (chosen per frame class) or a multiple of 64 in 64..512");
    if (persistent < 0 || persistent > 64)
        return fail(DPPIX_EINVAL, "persistent must be 0 (one workgroup per tile), 1 (resident grid) or 2..64 "
                                  "(workgroups per CU)");
    p->threads = threads;
    p->persistent = persistent;
    return DPPIX_OK;
}

dppix_status_t dp_pix_plan_bind(dppix_plan_t p, void* ws, size_t bytes, dppix_stream_t stream)
{
    if (p == nullptr || ws == nullptr)
        return fail(DPPIX_EINVAL, "NULL plan or workspace");
    if (p->bound != nullptr)
        return fail(DPPIX_EINVAL, "plan is already bound (its tables are immutable once uploaded)");
    if (bytes < p->ws.total)
        return fail(DPPIX_ENOMEM, "workspace smaller than workspace_bytes");
    if ((reinterpret_cast<uintptr_t>(ws) & 255) != 0)
        return fail(DPPIX_EINVAL, "workspace must be 256-byte aligned");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(ws, p->host_tables.data(), p->host_tables.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess)
        return dev_fail(e, "uploading plan tables");
    // the tables are on the device when bind returns, so calls on any stream
    // may use the plan from then on
    e = hipStreamSynchronize(s);
    if (e != hipSuccess)
        return dev_fail(e, "uploading plan tables");
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
        p->cus = n;
    else
        p->cus = 256;
    p->bound = static_cast<uint8_t*>(ws);
    p->bound_bytes = bytes;
    return DPPIX_OK;
}

dppix_status_t dp_pix_plan_workspace_size(const dppix_frame_desc_t* descs, int32_t n_frames, dppix_sizes_t* out)
{
    if (out == nullptr)
        return fail(DPPIX_EINVAL, "out is NULL");
    dppix_plan_t p = nullptr;
    dppix_status_t st = dp_pix_plan_create(descs, n_frames, &p);
    if (st != DPPIX_OK)
        return st;
    st = dp_pix_plan_sizes(p, out);
    dp_pix_plan_destroy(p);
    return st;
}

}  // extern "C"

namespace {

// Kernel arguments of one call: the plan's tables, and the per-call state
// (flags, counts, tile counts and prefixes, tickets) of the call's store.
TileArgs base_args(dppix_plan_t p, const dppix_store_t* store)
{
    TileArgs a;
    std::memset(&a, 0, sizeof a);
    uint8_t* w = p->bound;
    a.frames = reinterpret_cast<const FrameRec*>(w + p->ws.frames);
    a.tile_map = reinterpret_cast<const int32_t*>(w + p->ws.tile_map);
    a.n_frames = (int32_t)p->frames.size();
    a.n_tiles = p->n_tiles;
    a.unit_map = reinterpret_cast<const int32_t*>(w + p->ws.unit_map);
    a.simple_counts = reinterpret_cast<const uint64_t*>(w + p->ws.simple_counts);
    a.total_cells = p->total_cells;
    a.persistent = p->persistent;
    if (store != nullptr) {
        uint8_t* st = static_cast<uint8_t*>(store->state);
        a.flags = store->flags;
        a.counts = store->counts;
        a.bg = store->bg;
        a.fg = store->fg;
        a.tile_cnt = reinterpret_cast<uint32_t*>(st + p->st.tile_cnt);
        a.tile_fg = reinterpret_cast<uint32_t*>(st + p->st.tile_fg);
        a.ticket = reinterpret_cast<uint32_t*>(st + p->st.counters);
        a.noise = store->noise;
    }
    return a;
}

dppix_status_t need_bound(dppix_plan_t p)
{
    if (p == nullptr)
        return fail(DPPIX_EINVAL, "NULL plan");
    if (p->bound == nullptr)
        return fail(DPPIX_EINVAL, "plan has no workspace (call dp_pix_plan_bind)");
    return DPPIX_OK;
}

// Every call that takes a store needs its layout (flags, counts) and its
// per-call state; need_stats: also the statistics arrays.
dppix_status_t check_store(const dppix_store_t* s, bool need_stats)
{
    if (s == nullptr)
        return fail(DPPIX_EINVAL, "NULL store");
    if (s->flags == nullptr || s->counts == nullptr || s->state == nullptr)
        return fail(DPPIX_EINVAL, "store flags, counts and state are required");
    if ((reinterpret_cast<uintptr_t>(s->state) & 255) != 0)
        return fail(DPPIX_EINVAL, "store state must be 256-byte aligned");
    if ((reinterpret_cast<uintptr_t>(s->counts) & 7) != 0)
        return fail(DPPIX_EINVAL, "store counts must be 8-byte aligned");
    if ((reinterpret_cast<uintptr_t>(s->noise) & 7) != 0)
        return fail(DPPIX_EINVAL, "store noise counters must be 8-byte aligned");
    if (need_stats && (s->bg == nullptr || s->fg == nullptr))
        return fail(DPPIX_EINVAL, "store bg/fg are NULL");
    return DPPIX_OK;
}

// Workgroup size of the kernels outside the launch groups.
int plain_threads(dppix_plan_t p) { return p->threads ? p->threads : kDefaultThreads; }

// Workgroup size of a launch group's forward (or reconstruction) tiles.
int group_threads(dppix_plan_t p, const LaunchGroup& g, bool rec)
{
    return p->threads ? p->threads : (rec ? g.rec_threads : g.threads);
}

int grid_for(dppix_plan_t p, int layout, int C, int threads, int64_t tiles, size_t lds)
{
    if (!p->persistent)
        return (int)tiles;
    const int cus = p->cus > 0 ? p->cus : 256;
    int per_cu = p->persistent;
    if (per_cu == 1 && (occupancy_forward(layout, C, threads, lds, &per_cu) != hipSuccess || per_cu < 1))
        per_cu = 1;
    const int64_t g = std::min<int64_t>((int64_t)cus * per_cu, tiles);
    return (int)std::max<int64_t>(1, g);
}

// One launch per channel count that the batch has, over the units of its frames.
template <typename Launch>
hipError_t for_channels(dppix_plan_t p, const TileArgs& base, const std::vector<UnitSpan>& spans, size_t at, Launch launch)
{
    for (int C = 1; C <= 4; ++C) {
        const int32_t lo = p->chan[C - 1], n = p->chan[C] - lo;
        if (n == 0)
            continue;
        TileArgs a = base;
        a.spans = reinterpret_cast<const UnitSpan*>(p->bound + at) + lo;
        a.n_spans = n;
        a.span_units = equal_units(spans, lo, n);
        a.sched_offset = spans[lo].first;
        const hipError_t e = launch(a, C, spans[lo + n].first - spans[lo].first);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// One launch per group: its scheduling range and its own ticket pair.
template <typename Launch>
hipError_t for_groups(dppix_plan_t p, const TileArgs& base, bool rec, Launch launch)
{
    for (size_t gi = 0; gi < p->groups.size(); ++gi) {
        const LaunchGroup& g = p->groups[gi];
        TileArgs a = base;
        a.sched_offset = g.lo;
        a.n_tiles = g.hi - g.lo;
        a.ticket = base.ticket + 2 * gi;
        const size_t lds = rec ? g.lds_rec : g.lds_fwd;
        hipError_t e = launch(a, g, lds, grid_for(p, g.layout, g.C, group_threads(p, g, rec), a.n_tiles, lds));
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// Scratch of dp_pix_backward: gradient of every statistic (bg, fg in store
// order) and the class-local index of every grid cell.
size_t grad_scratch_need(dppix_plan_t p)
{
    return align256(4 * p->bg_cap) + align256(4 * p->fg_cap) + align256(4 * (size_t)p->total_cells);
}

dppix_status_t check_backward(dppix_plan_t p, const dppix_store_t* store, const float* const* grad_out,
                              const uint8_t* clip_bg, const uint8_t* clip_fg, float* const* grad_in)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (p->any_u8)
        return fail(DPPIX_EINVAL, "backward needs every frame in F32_CHW layout");
    if (grad_out == nullptr || grad_in == nullptr || clip_bg == nullptr || clip_fg == nullptr)
        return fail(DPPIX_EINVAL, "grad_out, grad_in and clip bits are required");
    return check_store(store, true);
}

dppix_status_t run_backward(dppix_plan_t p, const dppix_store_t* store, const float* const* grad_out,
                            const uint8_t* clip_bg, const uint8_t* clip_fg, float* const* grad_in, uint8_t* sc,
                            dppix_stream_t stream);

// Fixed device scratch of dp_pix_backward_static, for callers that cannot
// allocate.  Each device holds its own copy of the array from the library's
// load until the process ends.  In host code `scratch` names a host-side
// stand-in: kernels get the device address that hipGetSymbolAddress returns
// for the current device, looked up once per device and kept.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

std::mutex g_scratch_mu;
std::vector<uint8_t*> g_scratch_ptr;  // per device; nullptr until looked up

dppix_status_t static_scratch(uint8_t** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return dev_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if ((size_t)dev >= g_scratch_ptr.size())
        g_scratch_ptr.resize((size_t)dev + 1, nullptr);
    if (g_scratch_ptr[dev] == nullptr) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return dev_fail(e, "hipGetSymbolAddress(scratch)");
        if (ptr == nullptr || (reinterpret_cast<uintptr_t>(ptr) & 255) != 0)
            return fail(DPPIX_EDEVICE, "device scratch has no 256-byte aligned address");
        g_scratch_ptr[dev] = static_cast<uint8_t*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return DPPIX_OK;
}

}  // namespace

extern "C" {

dppix_status_t dp_pix_plan(dppix_plan_t p, const uint8_t* const* masks, const dppix_store_t* store,
                           dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if ((st = check_store(store, false)) != DPPIX_OK)
        return st;
    TileArgs a = base_args(p, store);
    a.masks = masks;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = launch_plan(a, p->n_units, plain_threads(p), p->lds[kPlan], p->prefix_scan, s);
    if (e != hipSuccess)
        return dev_fail(e, "plan launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_plan_labels(dppix_plan_t p, const void* const* images, int32_t threshold,
                                  const dppix_store_t* store, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (p->any_f32)
        return fail(DPPIX_EINVAL, "labels are computed from U8_HWC frames");
    if (images == nullptr)
        return fail(DPPIX_EINVAL, "images is NULL");
    if (threshold < 0 || threshold > 4 * 1024)
        return fail(DPPIX_EINVAL, "threshold must be in 0..4096");
    if ((st = check_store(store, false)) != DPPIX_OK)
        return st;
    TileArgs a = base_args(p, store);
    a.images = images;
    a.edge_threshold = threshold;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = for_channels(p, a, p->lab, p->ws.lab_spans, [&](const TileArgs& ca, int C, int64_t units) {
        return launch_plan_labels(ca, C, units, p->lab_threads, label_lds(p->lab_threads) + 4 * p->lab_cells, s);
    });
    if (e == hipSuccess)
        e = launch_scan(a, p->prefix_scan, s);
    if (e != hipSuccess)
        return dev_fail(e, "plan launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_store_index(dppix_plan_t p, const dppix_store_t* store, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if ((st = check_store(store, false)) != DPPIX_OK)
        return st;
    TileArgs a = base_args(p, store);
    hipError_t e = launch_store_index(a, p->prefix_scan, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return dev_fail(e, "store index launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_forward(dppix_plan_t p, const void* const* images, const dppix_store_t* store,
                              uint8_t* clip_bg, uint8_t* clip_fg, void* const* fused_out, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (images == nullptr)
        return fail(DPPIX_EINVAL, "images is NULL");
    if ((st = check_store(store, true)) != DPPIX_OK)
        return st;
    if ((clip_bg == nullptr) != (clip_fg == nullptr))
        return fail(DPPIX_EINVAL, "clip_bg and clip_fg must both be given or both be NULL");
    TileArgs a = base_args(p, store);
    a.images = images;
    a.outs = fused_out;
    a.clip_bg = clip_bg;
    a.clip_fg = clip_fg;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = for_groups(p, a, false, [&](const TileArgs& ga, const LaunchGroup& g, size_t lds, int grid) {
        return launch_forward(ga, g.layout, g.C, group_threads(p, g, false), lds, grid, s);
    });
    if (e != hipSuccess)
        return dev_fail(e, "forward launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_reconstruct(dppix_plan_t p, const dppix_store_t* store, void* const* out, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (out == nullptr)
        return fail(DPPIX_EINVAL, "out is NULL");
    if ((st = check_store(store, true)) != DPPIX_OK)
        return st;
    TileArgs a = base_args(p, store);
    a.outs = out;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = for_groups(p, a, true, [&](const TileArgs& ga, const LaunchGroup& g, size_t lds, int grid) {
        return launch_reconstruct(ga, g.layout, g.C, g.paced, group_threads(p, g, true), lds, grid, s);
    });
    if (e != hipSuccess)
        return dev_fail(e, "reconstruct launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_backward(dppix_plan_t p, const dppix_store_t* store, const float* const* grad_out,
                               const uint8_t* clip_bg, const uint8_t* clip_fg, float* const* grad_in, void* scratch,
                               size_t scratch_bytes, dppix_stream_t stream)
{
    dppix_status_t st = check_backward(p, store, grad_out, clip_bg, clip_fg, grad_in);
    if (st != DPPIX_OK)
        return st;
    if (scratch == nullptr || scratch_bytes < grad_scratch_need(p))
        return fail(DPPIX_ENOMEM, "scratch smaller than grad_scratch_bytes");
    return run_backward(p, store, grad_out, clip_bg, clip_fg, grad_in, static_cast<uint8_t*>(scratch), stream);
}

dppix_status_t dp_pix_backward_static(dppix_plan_t p, const dppix_store_t* store, const float* const* grad_out,
                                      const uint8_t* clip_bg, const uint8_t* clip_fg, float* const* grad_in,
                                      dppix_stream_t stream)
{
    dppix_status_t st = check_backward(p, store, grad_out, clip_bg, clip_fg, grad_in);
    if (st != DPPIX_OK)
        return st;
    if (grad_scratch_need(p) > kStaticScratchBytes)
        return fail(DPPIX_ENOMEM, "backward needs " + std::to_string(grad_scratch_need(p)) +
                                      " bytes of scratch; the fixed device scratch holds " +
                                      std::to_string(kStaticScratchBytes) + " (use dp_pix_backward)");
    uint8_t* sc = nullptr;
    if ((st = static_scratch(&sc)) != DPPIX_OK)
        return st;
    return run_backward(p, store, grad_out, clip_bg, clip_fg, grad_in, sc, stream);
}

}  // extern "C"

namespace {

dppix_status_t run_backward(dppix_plan_t p, const dppix_store_t* store, const float* const* grad_out,
                            const uint8_t* clip_bg, const uint8_t* clip_fg, float* const* grad_in, uint8_t* sc,
                            dppix_stream_t stream)
{
    TileArgs a = base_args(p, store);
    a.grad_out = grad_out;
    a.grad_in = grad_in;
    a.clip_bg = const_cast<uint8_t*>(clip_bg);
    a.clip_fg = const_cast<uint8_t*>(clip_fg);
    a.g_bg = reinterpret_cast<float*>(sc);
    a.g_fg = reinterpret_cast<float*>(sc + align256(4 * p->bg_cap));
    a.cell_index = reinterpret_cast<uint32_t*>(sc + align256(4 * p->bg_cap) + align256(4 * p->fg_cap));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // 1. gradient of every statistic (store layout): pass * sum of grad_out
    // over its real pixels / area, broadcast in the same tile to the real
    // pixels of the statistic (grad_in)
    hipError_t e = launch_backward_reduce(a, plain_threads(p), p->lds[kBwd],
                                          grid_for(p, 1, 1, plain_threads(p), p->n_tiles, p->lds[kBwd]), s);
    if (e != hipSuccess)
        return dev_fail(e, "backward launch");
    // 2. mirror terms of the pixels near padded borders: no launch at all
    // when no frame is padded
    if (span_total(p->border) > 0) {
        a.spans = reinterpret_cast<const UnitSpan*>(p->bound + p->ws.border_spans);
        a.n_spans = (int32_t)p->border.size() - 1;
        a.span_units = equal_units(p->border, 0, a.n_spans);
        e = launch_backward_mirror(a, span_total(p->border), plain_threads(p), s);
        if (e != hipSuccess)
            return dev_fail(e, "backward launch");
    }
    return DPPIX_OK;
}

}  // namespace

extern "C" {

dppix_status_t dp_pix_debug_sums(dppix_plan_t p, const void* const* images, const dppix_store_t* store,
                                 uint32_t* coarse, uint32_t* fine, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (p->any_f32)
        return fail(DPPIX_EINVAL, "debug sums are for U8_HWC frames");
    if (images == nullptr || coarse == nullptr || fine == nullptr)
        return fail(DPPIX_EINVAL, "images, coarse and fine are required");
    if ((st = check_store(store, true)) != DPPIX_OK)
        return st;
    TileArgs a = base_args(p, store);
    a.images = images;
    a.dbg_coarse = coarse;
    a.dbg_fine = fine;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = for_groups(p, a, false, [&](const TileArgs& ga, const LaunchGroup& g, size_t lds, int grid) {
        return launch_forward(ga, g.layout, g.C, group_threads(p, g, false), lds, grid, s);
    });
    if (e != hipSuccess)
        return dev_fail(e, "forward launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_edge_mask(dppix_plan_t p, const void* const* images, int32_t threshold, uint8_t* const* masks_out,
                                dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (p->any_f32)
        return fail(DPPIX_EINVAL, "edge masks are computed from U8_HWC frames");
    if (images == nullptr || masks_out == nullptr)
        return fail(DPPIX_EINVAL, "images and masks_out are required");
    if (threshold < 0 || threshold > 4 * 1024)
        return fail(DPPIX_EINVAL, "threshold must be in 0..4096");
    TileArgs a = base_args(p, nullptr);
    a.images = images;
    a.masks_out = masks_out;
    a.edge_threshold = threshold;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    a.edge_rows = p->edge_rows;
    hipError_t e = for_channels(p, a, p->edge, p->ws.edge_spans, [&](const TileArgs& ca, int C, int64_t units) {
        return launch_edge_mask(ca, C, units, p->edge_threads, label_lds(p->edge_threads), s);
    });
    if (e != hipSuccess)
        return dev_fail(e, "edge mask launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_metrics(dppix_plan_t p, const void* const* images, const void* const* recons, void* scratch,
                              size_t scratch_bytes, double* out, dppix_stream_t stream)
{
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (p->any_f32)
        return fail(DPPIX_EINVAL, "metrics are computed on U8_HWC frames");
    if (images == nullptr || recons == nullptr || out == nullptr)
        return fail(DPPIX_EINVAL, "images, recons and out are required");
    if (scratch == nullptr || scratch_bytes < 16 * (size_t)span_total(p->met))
        return fail(DPPIX_ENOMEM, "scratch smaller than metrics_scratch_bytes");
    TileArgs a = base_args(p, nullptr);
    a.images = images;
    a.outs = const_cast<void* const*>(recons);
    a.met_partial = static_cast<double*>(scratch);
    a.met_rows = p->met_rows;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipError_t e = for_channels(p, a, p->met, p->ws.met_spans, [&](const TileArgs& ca, int C, int64_t units) {
        return launch_metrics(ca, C, p->met_narrow[C - 1], units, s);
    });
    if (e != hipSuccess)
        return dev_fail(e, "metrics launch");
    a.spans = reinterpret_cast<const UnitSpan*>(p->bound + p->ws.met_spans);
    e = launch_metrics_reduce(a, out, s);
    if (e != hipSuccess)
        return dev_fail(e, "metrics reduce launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_noise_advance(uint64_t* noise, int32_t n_frames, uint64_t step, dppix_stream_t stream)
{
    if (n_frames < 0 || (n_frames > 0 && noise == nullptr))
        return fail(DPPIX_EINVAL, "noise must hold n_frames >= 0 counter pairs");
    if ((reinterpret_cast<uintptr_t>(noise) & 7) != 0)
        return fail(DPPIX_EINVAL, "noise must be 8-byte aligned");
    hipError_t e = launch_noise_advance(noise, n_frames, step, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return dev_fail(e, "noise advance launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_debug_philox(const uint32_t* in, uint32_t* words, int64_t n, dppix_stream_t stream)
{
    if (n < 0 || (n > 0 && (in == nullptr || words == nullptr)))
        return fail(DPPIX_EINVAL, "bad philox arguments");
    hipError_t e = launch_philox(in, words, n, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return dev_fail(e, "philox launch");
    return DPPIX_OK;
}

dppix_status_t dp_pix_graph_create(dppix_plan_t p, const uint8_t* const* masks, const void* const* images,
                                   const dppix_store_t* store, void* const* fused_out, dppix_stream_t stream,
                                   dppix_graph_t* out)
{
    if (out == nullptr)
        return fail(DPPIX_EINVAL, "out is NULL");
    *out = nullptr;
    dppix_status_t st = need_bound(p);
    if (st != DPPIX_OK)
        return st;
    if (images == nullptr || (st = check_store(store, true)) != DPPIX_OK)
        return st == DPPIX_OK ? fail(DPPIX_EINVAL, "images is NULL") : st;
    // The legacy default stream cannot be captured; capture on a private
    // non-blocking stream instead (the graph does not depend on it).
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipStream_t own = nullptr;
    if (s == nullptr) {
        hipError_t ec = hipStreamCreateWithFlags(&own, hipStreamNonBlocking);
        if (ec != hipSuccess)
            return dev_fail(ec, "capture stream");
        s = own;
    }
    hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        if (own)
            (void)hipStreamDestroy(own);
        return dev_fail(e, "begin capture");
    }
    dppix_stream_t cs = reinterpret_cast<dppix_stream_t>(s);
    dppix_status_t s1 = dp_pix_plan(p, masks, store, cs);
    dppix_status_t s2 = s1 == DPPIX_OK ? dp_pix_forward(p, images, store, nullptr, nullptr, fused_out, cs) : s1;
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(s, &g);
    if (own)
        (void)hipStreamDestroy(own);
    if (s2 != DPPIX_OK) {
        if (g)
            (void)hipGraphDestroy(g);
        return s2;
    }
    if (e != hipSuccess)
        return dev_fail(e, "end capture");
    dppix_graph* G = new (std::nothrow) dppix_graph;
    if (G == nullptr) {
        (void)hipGraphDestroy(g);
        return fail(DPPIX_ENOMEM, "host allocation failed");
    }
    G->graph = g;
    e = hipGraphInstantiate(&G->exec, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        delete G;
        return dev_fail(e, "graph instantiate");
    }
    *out = G;
    return DPPIX_OK;
}

dppix_status_t dp_pix_graph_launch(dppix_graph_t g, dppix_stream_t stream)
{
    if (g == nullptr)
        return fail(DPPIX_EINVAL, "NULL graph");
    hipError_t e = hipGraphLaunch(g->exec, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return dev_fail(e, "graph launch");
    return DPPIX_OK;
}

void dp_pix_graph_destroy(dppix_graph_t g)
{
    if (g == nullptr)
        return;
    if (g->exec)
        (void)hipGraphExecDestroy(g->exec);
    if (g->graph)
        (void)hipGraphDestroy(g->graph);
    delete g;
}

}  // extern "C"
