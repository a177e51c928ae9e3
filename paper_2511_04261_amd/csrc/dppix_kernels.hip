// dppix_kernels.hip — gfx950 kernels of libdppix.
//
// The path is bandwidth-bound: per pixel it reads the image (and, in the plan,
// the mask) once and writes the reconstruction once; the statistics are a few
// percent of that.  Nothing is a dense contraction, so there is no MFMA work.
// Every tile kernel follows one pattern:
//   1. a work item is one 16-byte strip of the tile's padded rows over one
//      (or a few) subgrid rows; it issues all of its row loads, then sums
//      them in registers (two 16-bit lanes per 32-bit register for bytes:
//      255 * 256 rows still fits);
//   2. the column sums go to LDS, where one lane per (subcell column,
//      channel) adds its s_b columns — exact integer sums of every s_b x s_b
//      subcell;
//   3. a coarse cell's sum is the exact total of its n x n subcell sums
//      (Eq. 16-17: b = n * s_b), so simple and complex cells cost the same;
//   4. each released statistic draws one Philox4x32-10 block, turns it into
//      Laplace noise in fp64, clips and rounds once to fp32 (the releases
//      of complex subcells are dealt evenly over the lanes);
//   5. with a fused output, the rounded values are expanded into one padded
//      row in LDS and the strips are stored on the s_b output rows.
// Mirror padding (Algorithm 2 step 4, Algorithm 3 step 3) is never
// materialised: padded rows fold to a source row per row, and a padded
// column's sums are copies of the sums of the column it mirrors, already in
// LDS.  The unpadded mode (Algorithm 1) skips those rows and columns and
// divides by real pixel counts.
#include "dppix_internal.h"
#include "dppix_tiles.h"

#include <math.h>

#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

// Register budget of the u8 forward kernel, as resident waves per SIMD: 4
// leaves 128 VGPRs for all of a subgrid row's loads in flight.  That is just
// short: the compiler keeps up to 20 bytes a lane in scratch (RGB) and about 190
// scalar registers in lanes of vector registers.
#ifndef DPPIX_FWD_WAVES_PER_EU
#define DPPIX_FWD_WAVES_PER_EU 4
#endif

namespace dppix {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// 16-byte streaming accesses through global (not flat) address space: frame
// pointers come from device tables, so the compiler cannot infer the address
// space, and flat accesses would make every wait cover LDS traffic as well.
// Rows start at any byte (any float): global vector accesses need no more
// than that, and a row of 16-byte strips off the line grid costs one more line
// per wave, where single bytes would cost sixteen times the accesses.
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(1)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) v4u_any g_v4u;
typedef __attribute__((address_space(1))) v4f_any g_v4f;
typedef __attribute__((address_space(1))) const uint8_t g_u8;
typedef __attribute__((address_space(1))) uint8_t g_u8w;
typedef __attribute__((address_space(1))) const float g_f32;
typedef __attribute__((address_space(1))) float g_f32w;

__device__ __forceinline__ v4u ld16_nt(const void* p) { return __builtin_nontemporal_load((const g_v4u*)p); }
// For groups of C vectors a lane: each of its loads touches lines that the
// others need too, so they are kept.
__device__ __forceinline__ v4u ld16(const void* p) { return *(const g_v4u*)p; }
__device__ __forceinline__ v4f ld16f_nt(const void* p) { return __builtin_nontemporal_load((const g_v4f*)p); }
__device__ __forceinline__ void st16_nt(void* p, v4u v) { __builtin_nontemporal_store(v, (g_v4u*)p); }
__device__ __forceinline__ void st16f_nt(void* p, v4f v) { __builtin_nontemporal_store(v, (g_v4f*)p); }

// --------------------------------------------------------------------------
// Counter-based noise.  Philox4x32 with ten rounds (Salmon et al., SC'11):
// per round the first and third words are multiplied by two fixed odd
// constants, the high halves of the products are xored with the other two
// words and the round key, and the key advances by two Weyl increments.
// --------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // one 32x32 -> 64-bit product per multiplier gives both halves
        const uint64_t pa = (uint64_t)0xD2511F53u * c.x;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4(xor3((uint32_t)(pb >> 32), c.y, k0), (uint32_t)pb, xor3((uint32_t)(pa >> 32), c.w, k1),
                       (uint32_t)pa);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// Natural log of x in (0, 1] (the Laplace draw's arguments are 2u and
// 2(1-u), never 0, infinite or subnormal), within one ulp: x = m 2^e with m in
// [sqrt(1/2), sqrt(2)), f = m - 1 (exact), s = f / (2 + f), and
// ln(1 + f) = 2 atanh(s) = 2s + sum_{k>=1} 2 s^(2k+1) / (2k+1).  Since
// 2s = f - f^2 / (2 + f), the sum is arranged as f - h + s (h + R) with
// h = f^2 / 2 and R = sum_{k=1..10} 2 z^k / (2k+1), z = s^2 <= 0.0295, so the
// two large terms are exact and the series (truncated below 2^-56 relative)
// only corrects.  ln 2 is split into 42 leading bits (e ln2_hi is exact) and
// the rest.  Against the C library's log on 2e7 such arguments it agrees
// exactly on 93 % and within one ulp on all.
//
// The draws are vector work (fine grids are bound by them), so the division
// is the plain refinement of the reciprocal, without the scaling and fix-up
// that operands of any magnitude need (f and 2 + f are normal and far from the
// ends of the range, and the quotient is the same, correctly rounded, one),
// the exponent comes off the high word, and each coefficient is an operand of
// its fma instead of a register filled beforehand.  A draw with its Philox
// block took about 450 cycles of a SIMD and takes 330; 16 x 1080p RGB, b 4 /
// s_b 2: forward 136 -> 128 us, b 2 / s_b 1, 8 frames: 234 -> 218.
// a b + c with c a constant in scalar registers.
__device__ __forceinline__ double fma_const(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

__device__ __forceinline__ double ln_unit(double x)
{
    // m = x 2^-e from sqrt(1/2) on (its high word's worth of it)
    const uint64_t bits = __builtin_bit_cast(uint64_t, x);
    const int32_t hi = (int32_t)(bits >> 32);
    const int32_t e = (hi - 0x3FE6A09E) >> 20;
    const double m = __builtin_bit_cast(double, (bits & 0xFFFFFFFFull) | ((uint64_t)(uint32_t)(hi - (e << 20)) << 32));
    const double f = m - 1.0;
    const double d = 2.0 + f;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    r = fma(r, fma(-d, r, 1.0), r);
    const double s0 = f * r;
    const double s = fma(fma(-d, s0, f), r, s0);
    const double z = s * s;
    double R = fma_const(2.0 / 21.0, z, 2.0 / 19.0);
    R = fma_const(R, z, 2.0 / 17.0);
    R = fma_const(R, z, 2.0 / 15.0);
    R = fma_const(R, z, 2.0 / 13.0);
    R = fma_const(R, z, 2.0 / 11.0);
    R = fma_const(R, z, 2.0 / 9.0);
    R = fma_const(R, z, 2.0 / 7.0);
    R = fma_const(R, z, 2.0 / 5.0);
    R = fma_const(R, z, 2.0 / 3.0);
    R *= z;
    const double h = 0.5 * f * f;
    const double de = (double)e;
    return de * 0x1.62e42fefa3800p-1 - ((h - (s * (h + R) + de * 0x1.ef35793c76730p-45)) - f);
}

// Laplace(0, sigma) sample of one statistic: words 0,1 of the block give a
// uniform u = (2k+1) 2^-53 with k the top 52 bits, inverted through the
// Laplace CDF (Eq. 9) in fp64.
__device__ __forceinline__ double laplace_sample(const FrameRec& F, uint32_t id, int ch, int level, double sigma)
{
    // The key is one frame's, the same in every lane (readfirstlane states
    // that, so it sits in scalar registers at any optimisation level).  The
    // empty asm makes it opaque here, so the ten round keys are recomputed by
    // one scalar add per round instead of being hoisted out of the caller's
    // release loop: there they would take 20 scalar registers the tile
    // kernels do not have, and be spilled to vector lanes and read back by a
    // vector instruction each.
    uint32_t k0 = __builtin_amdgcn_readfirstlane(F.key0), k1 = __builtin_amdgcn_readfirstlane(F.key1);
    asm volatile("" : "+s"(k0), "+s"(k1));
    const uint4 w = philox10(make_uint4(id, (uint32_t)ch | ((uint32_t)level << 8), F.fi0, F.fi1), k0, k1);
    // u - 1/2 and 2 min(u, 1 - u), exactly: 1 + k 2^-52 is built from its
    // bits, and every step below stays within 53 bits
    const uint64_t k = (((uint64_t)w.y << 32) | (uint64_t)w.x) >> 12;
    const double t = (__builtin_bit_cast(double, k | 0x3FF0000000000000ull) - 1.5) + 0x1p-53;
    // one log per lane: the two tails differ only in its argument and sign
    return copysign(sigma * ln_unit(fma(-2.0, fabs(t), 1.0)), t);
}

// Release one statistic: mean = sum / area, plus noise (Eq. 11 scale given by
// the host), clipped to [0, 255] (Algorithm 3 steps 10, 17), one rounding to
// fp32.  pass = the clip did not bind (gradient flows).  inv_area: 1 / area
// when that is exact (area a power of two: the product then equals the
// quotient bit for bit), else 0 (divide).
// FLOATS: the sum is of fp32 pixels and may be NaN (a NaN pixel, or both
// infinities in one cell), which the comparisons let through as they let it
// through in the oracle: a diverged input must not come out as a valid black.
// Sums of bytes are finite, and take the min and max of half the instructions.
template <bool FLOATS>
__device__ __forceinline__ float release(double sum, double area, double inv_area, int noisy, double sigma,
                                         const FrameRec& F, uint32_t id, int ch, int level, uint8_t& pass)
{
    if (area == 0.0) {   // unpadded mode: a subcell with no real pixel releases nothing
        pass = 0;
        return 0.f;
    }
    const double mu = inv_area != 0.0 ? sum * inv_area : sum / area;
    const double z = noisy ? mu + laplace_sample(F, id, ch, level, sigma) : mu;
    pass = (uint8_t)(z >= 0.0 && z <= 255.0);
    if constexpr (FLOATS)
        return (float)(z < 0.0 ? 0.0 : (z > 255.0 ? 255.0 : z));
    return (float)fmin(fmax(z, 0.0), 255.0);
}

__device__ __forceinline__ uint8_t to_u8(float v) { return (uint8_t)rintf(v); }

// Quotients x / d of item numbers by one divisor, 0 <= x < 2^20: the rounded
// (x + 1/2) / d is off by less than 2^-22 of itself, so less than the half
// step that keeps it from the next integer.  Three instructions, where the
// division of any two integers takes about 25.
struct FastDiv {
    float inv, half;
    __device__ __forceinline__ explicit FastDiv(int d) : inv(__builtin_amdgcn_rcpf((float)d)), half(0.5f * inv) {}
    __device__ __forceinline__ int operator()(int x) const { return (int)fmaf((float)x, inv, half); }
};

// The same for 0 <= x < 2^24: the quotient is at most one off (a reciprocal one
// ulp off, d >= 3; those of 1 and 2 are exact), and the remainder says which way.
struct WideDiv {
    FastDiv by;
    int d;
    __device__ __forceinline__ explicit WideDiv(int d_) : by(d_), d(d_) {}
    __device__ __forceinline__ int operator()(int x) const
    {
        const int q = by(x), r = x - q * d;
        return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
    }
};

// 1 / side^2 when that is exact and every statistic of that side has area
// side^2 (mirror padding, side a power of two), else 0.
__device__ __forceinline__ double exact_inv_area(const FrameRec& F, int side)
{
    return (F.pad != kPadNone && (side & (side - 1)) == 0) ? 1.0 / ((double)side * (double)side) : 0.0;
}

// Real-pixel area of the statistic whose (sub)cell starts at padded (y0, x0)
// with the given side: side^2 when the frame is mirror-padded; h*w real
// pixels in the unpadded mode (0 for a subcell wholly past the frame).
__device__ __forceinline__ double stat_area(const FrameRec& F, int y0, int x0, int side)
{
    if (F.pad != kPadNone)
        return (double)side * (double)side;
    const int h = min(side, F.H - y0), w = min(side, F.W - x0);
    return (h > 0 && w > 0) ? (double)h * (double)w : 0.0;
}

__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Workgroup barrier for LDS hand-offs only.  The tile kernels never read
// global memory written by their own workgroup, so outstanding global stores
// (the reconstruction, the store) need not drain at every barrier, which a
// full __syncthreads() would force.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Bytes 1 and 3 of a dword in the low bytes of its two 16-bit halves: one
// byte permute (selector bytes 1, zero, 3, zero) instead of a shift and a mask.
__device__ __forceinline__ uint32_t odd_bytes(uint32_t w) { return __builtin_amdgcn_perm(0u, w, 0x0C030C01u); }

// Add the bytes of one 16-byte strip into 16-bit lane pairs: e[d] holds bytes
// 4d and 4d+2, o[d] bytes 4d+1 and 4d+3.
__device__ __forceinline__ void acc_bytes(const v4u& w, uint32_t (&e)[4], uint32_t (&o)[4])
{
    e[0] += w.x & 0x00FF00FFu; o[0] += odd_bytes(w.x);
    e[1] += w.y & 0x00FF00FFu; o[1] += odd_bytes(w.y);
    e[2] += w.z & 0x00FF00FFu; o[2] += odd_bytes(w.z);
    e[3] += w.w & 0x00FF00FFu; o[3] += odd_bytes(w.w);
}

// Nonzero bytes of a dword as 0/1 bytes.
__device__ __forceinline__ uint32_t nz_bytes(uint32_t w)
{
    return ((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) >> 7) & 0x01010101u;
}

// Column sums of a strip as 16-bit values in natural byte-column order (a
// subgrid row has at most 256 rows of bytes, so 255 * 256 fits).
__device__ __forceinline__ void store_colsums16(uint16_t* dst, const uint32_t (&e)[4], const uint32_t (&o)[4])
{
    if ((reinterpret_cast<uintptr_t>(dst) & 15) != 0) {
        // the last strip of a tile's real columns, moved back to end with them
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            dst[4 * d] = (uint16_t)e[d];
            dst[4 * d + 1] = (uint16_t)o[d];
            dst[4 * d + 2] = (uint16_t)(e[d] >> 16);
            dst[4 * d + 3] = (uint16_t)(o[d] >> 16);
        }
        return;
    }
    v4u* d4 = reinterpret_cast<v4u*>(dst);
    d4[0] = v4u{(e[0] & 0xFFFFu) | (o[0] << 16), (e[0] >> 16) | (o[0] & 0xFFFF0000u),
                (e[1] & 0xFFFFu) | (o[1] << 16), (e[1] >> 16) | (o[1] & 0xFFFF0000u)};
    d4[1] = v4u{(e[2] & 0xFFFFu) | (o[2] << 16), (e[2] >> 16) | (o[2] & 0xFFFF0000u),
                (e[3] & 0xFFFFu) | (o[3] << 16), (e[3] >> 16) | (o[3] & 0xFFFF0000u)};
}

// How a tile's rows are cut into strips of `unit` elements (16 bytes, or 4
// floats): `real` elements of the tile's padded width lie in the frame.  With
// `vec` every real element is read by a whole vector (`nvec` strips, the last
// one moved back to end with the real columns: the columns it shares with its
// neighbour are written twice with equal sums), and the padded columns after
// them are copies of column sums the tile already has (a column's mirror
// image has its sum) or zero.  A tile of fewer real columns than one strip,
// or than its padding mirrors, is read element by element instead.
// 24 RGB photos of odd widths (22.9 MP, b 16 / s_b 4), before (strips off the
// 16-byte grid and at the right edge gathered and stored byte by byte) and
// after: forward 151 -> 44 us, reconstruction 89 -> 27 us (23 with the present
// workgroup sizes), plan 53 -> 14 us; 64 fp32 crops of 218 x 178: forward 40 -> 30
// us (18 with them).  Aligned batches unchanged.
struct Strips {
    int real, nvec;
    bool vec;
};

__device__ __forceinline__ Strips tile_strips_of(int width, int real, int unit, int per_pixel, int pad)
{
    Strips s;
    s.real = real;
    const int padded = (width - real) / per_pixel, px = real / per_pixel;
    s.vec = real >= unit && (padded == 0 || pad == kPadNone || padded <= px - (pad == 1 ? 1 : 0));
    s.nvec = (real + unit - 1) / unit;
    return s;
}

// Tile-local source column of padded column x (both in pixels; px real ones).
__device__ __forceinline__ int mirror_col(int x, int px, int pad) { return pad == 1 ? 2 * px - 2 - x : 2 * px - 1 - x; }

// 16 bytes of LDS from any byte address.
__device__ __forceinline__ v4u lds16(const uint8_t* p)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(p);
    if ((at & 15) == 0)
        return *reinterpret_cast<const v4u*>(p);
    const uint32_t sh = (uint32_t)(at & 3);
    const uint32_t* w = reinterpret_cast<const uint32_t*>(p - sh);
    const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3], w4 = sh ? w[4] : 0u;
    return v4u{__builtin_amdgcn_alignbyte(w1, w0, sh), __builtin_amdgcn_alignbyte(w2, w1, sh),
               __builtin_amdgcn_alignbyte(w3, w2, sh), __builtin_amdgcn_alignbyte(w4, w3, sh)};
}

// Cell classes and class-local indices of the tile's cells (wave 0):
// complex cells count from the number of complex cells of the frame before
// the tile, simple cells from the simple ones — row-major order, which is the
// order of the compact store.
// With cxl, also the list of the tile's complex cells in order (cxl[q] = kc
// of the q-th complex cell) and their number in *ncx.
__device__ __forceinline__ void tile_cells(const TileArgs& a, const FrameRec& F, int64_t t, int r, int x0c, int Kt,
                                           uint32_t* cidx, uint8_t* cflag, uint16_t* cxl = nullptr,
                                           uint32_t* ncx = nullptr)
{
    if (threadIdx.x >= 64)
        return;
    const int lane = threadIdx.x;
    uint32_t run_fg = a.tile_fg[t];
    const uint32_t fg0 = run_fg;
    const uint32_t before = (uint32_t)(r * F.GC + x0c);
    uint32_t run_bg = before - run_fg;
    for (int base = 0; base < Kt; base += 64) {
        const int kc = base + lane;
        const bool in = kc < Kt;
        const uint8_t fl = in ? a.flags[F.cell_base + before + kc] : (uint8_t)0;
        const uint64_t m = __ballot(fl != 0);
        const uint64_t below = lane ? (m & (~0ull >> (64 - lane))) : 0ull;
        const uint32_t pc = (uint32_t)__popcll(below);
        if (in) {
            cflag[kc] = fl;
            cidx[kc] = fl ? run_fg + pc : run_bg + (uint32_t)lane - pc;
            if (cxl && fl)
                cxl[run_fg - fg0 + pc] = (uint16_t)kc;
            if (a.cell_index)
                a.cell_index[F.cell_base + before + kc] = cidx[kc];
        }
        const uint32_t nf = (uint32_t)__popcll(m);
        const uint32_t nv = (uint32_t)min(64, Kt - base);
        run_fg += nf;
        run_bg += nv - nf;
    }
    if (ncx && lane == 0)
        *ncx = run_fg - fg0;
}

struct TileCoord {
    int f;
    int64_t t;
    int r, ct;
};

__device__ __forceinline__ TileCoord tile_of(const TileArgs& a, int64_t sched_idx, FrameRec& F)
{
    TileCoord tc;
    // one load: (frame, tile within frame) of this scheduling index
    const int64_t idx = a.sched_offset + sched_idx;
    tc.f = (int)uniform_u32((uint32_t)a.tile_map[2 * idx]);
    const uint32_t local = uniform_u32((uint32_t)a.tile_map[2 * idx + 1]);
    F = a.frames[tc.f];
    if (a.noise != nullptr) {
        // this call's noise counters, read at launch time (a replayed graph
        // draws fresh noise once the caller has advanced them)
        const uint64_t key = a.noise[2 * tc.f], ctr = a.noise[2 * tc.f + 1];
        F.key0 = (uint32_t)key;
        F.key1 = (uint32_t)(key >> 32);
        F.fi0 = (uint32_t)ctr;
        F.fi1 = (uint32_t)(ctr >> 32);
    }
    tc.t = F.tile_base + local;
    tc.r = (int)(local / (uint32_t)F.TX);
    tc.ct = (int)(local - (uint32_t)tc.r * (uint32_t)F.TX);
    return tc;
}

// The frame of a unit and the unit's number within it, by the launch's spans.
// Where all frames have as many units, by a division (metrics of 4 x 1080p 55.5
// us, with the search 56.7; of 512 x 32 x 32 10.7 / 11.2; label plan of 16 x
// 1080p 33.6 / 33.9); else each wave compares 64 spans at a time (one load up to
// 64 frames, two up to 4096).  Every lane of the wave calls it.
struct UnitCoord {
    int f, local;
};

__device__ __forceinline__ UnitCoord unit_of(const TileArgs& a, int64_t unit)
{
    UnitCoord u;
    if (a.span_units != 0) {
        const uint32_t k = (uint32_t)(unit - a.sched_offset) / (uint32_t)a.span_units;
        u.f = (int)uniform_u32((uint32_t)a.spans[k].frame);
        u.local = (int)((uint32_t)(unit - a.sched_offset) - k * (uint32_t)a.span_units);
        return u;
    }
    const int lane = threadIdx.x & 63;
    const auto* spans = (const __attribute__((address_space(1))) UnitSpan*)a.spans;
    int lo = 0, n = a.n_spans;
    while (n > 64) {
        const int step = (n + 63) >> 6, at = lane * step;
        const bool before = at < n && spans[lo + at].first <= unit;
        const int last = __popcll(__ballot(before)) - 1;
        lo += last * step;
        n = min(step, n - last * step);
    }
    UnitSpan s = {0, 0, 0};
    if (lane < n) {
        s.first = spans[lo + lane].first;
        s.frame = spans[lo + lane].frame;
    }
    const int last = __popcll(__ballot(lane < n && s.first <= unit)) - 1;
    u.f = __builtin_amdgcn_readlane(s.frame, last);
    u.local = (int)unit - __builtin_amdgcn_readlane((int)s.first, last);   // (below 2^31, whatever the high words)
    return u;
}

// ==========================================================================
// Scans of the plan.
// ==========================================================================
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* wave_tot, T& total)
{
    // inclusive scan inside the wavefront
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    T x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T y = __shfl_up(x, d, 64);
        if (lane >= d)
            x += y;
    }
    if (lane == 63)
        wave_tot[wid] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int i = 0; i < nw; ++i) {
            const T w = wave_tot[i];
            wave_tot[i] = run;
            run += w;
        }
        wave_tot[nw] = run;
    }
    __syncthreads();
    const T excl = x - v + wave_tot[wid];
    total = wave_tot[nw];
    __syncthreads();
    return excl;
}

// Frame-level pass of the scan (k_scan_frames, one workgroup, launched after
// k_scan_tiles): store offsets of every frame (frames concatenated in batch
// order) from the per-frame counts the tile pass wrote, ticket words reset.
__device__ void scan_frames(const TileArgs& a, uint64_t* wave_tot)
{
    uint64_t carry_bg = 0, carry_fg = 0;
    for (int base = 0; base < a.n_frames; base += blockDim.x) {
        const int f = base + threadIdx.x;
        uint64_t vb = 0, vf = 0;
        if (f < a.n_frames) {
            const FrameRec F = a.frames[f];
            vb = a.counts[4 * f] * (uint64_t)F.C;
            vf = a.counts[4 * f + 1] * (uint64_t)F.n * (uint64_t)F.n * (uint64_t)F.C;
        }
        uint64_t tb, tf;
        const uint64_t eb = block_exclusive_scan<uint64_t>(vb, wave_tot, tb);
        const uint64_t ef = block_exclusive_scan<uint64_t>(vf, wave_tot, tf);
        if (f < a.n_frames) {
            a.counts[4 * f + 2] = carry_bg + eb;
            a.counts[4 * f + 3] = carry_fg + ef;
        }
        carry_bg += tb;
        carry_fg += tf;
    }
    if (threadIdx.x < kTicketWords)
        a.ticket[threadIdx.x] = 0;
}

// ==========================================================================
// Plan (Algorithm 3 steps 3-6): classify every cell from the mirror-padded
// mask (k_plan), then scan the complex counts into store offsets (k_scan_prefix,
// or k_scan_tiles and k_scan_frames).
// A plan unit is `cnb` bands x `ctx` tiles of one frame.  Each lane sums one
// 16-byte strip of the mask down up to kPlanRows padded rows with all its
// loads in flight, then hands the strip's column counts to per-cell counters
// in LDS (at most two cells per strip when b >= 16).  Where every strip is
// whole and b a multiple of 4, four columns are counted by one dot product;
// whole bands of 2 or 4 rows take eight rows an item and count cell by cell.
// 16 x 1080p, b 4: plan 24.5 -> 15.5 us (with the units halved), b 8: 14.5 -> 11.9;
// 8 x 1080p, b 2: 30.1 -> 19.4; 64 x 1080p, b 32: 25.8 -> 25.2 (HBM-bound).  With
// the scan's eight tiles a lane the first three are 13.6, 11.7 and 16.2.
// ==========================================================================
constexpr int kPlanRows = 16;   // padded mask rows one lane sums per item
constexpr int kPlanBatch = 8;   // row loads issued back to back

__device__ __forceinline__ v4u nz_strip(const v4u& w)
{
    return v4u{nz_bytes(w.x), nz_bytes(w.y), nz_bytes(w.z), nz_bytes(w.w)};
}

// Column x (0..15) of a strip's packed counts (see acc_bytes).
template <int X>
__device__ __forceinline__ uint32_t col_count(const uint32_t (&e)[4], const uint32_t (&o)[4])
{
    const uint32_t v = (X & 1) ? o[X >> 2] : e[X >> 2];
    return (X & 2) ? (v >> 16) : (v & 0xFFFFu);
}

template <int X>
__device__ __forceinline__ void spread_col(const uint32_t (&e)[4], const uint32_t (&o)[4], uint32_t* cc, int KC,
                                           int b, int& cell, int& next, uint32_t& run)
{
    if (X == next) {
        if (run != 0u && cell < KC)
            atomicAdd(cc + cell, run);
        run = 0u;
        ++cell;
        next += b;
    }
    run += col_count<X>(e, o);
}

// Add the 16 column counts of one strip that starts at padded column p0 of
// the unit to the counters of the cells they fall in.
__device__ __forceinline__ void spread_strip(const uint32_t (&e)[4], const uint32_t (&o)[4], uint32_t* cc, int KC,
                                             int b, int p0)
{
    int cell = p0 / b;
    int next = (cell + 1) * b - p0;
    uint32_t run = 0u;
    spread_col<0>(e, o, cc, KC, b, cell, next, run);
    spread_col<1>(e, o, cc, KC, b, cell, next, run);
    spread_col<2>(e, o, cc, KC, b, cell, next, run);
    spread_col<3>(e, o, cc, KC, b, cell, next, run);
    spread_col<4>(e, o, cc, KC, b, cell, next, run);
    spread_col<5>(e, o, cc, KC, b, cell, next, run);
    spread_col<6>(e, o, cc, KC, b, cell, next, run);
    spread_col<7>(e, o, cc, KC, b, cell, next, run);
    spread_col<8>(e, o, cc, KC, b, cell, next, run);
    spread_col<9>(e, o, cc, KC, b, cell, next, run);
    spread_col<10>(e, o, cc, KC, b, cell, next, run);
    spread_col<11>(e, o, cc, KC, b, cell, next, run);
    spread_col<12>(e, o, cc, KC, b, cell, next, run);
    spread_col<13>(e, o, cc, KC, b, cell, next, run);
    spread_col<14>(e, o, cc, KC, b, cell, next, run);
    spread_col<15>(e, o, cc, KC, b, cell, next, run);
    if (run != 0u && cell < KC)
        atomicAdd(cc + cell, run);
}

// Nonzero bytes of a dword as 0x80 bytes.
__device__ __forceinline__ uint32_t hit_bytes(uint32_t w)
{
    return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
}

// A row of a strip into its counts: column by column, or four columns a dword.
template <bool QUADS>
__device__ __forceinline__ void count_strip(const v4u& w, uint32_t (&e)[4], uint32_t (&o)[4])
{
    if constexpr (QUADS) {
#pragma unroll
        for (int d = 0; d < 4; ++d)
            e[d] = __builtin_amdgcn_udot4(hit_bytes(w[d]), 0x01010101u, e[d], false);
    } else {
        acc_bytes(nz_strip(w), e, o);
    }
}

// Eight rows of a strip, bands of B = 2 or 4 rows: 16 / B whole cells of each
// band, whose counts go to cc[band * KCs + cell].
template <int B>
__device__ __forceinline__ void count_bands(const v4u (&w)[8], uint32_t* cc, int KCs)
{
#pragma unroll
    for (int q = 0; q < 8 / B; ++q)
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t c[4 / B] = {};
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const uint32_t h = hit_bytes(w[q * B + i][d]);
#pragma unroll
                for (int k = 0; k < 4 / B; ++k)
                    c[k] = __builtin_amdgcn_udot4(h, B == 4 ? 0x01010101u : (k ? 0x01010000u : 0x00000101u), c[k], false);
            }
#pragma unroll
            for (int k = 0; k < 4 / B; ++k)
                if (c[k] != 0u)
                    atomicAdd(cc + q * KCs + d * (4 / B) + k, c[k] >> 7);
        }
}

// Clear the counts of a strip's columns outside [c0, c1).
__device__ __forceinline__ void mask_cols(uint32_t (&e)[4], uint32_t (&o)[4], int c0, int c1)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int x = 4 * d;
        e[d] &= (x >= c0 && x < c1 ? 0xFFFFu : 0u) | (x + 2 >= c0 && x + 2 < c1 ? 0xFFFF0000u : 0u);
        o[d] &= (x + 1 >= c0 && x + 1 < c1 ? 0xFFFFu : 0u) | (x + 3 >= c0 && x + 3 < c1 ? 0xFFFF0000u : 0u);
    }
}

// Mask counts of every cell of the unit into cellcnt[j * KCs + kc].
__device__ void plan_count(const TileArgs& a, const FrameRec& F, const uint8_t* mask, int r0, int nb, int c0, int KC,
                           int KCs, uint32_t* cellcnt)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, H = F.H, W = F.W, pad = F.pad;
    const int64_t X0 = (int64_t)c0 * b;
    const int WB = KC * b;
    const int RI = min(b, kPlanRows);
    const int groups = (b + RI - 1) / RI;
    const int64_t lim = min(X0 + WB, (int64_t)W);
    // Strips [0, nfast) cover the unit's real columns, the last one moved back
    // to end with them (the columns it shares with its neighbour masked off).
    // The padded columns all lie in the frame's last cell (there are fewer
    // than b of them), so their count is that of the columns they mirror,
    // [ms, me): strips [nfast, nfast + nmir), added to that cell whole.
    // Without whole vectors (fewer than 16 real columns, or than the padding
    // mirrors) every column is counted byte by byte.
    const int real = (int)(lim - X0);
    const int padded = WB - real;
    const bool vec = real >= 16 && (padded == 0 || pad == kPadNone || padded <= W - (pad == 1 ? 1 : 0));
    const int nfast = vec ? (real + 15) >> 4 : 0;
    const int me = pad == 1 ? W - 1 : W, ms = me - padded;
    const int nmir = vec && pad != kPadNone ? (padded + 15) >> 4 : 0;
    const int ncol = nfast + nmir;
    const int per_band = ncol * groups;
    const FastDiv by_band(per_band), by_col(ncol), by_cell(b);
    // Short bands, whole and inside the frame: eight rows an item, counted a
    // cell at a time.  What is left of the unit goes strip by strip.
    const int Q = vec && (b == 2 || b == 4) ? 8 / b : 0;
    const int whole = Q ? real >> 4 : 0, nbq = Q ? max(0, min(nb, H / b - r0)) / Q : 0;
    const FastDiv by_whole(whole);
    for (int item = tid; item < nbq * whole; item += NT) {
        const int jq = by_whole(item), st = item - jq * whole;
        const uint8_t* col = mask + (int64_t)(r0 + jq * Q) * b * W + X0 + 16 * st;
        v4u w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            w[i] = ld16_nt(col + (int64_t)i * W);
        uint32_t* cc = cellcnt + jq * Q * KCs;
        if (b == 4)
            count_bands<4>(w, cc + 4 * st, KCs);
        else
            count_bands<2>(w, cc + 8 * st, KCs);
    }
    if (nbq * Q == nb && whole == ncol)
        return;
    auto strips = [&](auto quads) {
        for (int item = tid; item < nb * per_band; item += NT) {
            const int j = by_band(item);
            const int rem = item - j * per_band;
            const int g = by_col(rem);
            const int st = rem - g * ncol;
            if (j < nbq * Q && st < whole)
                continue;
            const bool mir = st >= nfast;
            // first column of the strip, and the columns [va, vb) it counts
            const int va = mir ? ms + 16 * (st - nfast) : (int)X0 + 16 * st;
            const int vb = min(va + 16, mir ? me : (int)lim);
            const int64_t p0 = min(va, mir ? W - 16 : (int)lim - 16);
            const int row0 = (r0 + j) * b;
            const int k0 = g * RI, k1 = min(b, k0 + RI);
            uint32_t e[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};   // quads: e only, 128 a hit
            if (row0 + k1 <= H) {
                // rows inside the frame: no folding
                const uint8_t* col = mask + (int64_t)row0 * W + p0;
                int k = k0;
                for (; k + kPlanBatch <= k1; k += kPlanBatch) {
                    v4u w[kPlanBatch];
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i)
                        w[i] = ld16_nt(col + (int64_t)(k + i) * W);
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i)
                        count_strip<quads>(w[i], e, o);
                }
                if (k < k1) {
                    // the last partial batch (b not a multiple of the batch)
                    v4u w[kPlanBatch];
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i)
                        w[i] = k + i < k1 ? ld16_nt(col + (int64_t)(k + i) * W) : v4u{0u, 0u, 0u, 0u};
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i)
                        count_strip<quads>(w[i], e, o);
                }
            } else {
                // bottom border: mirrored rows (absent without padding), still
                // issued a batch at a time so that their latencies overlap
                for (int k = k0; k < k1; k += kPlanBatch) {
                    v4u w[kPlanBatch];
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i) {
                        const int r = row0 + k + i;
                        w[i] = (k + i < k1 && (r < H || pad != kPadNone))
                                   ? ld16_nt(mask + (int64_t)fold(r, H, pad) * W + p0)
                                   : v4u{0u, 0u, 0u, 0u};
                    }
#pragma unroll
                    for (int i = 0; i < kPlanBatch; ++i)
                        count_strip<quads>(w[i], e, o);
                }
            }
            if constexpr (quads) {
                // four neighbouring columns lie in one cell
                if ((b & 15) == 0) {
                    const uint32_t cnt = ((e[0] + e[1]) + (e[2] + e[3])) >> 7;
                    if (cnt != 0u)
                        atomicAdd(cellcnt + j * KCs + by_cell(16 * st), cnt);
                } else {
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        if (e[d] != 0u)
                            atomicAdd(cellcnt + j * KCs + by_cell(16 * st + 4 * d), e[d] >> 7);
                }
                continue;
            }
            if (vb - va < 16 || va != p0)
                mask_cols(e, o, va - (int)p0, vb - (int)p0);
            if (mir) {
                const uint32_t t = (e[0] + e[1] + e[2] + e[3]) + (o[0] + o[1] + o[2] + o[3]);
                const uint32_t cnt = (t & 0xFFFFu) + (t >> 16);
                if (cnt != 0u)
                    atomicAdd(cellcnt + j * KCs + KC - 1, cnt);
            } else if (va != p0) {
                spread_strip(e, o, cellcnt + j * KCs, KC, b, (int)(p0 - X0));
            } else if ((b & 15) == 0) {
                // b a multiple of 16: the strip lies in one cell, one counter
                // update (a 16-bit half sums at most 8 columns of 16 rows)
                const uint32_t t = (e[0] + e[1] + e[2] + e[3]) + (o[0] + o[1] + o[2] + o[3]);
                const uint32_t cnt = (t & 0xFFFFu) + (t >> 16);
                const int cell = by_cell(16 * st);
                if (cnt != 0u && cell < KC)
                    atomicAdd(cellcnt + j * KCs + cell, cnt);
            } else {
                spread_strip(e, o, cellcnt + j * KCs, KC, b, 16 * st);
            }
        }
    };
    if (vec && (b & 3) == 0 && (real & 15) == 0 && nmir == 0)
        strips(std::true_type());
    else
        strips(std::false_type());
    if (!vec) {
        for (int item = tid; item < nb * WB; item += NT) {
            const int j = item / WB, p = item - j * WB;
            const int x = (int)X0 + p;
            const int row0 = (r0 + j) * b;
            const int rows = pad == kPadNone ? (x < W ? min(b, H - row0) : 0) : b;
            const g_u8* src = (const g_u8*)(mask + (pad == kPadNone ? x : fold(x, W, pad)));
            uint32_t cnt = 0u;
            for (int k = 0; k < rows; ++k)
                cnt += src[(int64_t)fold(row0 + k, H, pad) * W] != 0;
            if (cnt != 0u)
                atomicAdd(cellcnt + j * KCs + p / b, cnt);
        }
    }
}

// One plan unit: its cell counters cleared, counted by `count(F, f, r0, nb, c0,
// KC, KCs, cellcnt)`, then every cell flagged (count >= tau) and the complex
// cells of every tile counted.
template <typename Count>
__device__ __forceinline__ void plan_unit(const TileArgs& a, uint8_t* lds, Count count)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int f = (int)uniform_u32((uint32_t)a.unit_map[2 * (int64_t)blockIdx.x]);
    const int lu = (int)uniform_u32((uint32_t)a.unit_map[2 * (int64_t)blockIdx.x + 1]);
    const FrameRec F = a.frames[f];
    const int chunks = (F.TX + F.ctx - 1) / F.ctx;
    const int band_grp = lu / chunks;
    const int r0 = band_grp * F.cnb;
    const int nb = min(F.cnb, F.GR - r0);
    const int t0 = (lu - band_grp * chunks) * F.ctx;
    const int nt = min(F.ctx, F.TX - t0);
    const int c0 = t0 * F.K;
    const int KC = min(nt * F.K, F.GC - c0);
    const int KCs = F.ctx * F.K;
    uint32_t* cellcnt = reinterpret_cast<uint32_t*>(lds);
    uint32_t* tcnt = cellcnt + F.cnb * KCs;
    for (int i = tid; i < F.cnb * (KCs + F.ctx); i += NT)
        cellcnt[i] = 0u;
    // the store's ticket words start at zero for the scan and later launches
    // of this call sequence (stream order: no earlier launch still uses them)
    if (blockIdx.x == 0 && tid < kTicketWords)
        a.ticket[tid] = 0u;
    lds_barrier();
    count(F, f, r0, nb, c0, KC, KCs, cellcnt);
    lds_barrier();
    const FastDiv by_kc(KC), by_k(F.K), by_nt(nt);
    for (int i = tid; i < nb * KC; i += NT) {
        const int j = by_kc(i), kc = i - j * KC;
        // tau = 0 (unpadded mode only): majority of the cell's real pixels
        const uint32_t tau = F.tau > 0 ? (uint32_t)F.tau
                                       : ((uint32_t)stat_area(F, (r0 + j) * F.b, (c0 + kc) * F.b, F.b) + 1u) / 2u;
        const uint8_t fl = (uint8_t)(cellcnt[j * KCs + kc] >= tau);
        a.flags[F.cell_base + (int64_t)(r0 + j) * F.GC + c0 + kc] = fl;
        if (fl)
            atomicAdd(&tcnt[j * F.ctx + by_k(kc)], 1u);
    }
    lds_barrier();
    for (int i = tid; i < nb * nt; i += NT) {
        const int j = by_nt(i), ti = i - j * nt;
        a.tile_cnt[F.tile_base + (int64_t)(r0 + j) * F.TX + t0 + ti] = tcnt[j * F.ctx + ti];
    }
}

// Five waves per SIMD (96 VGPRs): the loads of more items in flight.
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_plan(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    plan_unit(a, lds, [&](const FrameRec& F, int f, int r0, int nb, int c0, int KC, int KCs, uint32_t* cellcnt) {
        const uint8_t* mask = a.masks ? a.masks[f] : nullptr;
        if (mask != nullptr)
            plan_count(a, F, mask, r0, nb, c0, KC, KCs, cellcnt);
    });
}

// --------------------------------------------------------------------------
// Plan from complexity labels (Sec. VI-A names an edge detector such as the
// Sobel operator as a source of the region mask), in the same pass: a cell's
// count is the number of edge pixels among its b x b mirror-padded
// positions, each position taking the label of the real pixel it folds onto
// (the label dp_pix_edge_mask writes).  No mask is written or read.  The 3x3
// stencil evaluated on the padded grid of channel sums, every coordinate
// folded as the label's border rule folds it (edge_fold), gives exactly the
// label of the folded pixel: a mirror maps the pair of neighbours of a padded
// position onto the pair of neighbours of its image, at most swapped, and a
// swap only flips the sign of Gy.  So each chunk of padded rows and columns is
// staged as channel sums in LDS (one halo row and column on every side) and
// counted without knowing which positions are real.
//
// The walk (label_walk) is shared with the mask kernel: up to kLabCols columns
// times any number of rows.  A lane takes four columns and walks down the
// rows with the stencil's last two rows in registers, so no row is staged
// twice; rows come in blocks of kLabBlock, each block's 16-pixel vectors
// loaded while the block before is labelled (two LDS buffers, one barrier a
// block).  What bounds it is HBM and the vector instructions of the staging
// together: without the stencil's sums it takes as long, without the loads 98
// of 130 us (plan, 64 x 1080p) and 63 of 133 (masks).  The loads are cached
// ones: a lane's C vectors share their lines with its neighbours' (masks, 64 x
// 1080p RGB: streaming loads 132 us, cached 106).
// 16 x 1080p RGB: plan 62.5 -> 33.5 us, masks 53 -> 24.5 us; 64 x 1080p: 145 ->
// 96 us and 153 -> 95 us; 24 photos of odd widths: 217 -> 31 us and 83 -> 24.5
// us (before: chunks of 16 rows x 512 columns staged whole, two columns a
// lane, no load in flight while a chunk was labelled, and frames off the
// 16-byte grid staged pixel by pixel).
// --------------------------------------------------------------------------
// Channel sums of 16 consecutive pixels from their 16 C bytes, as eight
// dwords of two 16-bit sums each (pixel 2k low, 2k + 1 high).
template <int C>
__device__ __forceinline__ void pixel_sums16(const v4u (&w)[C], v4u& lo, v4u& hi)
{
    uint32_t d[4 * C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        d[4 * i + 0] = w[i].x;
        d[4 * i + 1] = w[i].y;
        d[4 * i + 2] = w[i].z;
        d[4 * i + 3] = w[i].w;
    }
    uint32_t pr[8];   // pixel pairs (2k low, 2k + 1 high)
    if constexpr (C == 1) {
        // each byte is its own sum: bytes 0, 1 and 2, 3 of a dword into halves
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pr[2 * i] = __builtin_amdgcn_perm(0u, d[i], 0x0C010C00u);
            pr[2 * i + 1] = __builtin_amdgcn_perm(0u, d[i], 0x0C030C02u);
        }
    } else if constexpr (C == 2) {
        // a dword is two pixels: (b0 + b1, b2 + b3) as halves
#pragma unroll
        for (int i = 0; i < 8; ++i)
            pr[i] = __builtin_amdgcn_perm(0u, d[i], 0x0C020C00u) + __builtin_amdgcn_perm(0u, d[i], 0x0C030C01u);
    } else if constexpr (C == 3) {
        // three dwords are four pixels: bytes 0-2 | 3-5 | 6-8 | 9-11, each
        // pixel's bytes added by byte dot products with 0/1 weights
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t a = d[3 * i], b = d[3 * i + 1], c = d[3 * i + 2];
            const uint32_t s0 = __builtin_amdgcn_udot4(a, 0x00010101u, 0u, false);
            const uint32_t s1 = __builtin_amdgcn_udot4(b, 0x00000101u, __builtin_amdgcn_udot4(a, 0x01000000u, 0u, false), false);
            const uint32_t s2 = __builtin_amdgcn_udot4(c, 0x00000001u, __builtin_amdgcn_udot4(b, 0x01010000u, 0u, false), false);
            const uint32_t s3 = __builtin_amdgcn_udot4(c, 0x01010100u, 0u, false);
            pr[2 * i] = s0 | (s1 << 16);
            pr[2 * i + 1] = s2 | (s3 << 16);
        }
    } else {
        // a dword is one pixel
#pragma unroll
        for (int i = 0; i < 8; ++i)
            pr[i] = __builtin_amdgcn_udot4(d[2 * i], 0x01010101u, 0u, false) |
                    (__builtin_amdgcn_udot4(d[2 * i + 1], 0x01010101u, 0u, false) << 16);
    }
    lo = v4u{pr[0], pr[1], pr[2], pr[3]};
    hi = v4u{pr[4], pr[5], pr[6], pr[7]};
}

// A lane's group and its sums into the staged row S: from the vectors of its
// source pixels, or, pixel by pixel, from the row itself.
template <int C>
struct LabStage : LabPlace {
    __device__ __forceinline__ void store(const v4u (&w)[C], const uint8_t* row, uint16_t* S, int px0, int W,
                                          int pad) const
    {
        if (kind == kLabSingle) {
            for (int c = pa; c < pb; ++c) {
                const g_u8* p = (const g_u8*)(row + (int64_t)edge_fold(c, W, pad) * C);
                uint32_t sum = 0u;
#pragma unroll
                for (int ch = 0; ch < C; ++ch)
                    sum += p[ch];
                S[kLabLeft + c - px0] = (uint16_t)sum;
            }
            return;
        }
        v4u lo, hi;
        pixel_sums16<C>(w, lo, hi);
        put(lo, hi, S, px0, W, pad);
    }
};

// The stencil, two neighbouring columns in the 16-bit halves of one register:
// Gx = dx(-1) + 2 dx(0) + dx(+1), Gy = sx(+1) - sx(-1), with
// dx(r) = S[r][+1] - S[r][-1], sx(r) = S[r][-1] + 2 S[r][0] + S[r][+1].
// With S <= 4 * 255 every intermediate fits a signed 16-bit half exactly
// (|Gx|, |Gy| <= 4080), and so does thr - 1 - (|Gx| + |Gy|) for thr <= 16384:
// its sign is the label.
typedef short s16x2 __attribute__((ext_vector_type(2)));

// 2 a + b in both halves.
__device__ __forceinline__ s16x2 twice_plus(s16x2 a, s16x2 b)
{
    s16x2 d;
    asm("v_pk_mad_u16 %0, %1, 2, %2 op_sel_hi:[1,0,1]" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

struct SobelRow {
    s16x2 dx[2], sx[2];   // of the columns 0, 1 and 2, 3 of a lane

    // w: the dword before the lane's two dwords of the row, they, and the one after.
    __device__ __forceinline__ void set(const uint32_t* w)
    {
        const s16x2 l = __builtin_bit_cast(s16x2, __builtin_amdgcn_alignbit(w[1], w[0], 16));   // S[-1], S[0]
        const s16x2 m = __builtin_bit_cast(s16x2, __builtin_amdgcn_alignbit(w[2], w[1], 16));   // S[1], S[2]
        const s16x2 r = __builtin_bit_cast(s16x2, __builtin_amdgcn_alignbit(w[3], w[2], 16));   // S[3], S[4]
        const s16x2 a = __builtin_bit_cast(s16x2, w[1]), b = __builtin_bit_cast(s16x2, w[2]);
        dx[0] = m - l;
        dx[1] = r - m;
        sx[0] = twice_plus(a, l + m);
        sx[1] = twice_plus(b, m + r);
    }
};

// Labels of the lane's four columns in the row between a and c, as 0 / 1 bytes.
__device__ __forceinline__ uint32_t sobel_labels(const SobelRow& a, const SobelRow& b, const SobelRow& c, int thr)
{
    const s16x2 t = {(short)(thr - 1), (short)(thr - 1)};
    uint32_t d[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const s16x2 gx = twice_plus(b.dx[h], a.dx[h] + c.dx[h]), gy = c.sx[h] - a.sx[h];
        d[h] = __builtin_bit_cast(uint32_t, t - (__builtin_elementwise_abs(gx) + __builtin_elementwise_abs(gy)));
    }
    // selectors 8 .. 11: the signs of the four halves, as whole bytes
    return __builtin_amdgcn_perm(d[1], d[0], 0x0B0A0908u) & 0x01010101u;
}

// Walk down `rows` padded rows from py0 over the padded columns [px0, px0 +
// cols): for each block emit(y0, ya, yb, lab), lab[j] = the labels of row y0 + j
// (rows ya <= y0 + j < yb only) in columns px0 + 4 lane .. + 3, as bytes
// (columns past the end hold anything), rows in order.  Every lane of the
// workgroup calls it; it has a lane per four columns and per staged group of
// a block (label_threads), and S holds two blocks of `stride` columns a row.
template <int C, typename Emit>
__device__ __forceinline__ void label_walk(const uint8_t* img, int64_t pitch, int H, int W, int pad, int py0, int rows,
                                           int px0, int cols, int thr, uint16_t* S, int stride, Emit emit)
{
    const int tid = threadIdx.x;
    const int G = label_groups(cols);
    const int srow = tid / G;
    const int nst = rows + 2, nblk = (nst + kLabBlock - 1) / kLabBlock;
    LabStage<C> st;
    st.setup(tid - srow * G, px0, cols, W, pad);
    const bool stages = srow < kLabBlock && st.kind != kLabNone;
    v4u w[C];
    // rows that lie in the frame one after another need no folding
    const bool plain = py0 >= 1 && py0 - 1 + nst <= H;
    auto row_of = [&](int blk) { return img + (int64_t)edge_fold(py0 - 1 + blk * kLabBlock + srow, H, pad) * pitch; };
    const uint8_t* next = plain ? row_of(0) + (int64_t)st.from * C : nullptr;
    auto load = [&](int blk) {
        if (stages && st.vector() && blk * kLabBlock + srow < nst) {
            const uint8_t* p = plain ? next : row_of(blk) + (int64_t)st.from * C;
#pragma unroll
            for (int i = 0; i < C; ++i)
                w[i] = ld16(p + 16 * i);
        }
        next += kLabBlock * pitch;
    };
    auto store = [&](int blk) {
        if (stages && blk * kLabBlock + srow < nst)
            st.store(w, st.kind == kLabSingle ? row_of(blk) : nullptr,
                     S + ((blk & 1) * kLabBlock + srow) * stride, px0, W, pad);
    };
    SobelRow a, b;
    uint32_t lab[kLabBlock];
    // A block's labels go out after the next block's barrier, before its
    // loads: what waits for those loads then waits for no newer store.
    auto give = [&](int blk) {
        const int y0 = blk * kLabBlock - 2;          // the row whose labels the block's first staged row completed
        if (4 * tid < cols)
            emit(y0, max(y0, 0), min(y0 + kLabBlock, rows), lab);
    };
    load(0);
    for (int blk = 0; blk < nblk; ++blk) {
        store(blk);
        lds_barrier();
        if (blk > 0)
            give(blk - 1);
        if (blk + 1 < nblk)
            load(blk + 1);
        const uint32_t* r0 = reinterpret_cast<const uint32_t*>(S + (blk & 1) * kLabBlock * stride + kLabLeft) +
                             2 * min(tid, cols >> 2) - 1;
        uint32_t q[kLabBlock][4];   // (rows past the last hold anything)
#pragma unroll
        for (int j = 0; j < kLabBlock; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                q[j][i] = r0[j * (stride / 2) + i];
#pragma unroll
        for (int j = 0; j < kLabBlock; ++j) {
            SobelRow c;
            c.set(q[j]);
            lab[j] = sobel_labels(a, b, c, thr);
            a = b;
            b = c;
        }
    }
    give(nblk - 1);
    lds_barrier();
}

// A unit is one tile's columns x F.lnb bands: counted in walks of at most
// kLabCols columns, a lane's four byte counters added to the cells' at the
// end of every band (and after 128 rows of one, before a byte could overflow).
template <int C>
__global__ __launch_bounds__(256) void k_plan_labels(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x, NT = blockDim.x;
    const int64_t unit = a.sched_offset + blockIdx.x;
    const UnitCoord u = unit_of(a, unit);
    const int f = u.f, local = u.local;
    const FrameRec& F = a.frames[f];
    const int b = F.b, K = F.K, W = F.W, pad = F.pad;
    const int r0 = (local / F.TX) * F.lnb, ct = local % F.TX;
    const int nb = min(F.lnb, F.GR - r0), c0 = ct * K, KC = min(K, F.GC - c0);
    const int stride = label_stride(4 * NT);
    uint16_t* S = reinterpret_cast<uint16_t*>(lds);
    uint32_t* cellcnt = reinterpret_cast<uint32_t*>(lds + 4 * kLabBlock * stride);   // [nb][K]
    uint32_t* tcnt = cellcnt + F.lnb * K;                                            // [nb]
    for (int i = tid; i < F.lnb * (K + 1); i += NT)
        cellcnt[i] = 0u;
    // the store's ticket words start at zero for the scan and later launches
    // of this call sequence (stream order: no earlier launch still uses them)
    if (blockIdx.x == 0 && tid < kTicketWords)
        a.ticket[tid] = 0u;
    lds_barrier();
    const int X0 = c0 * b, XW = KC * b;
    // unpadded mode: rows and columns past the frame are absent
    const int rows = pad == kPadNone ? min(nb * b, F.H - r0 * b) : nb * b;
    const int xend = pad == kPadNone ? min(XW, W - X0) : XW;
    for (int cx = 0; cx < xend; cx += kLabCols) {
        const int cols = min(kLabCols, xend - cx);
        const int x = cx + 4 * tid, n = min(4, cols - 4 * tid);
        uint32_t cnt = 0u;
        int j = 0, left = b, batch = min(b, 128);
        label_walk<C>(static_cast<const uint8_t*>(a.images[f]), F.pitch, F.H, W, pad, r0 * b, rows, X0 + cx, cols,
                      a.edge_threshold * C, S, stride, [&](int y0, int ya, int yb, const uint32_t (&lab)[kLabBlock]) {
#pragma unroll 1
            while (ya < yb) {
                // up to the end of the band, or of a batch of its rows
                const int stop = min(yb, ya + batch);
#pragma unroll
                for (int i = 0; i < kLabBlock; ++i)
                    cnt += (y0 + i >= ya && y0 + i < stop) ? lab[i] : 0u;
                batch -= stop - ya;
                ya = stop;
                if (batch != 0 && ya < rows)
                    break;
                uint32_t* cc = cellcnt + j * K;
                if ((b & 3) == 0) {
                    // the four columns lie in one cell (walks start on multiples of 4)
                    const uint32_t sum = __builtin_amdgcn_udot4(cnt, 0x01010101u >> (8 * (4 - n)), 0u, false);
                    if (sum != 0u)
                        atomicAdd(cc + x / b, sum);
                } else {
                    for (int q = 0; q < n; ++q)
                        if (((cnt >> (8 * q)) & 0xFFu) != 0u)
                            atomicAdd(cc + (x + q) / b, (cnt >> (8 * q)) & 0xFFu);
                }
                cnt = 0u;
                left -= min(b, 128);
                if (left <= 0) {
                    left = b;
                    ++j;
                }
                batch = min(left, 128);
            }
        });
    }
    lds_barrier();
    for (int i = tid; i < nb * KC; i += NT) {
        const int j = i / KC, kc = i - j * KC;
        // tau = 0 (unpadded mode only): majority of the cell's real pixels
        const uint32_t tau = F.tau > 0 ? (uint32_t)F.tau
                                       : ((uint32_t)stat_area(F, (r0 + j) * b, (c0 + kc) * b, b) + 1u) / 2u;
        const uint8_t fl = (uint8_t)(cellcnt[j * K + kc] >= tau);
        a.flags[F.cell_base + (int64_t)(r0 + j) * F.GC + c0 + kc] = fl;
        if (fl)
            atomicAdd(&tcnt[j], 1u);
    }
    lds_barrier();
    for (int j = tid; j < nb; j += NT)
        a.tile_cnt[F.tile_base + (int64_t)(r0 + j) * F.TX + ct] = tcnt[j];
}

// Plan of a call without masks (Algorithm 3 with every cell simple): flags
// cleared, no complex cell in any tile, and each frame's counts and offsets
// copied from the table the host derived from the geometry alone.  One
// launch in place of the count and scan passes.
__global__ __launch_bounds__(256) void k_plan_simple(TileArgs a)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 < kTicketWords)
        a.ticket[i0] = 0u;
    for (int64_t i = i0; i < a.total_cells; i += stride)
        a.flags[i] = 0;
    for (int64_t i = i0; i < a.n_tiles; i += stride) {
        a.tile_cnt[i] = 0u;
        a.tile_fg[i] = 0u;
    }
    for (int64_t i = i0; i < 4 * (int64_t)a.n_frames; i += stride)
        a.counts[i] = a.simple_counts[i];
}

// Exclusive scan of a frame's per-tile complex counts into each tile's count of
// complex cells before it; returns the frame's total.  The rounds are a chain of
// a load, a scan and two barriers, about 0.8 us each: where one tile a lane would
// take several, a lane takes eight consecutive ones (8 x 1080p, b 2, 1620 tiles a
// frame: plan 19.4 -> 16.2 us; 16 x 1080p, b 4, 810: 15.3 -> 13.6; 24 frames of four
// sizes, up to 2250: 49.9 -> 45.8, k_scan_tiles 9.1 -> 5.5 of it).
template <int TILES>
__device__ __forceinline__ uint32_t scan_tiles_n(const TileArgs& a, int64_t t0, int64_t nt, uint32_t* wave_tot)
{
    const auto* cnt = (const __attribute__((address_space(1))) uint32_t*)(a.tile_cnt + t0);
    auto* fg = (__attribute__((address_space(1))) uint32_t*)(a.tile_fg + t0);
    uint32_t carry = 0;
    for (int64_t base = 0; base < nt; base += TILES * (int64_t)blockDim.x) {
        const int64_t i = base + TILES * (int64_t)threadIdx.x;
        uint32_t v[TILES], sum = 0;
#pragma unroll
        for (int k = 0; k < TILES; ++k)
            v[k] = i + k < nt ? cnt[i + k] : 0u;
#pragma unroll
        for (int k = 0; k < TILES; ++k)
            sum += v[k];
        uint32_t tot;
        uint32_t run = carry + block_exclusive_scan<uint32_t>(sum, wave_tot, tot);
#pragma unroll
        for (int k = 0; k < TILES; ++k) {
            if (i + k < nt)
                fg[i + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    return carry;
}

__device__ __forceinline__ uint32_t scan_frame_tiles(const TileArgs& a, int64_t t0, int64_t nt, uint32_t* wave_tot)
{
    return nt <= blockDim.x ? scan_tiles_n<1>(a, t0, nt, wave_tot) : scan_tiles_n<8>(a, t0, nt, wave_tot);
}

// One workgroup per frame: the tile prefixes and the frame's simple and complex
// cell counts; k_scan_frames, launched next, turns the per-frame counts into
// store offsets.  (Electing a last workgroup here instead needs an agent-scope
// release in every workgroup, an L2 write-back on gfx950: the plan call of the
// 256-frame batch took 3 us longer that way.)
__global__ __launch_bounds__(256) void k_scan_tiles(TileArgs a)
{
    __shared__ uint32_t wave_tot[9];
    const int f = blockIdx.x;
    const FrameRec F = a.frames[f];
    const uint32_t total = scan_frame_tiles(a, F.tile_base, (int64_t)F.GR * F.TX, wave_tot);
    if (threadIdx.x == 0) {
        const uint64_t cells = (uint64_t)F.GR * F.GC;
        a.counts[4 * f + 0] = cells - total;
        a.counts[4 * f + 1] = (uint64_t)total;
    }
}

__global__ __launch_bounds__(256) void k_scan_frames(TileArgs a)
{
    __shared__ uint64_t wave_tot64[9];
    scan_frames(a, wave_tot64);
}

// The scan without a hand-off between workgroups, for batches whose frames
// share C and n (a frame's store size is then a fixed weight times its
// counts) and whose tile counts are few: frames are concatenated, so the
// complex cells of every earlier frame are one prefix of the tile array,
// which workgroup f adds up itself before scanning its own tiles.
__global__ __launch_bounds__(256) void k_scan_prefix(TileArgs a)
{
    __shared__ uint32_t wave_tot[9];
    const int f = blockIdx.x, tid = threadIdx.x, NT = blockDim.x;
    const FrameRec F = a.frames[f];
    const int64_t t0 = F.tile_base;
    // tile counts of the earlier frames: 16 bytes a load, all in flight
    const int64_t n4 = t0 >> 2;
    const v4u* c4 = reinterpret_cast<const v4u*>(a.tile_cnt);
    uint32_t part = tid < (int)(t0 & 3) ? a.tile_cnt[4 * n4 + tid] : 0u;
    for (int64_t base = 0; base < n4; base += 8 * (int64_t)NT) {
        v4u w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = base + (int64_t)k * NT + tid;
            w[k] = i < n4 ? c4[i] : v4u{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            part += (w[k].x + w[k].y) + (w[k].z + w[k].w);
    }
    uint32_t before;
    block_exclusive_scan<uint32_t>(part, wave_tot, before);
    const uint32_t total = scan_frame_tiles(a, t0, (int64_t)F.GR * F.TX, wave_tot);
    if (tid == 0) {
        const uint64_t nf = total, nb = (uint64_t)F.GR * (uint64_t)F.GC - nf;
        const uint64_t bb = (uint64_t)F.C * ((uint64_t)F.cell_base - before);
        const uint64_t fb = (uint64_t)F.n * (uint64_t)F.n * (uint64_t)F.C * (uint64_t)before;
        a.counts[4 * f + 0] = nb;
        a.counts[4 * f + 1] = nf;
        a.counts[4 * f + 2] = bb;
        a.counts[4 * f + 3] = fb;
    }
    if (f == 0 && tid < kTicketWords)
        a.ticket[tid] = 0;
}

// Complex cells per tile from the store's flags alone (a store that was
// written elsewhere, e.g. decoded from its serialised form), one lane per
// tile; the scan then rebuilds the tile prefixes and the frame counts and
// offsets.  Workgroup 0 clears the ticket words as k_plan does.
__global__ __launch_bounds__(256) void k_tile_count(TileArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < kTicketWords)
        a.ticket[threadIdx.x] = 0u;
    if (i >= a.n_tiles)
        return;
    const int f = a.tile_map[2 * i];
    const int64_t local = a.tile_map[2 * i + 1];
    const FrameRec F = a.frames[f];
    const int r = (int)(local / F.TX), ct = (int)(local - (int64_t)r * F.TX);
    const int x0c = ct * F.K, Kt = min(F.K, F.GC - x0c);
    const uint8_t* fl = a.flags + F.cell_base + (int64_t)r * F.GC + x0c;
    uint32_t cnt = 0;
    for (int k = 0; k < Kt; ++k)
        cnt += fl[k] != 0;
    a.tile_cnt[F.tile_base + local] = cnt;
}

// Subgrid rows per phase-1 item: with short subgrid rows an item takes
// several, so that every lane has about eight row loads in flight.
__device__ __forceinline__ int rows_per_item(int s) { return s == 2 ? 4 : ((s == 3 || s == 4) ? 2 : 1); }

// Column sums of up to 8 / S consecutive subgrid rows of S rows each (qq of
// them), one 16-byte strip: every load is issued before the first add.
template <int S>
__device__ __forceinline__ void strip_rows_q(const uint8_t* base, uint32_t off, uint32_t upitch, int qq,
                                             uint16_t* dst, int rowbuf)
{
    constexpr int Q = 8 / S;
    uint32_t e[Q][4], o[Q][4];
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
        for (int d = 0; d < 4; ++d)
            e[j][d] = o[j][d] = 0u;
    v4u w[Q * S];
    if (qq == Q) {
        // every row of the item (the common case): no per-load guards
#pragma unroll
        for (int i = 0; i < Q * S; ++i)
            w[i] = ld16_nt(base + (off + (uint32_t)i * upitch));
#pragma unroll
        for (int i = 0; i < Q * S; ++i)
            acc_bytes(w[i], e[i / S], o[i / S]);
#pragma unroll
        for (int j = 0; j < Q; ++j)
            store_colsums16(dst + j * rowbuf, e[j], o[j]);
        return;
    }
#pragma unroll
    for (int i = 0; i < Q * S; ++i)
        if (i < qq * S)
            w[i] = ld16_nt(base + (off + (uint32_t)i * upitch));
#pragma unroll
    for (int i = 0; i < Q * S; ++i)
        if (i < qq * S)
            acc_bytes(w[i], e[i / S], o[i / S]);
#pragma unroll
    for (int j = 0; j < Q; ++j)
        if (j < qq)
            store_colsums16(dst + j * rowbuf, e[j], o[j]);
}

// Column sums of one subgrid row of s padded rows from row0 on, folded into
// the frame (last band), one strip; loads in batches of 4.
__device__ __forceinline__ void strip_rows_fold(const uint8_t* col, int64_t pitch, int row0, int s, int H, int pad,
                                                uint16_t* dst)
{
    uint32_t e[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};
    if (pad == kPadNone)   // rows past the frame are absent
        s = max(0, min(s, H - row0));
    int k = 0;
    for (; k + 4 <= s; k += 4) {
        v4u w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = ld16_nt(col + (int64_t)fold(row0 + k + i, H, pad) * pitch);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc_bytes(w[i], e, o);
    }
    for (; k < s; ++k)
        acc_bytes(ld16_nt(col + (int64_t)fold(row0 + k, H, pad) * pitch), e, o);
    store_colsums16(dst, e, o);
}

// Column sums of one subgrid row of s rows, one strip, loads in batches of 8.
__device__ __forceinline__ void strip_rows_1(const uint8_t* base, uint32_t off, uint32_t upitch, int s, uint16_t* dst)
{
    uint32_t e[4] = {0, 0, 0, 0}, o[4] = {0, 0, 0, 0};
    int k = 0;
    for (; k + 8 <= s; k += 8) {
        v4u w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            w[i] = ld16_nt(base + (off + (uint32_t)(k + i) * upitch));
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc_bytes(w[i], e, o);
    }
    for (; k + 4 <= s; k += 4) {
        v4u w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = ld16_nt(base + (off + (uint32_t)(k + i) * upitch));
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc_bytes(w[i], e, o);
    }
    for (; k < s; ++k)
        acc_bytes(ld16_nt(base + (off + (uint32_t)k * upitch)), e, o);
    store_colsums16(dst, e, o);
}

// The C bytes at p (any byte of LDS) as the low bytes of a dword.
template <int C>
__device__ __forceinline__ uint32_t lds_pixel(const uint8_t* p)
{
    if constexpr (C == 4)
        return *reinterpret_cast<const uint32_t*>(p);
    else if constexpr (C == 3) {
        // two dwords and a byte align (the allocation reaches past the last pixel's)
        const uint32_t sh = (uint32_t)(reinterpret_cast<uintptr_t>(p) & 3);
        const uint32_t* w = reinterpret_cast<const uint32_t*>(p - sh);
        return __builtin_amdgcn_alignbyte(w[1], w[0], sh) & 0x00FFFFFFu;
    } else if constexpr (C == 2)
        return *reinterpret_cast<const uint16_t*>(p);
    else
        return *p;
}

// One padded row of a band's rounded values, expanded in LDS for the row
// stores: subcell column fc (cell fc / n) covers s_b pixels of C bytes from
// byte fc * s_b * C.  Where that span is whole dwords, a lane writes one
// subcell's: the pixel's C-byte pattern, a dword at a time (for C = 3 it repeats
// every three dwords).  Else a lane writes four pixels, C dwords: the values of
// the up to four subcells they lie in.  Either way no two lanes write into
// the same dword.  (16 x 1080p RGB, b 4 / s_b 2: forward 121 -> 114 us, b 2 /
// s_b 1, 8 frames: 204 -> 185; before, a lane per subcell and channel wrote
// single bytes there.)  The row buffer holds whole 16-byte strips.
template <int C>
__device__ __forceinline__ void expand_row_u8(uint8_t* exb, int kn, int n, int s, int fr, const uint8_t* cflag,
                                              const uint8_t* vgs, const uint8_t* vgc)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const FastDiv by_n(n);
    const uint8_t* row = vgc + fr * kn * C;
    if (((s * C) & 3) == 0) {
        const int words = (s * C) >> 2;
        for (int fc = tid; fc < kn; fc += NT) {
            const int kc = by_n(fc);
            const uint32_t pix = lds_pixel<C>(cflag[kc] ? row + fc * C : vgs + kc * C);
            uint32_t* d = reinterpret_cast<uint32_t*>(exb + fc * s * C);
            if (C == 3) {
                const uint32_t d0 = pix | (pix << 24), d1 = (pix >> 8) | (pix << 16), d2 = (pix >> 16) | (pix << 8);
                for (int k = 0; k < words; k += 3) {
                    d[k] = d0;
                    d[k + 1] = d1;
                    d[k + 2] = d2;
                }
            } else {
                const uint32_t w = C == 1 ? pix * 0x01010101u : (C == 2 ? pix | (pix << 16) : pix);
                for (int k = 0; k < words; ++k)
                    d[k] = w;
            }
        }
        return;
    }
    const FastDiv by_s(s);
    const int dwords = ((kn * s * C + 15) >> 4) << 2;     // of the row's strips
    for (int g = tid; 4 * g < kn * s; g += NT) {
        int fc = by_s(4 * g), in = 4 * g - fc * s, kc = by_n(fc), jj = fc - kc * n;
        uint32_t pix[4], cur = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((q == 0 || in == 0) && fc < kn)
                cur = lds_pixel<C>(cflag[kc] ? row + fc * C : vgs + kc * C);
            pix[q] = cur;
            if (++in == s) {
                in = 0;
                ++fc;
                if (++jj == n) {
                    jj = 0;
                    ++kc;
                }
            }
        }
        uint32_t w[C];
        if constexpr (C == 1)
            w[0] = pix[0] | (pix[1] << 8) | (pix[2] << 16) | (pix[3] << 24);
        else if constexpr (C == 2) {
            w[0] = pix[0] | (pix[1] << 16);
            w[1] = pix[2] | (pix[3] << 16);
        } else if constexpr (C == 3) {
            w[0] = pix[0] | (pix[1] << 24);
            w[1] = (pix[1] >> 8) | (pix[2] << 16);
            w[2] = (pix[2] >> 16) | (pix[3] << 8);
        } else {
#pragma unroll
            for (int q = 0; q < C; ++q)
                w[q] = pix[q];
        }
        uint32_t* d = reinterpret_cast<uint32_t*>(exb);
#pragma unroll
        for (int k = 0; k < C; ++k)
            if (g * C + k < dwords)
                d[g * C + k] = w[k];
    }
}

// Sums per channel of one subcell's s_b packed 16-bit column sums of one
// subgrid row (s_b pixels of C channels, contiguous in LDS).  For even s_b * C
// the span starts on a dword and is read two columns at a time.
template <int C>
__device__ __forceinline__ void subcell_sums(const uint16_t* cp, int s, uint32_t (&S)[C])
{
#pragma unroll
    for (int ch = 0; ch < C; ++ch)
        S[ch] = 0u;
    if (((s * C) & 1) != 0) {
        for (int x = 0; x < s; ++x)
#pragma unroll
            for (int ch = 0; ch < C; ++ch)
                S[ch] += cp[x * C + ch];
        return;
    }
    const uint32_t* w = reinterpret_cast<const uint32_t*>(cp);
    const int dw = (s * C) >> 1;
    if (C == 3) {
        // two pixels per three dwords: (c0 c1) (c2 c0) (c1 c2)
        for (int k = 0; k < dw; k += 3) {
            const uint32_t w0 = w[k], w1 = w[k + 1], w2 = w[k + 2];
            S[0] += (w0 & 0xFFFFu) + (w1 >> 16);
            S[1 % C] += (w0 >> 16) + (w2 & 0xFFFFu);
            S[2 % C] += (w1 & 0xFFFFu) + (w2 >> 16);
        }
    } else if (C == 1) {
        for (int k = 0; k < dw; ++k)
            S[0] += (w[k] & 0xFFFFu) + (w[k] >> 16);
    } else if (C == 2) {
        for (int k = 0; k < dw; ++k) {
            S[0] += w[k] & 0xFFFFu;
            S[1 % C] += w[k] >> 16;
        }
    } else {
        // C = 4: one pixel per two dwords, (c0 c1) (c2 c3)
        for (int k = 0; k < dw; k += 2) {
            S[0] += w[k] & 0xFFFFu;
            S[1 % C] += w[k] >> 16;
            S[2 % C] += w[k + 1] & 0xFFFFu;
            S[3 % C] += w[k + 1] >> 16;
        }
    }
}

// Phase 2a of the u8 forward for even s_b: one lane per subcell column
// adds, for every subgrid row of the group, the subcell's s_b * C packed
// 16-bit column sums (contiguous in LDS: s_b pixels of C channels) read two
// at a time as dwords, into one sum per channel, and keeps the running sums
// over subgrid rows in cspart[fc * C + ch].  (Per-(column, channel) lanes
// would read each 16-bit sum on its own, C lanes into the same dwords.)
// dbg: optional exact subcell sums, row-major over the fine grid from
// dbg_base (first subgrid row of the group, first subcell column of the
// tile), dbg_row fine cells per row.
template <int C>
__device__ __forceinline__ void subcell_sums_pairs(const uint16_t* col16, int rowbuf, int kn, int s, int ng, int fr0,
                                                   uint32_t* cspart, uint32_t* dbg, int64_t dbg_base, int64_t dbg_row)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    for (int fc = tid; fc < kn; fc += NT) {
        uint32_t tot[C];
#pragma unroll
        for (int ch = 0; ch < C; ++ch)
            tot[ch] = fr0 == 0 ? 0u : cspart[fc * C + ch];
        for (int g = 0; g < ng; ++g) {
            uint32_t S[C];
            subcell_sums<C>(col16 + g * rowbuf + fc * s * C, s, S);
#pragma unroll
            for (int ch = 0; ch < C; ++ch) {
                tot[ch] += S[ch];
                if (dbg)
                    dbg[(dbg_base + (int64_t)g * dbg_row + fc) * C + ch] = S[ch];
            }
        }
#pragma unroll
        for (int ch = 0; ch < C; ++ch)
            cspart[fc * C + ch] = tot[ch];
    }
}

// ==========================================================================
// Forward, uint8 HWC (Algorithm 3 steps 7-19, fused steps 11, 18-21).
// ==========================================================================
// DBG: also write the exact sums of every cell and subcell (dp_pix_debug_sums);
// a separate instantiation, so the release kernel carries none of that state.
template <int C, bool DBG>
__device__ void forward_tile_u8(const TileArgs& a, const FrameRec& F, const TileCoord& tc, uint8_t* lds)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, s = F.s, n = F.n, H = F.H, W = F.W, pad = F.pad;
    const int r = tc.r;
    const int x0c = tc.ct * F.K;
    const int Kt = min(F.K, F.GC - x0c);
    const int WB = Kt * b * C;
    const int nstr = (WB + 15) >> 4;
    const int64_t X0 = (int64_t)x0c * b * C;
    const int64_t tile_end = X0 + WB;
    const int64_t real_end = (int64_t)W * C;
    const int64_t lim = min(tile_end, real_end);
    const int64_t pitch = F.pitch;
    const uint8_t* img = static_cast<const uint8_t*>(a.images[tc.f]);
    uint8_t* out = a.outs ? static_cast<uint8_t*>(a.outs[tc.f]) : nullptr;
    const Strips sp = tile_strips_of(WB, (int)(lim - X0), 16, C, pad);
    // bands without vertical padding address rows by 32-bit offsets from the
    // band's first byte of the tile (uniform base, one offset register)
    const bool band_inside = F.off32 && (r + 1) * b <= H;
    const uint32_t upitch = (uint32_t)pitch;
    const uint8_t* band_in = img + (int64_t)r * b * pitch + X0;

    const LdsPlan L = lds_plan(kFwdU8, F.K, b, n, C);
    uint16_t* col16 = reinterpret_cast<uint16_t*>(lds + L.colsum);
    uint8_t* ex = lds + L.colsum;
    uint32_t* cspart = reinterpret_cast<uint32_t*>(lds + L.cspart);
    uint32_t* cidx = reinterpret_cast<uint32_t*>(lds + L.cidx);
    uint8_t* cflag = lds + L.cflag;
    uint8_t* vgs = lds + L.vgs;
    uint8_t* vgc = lds + L.vgc;
    uint16_t* cxl = reinterpret_cast<uint16_t*>(lds + L.cxl);
    __shared__ uint32_t s_ncx;

    tile_cells(a, F, tc.t, r, x0c, Kt, cidx, cflag, cxl, &s_ncx);
    const uint64_t bg_base = a.counts[4 * tc.f + 2];
    const uint64_t fg_base = a.counts[4 * tc.f + 3];
    const int items = Kt * n * C;
    const int nn = n * n;
    const int rowbuf = 16 * nstr;           // 16-bit column sums of one subgrid row
    const double area_s = (double)s * (double)s, inv_s = exact_inv_area(F, s);

    // ---- subgrid rows, up to kRowGroup at a time: each lane streams its strip
    // down all rows of the group (exact 16-bit column sums per subgrid row,
    // one LDS buffer each), then one lane per (subcell column, channel) adds
    // s_b columns per subgrid row and releases complex subcells ----
    for (int fr0 = 0; fr0 < n; fr0 += kRowGroup) {
        const int ng = min(kRowGroup, n - fr0);
        // Whole-vector strips ([0, nfast)): one item per (q subgrid rows,
        // strip); consecutive lanes read consecutive strips of a row and all
        // q * s_b rows of an item (8 or fewer) are loaded before they are
        // added.
        const int nfast = sp.vec ? sp.nvec : 0;
        const int q = band_inside ? rows_per_item(s) : 1;
        const int ngq = (ng + q - 1) / q;
        const FastDiv by_strip(nfast);
        for (int it = tid; it < nfast * ngq; it += NT) {
            const int gq = by_strip(it);
            const int st = it - gq * nfast;
            const int g0 = gq * q;
            const int qq = min(q, ng - g0);
            const int po = min(16 * st, sp.real - 16);   // the last strip ends with the real columns
            uint16_t* dst = col16 + g0 * rowbuf + po;
            if (!band_inside) {
                // last band: padded rows fold back into the frame
                strip_rows_fold(img + X0 + po, pitch, r * b + (fr0 + g0) * s, s, H, pad, dst);
                continue;
            }
            // rows inside the frame: 32-bit offsets from the band's first row
            const uint32_t off = (uint32_t)((fr0 + g0) * s) * upitch + (uint32_t)po;
            switch (q) {
            case 4: strip_rows_q<2>(band_in, off, upitch, qq, dst, rowbuf); break;
            case 2:
                if (s == 4)
                    strip_rows_q<4>(band_in, off, upitch, qq, dst, rowbuf);
                else
                    strip_rows_q<3>(band_in, off, upitch, qq, dst, rowbuf);
                break;
            default: strip_rows_1(band_in, off, upitch, s, dst); break;
            }
        }
        if (!sp.vec) {
            // a tile too narrow for vectors: one byte column per item
            for (int it = tid; it < ng * WB; it += NT) {
                const int g = it / WB, p = it - g * WB;
                const int x = x0c * b + p / C;
                const int sx = pad == kPadNone ? x : fold(x, W, pad);
                const int row0 = r * b + (fr0 + g) * s;
                const int rows = pad == kPadNone ? (x < W ? max(0, min(s, H - row0)) : 0) : s;
                const g_u8* src = (const g_u8*)(img + (int64_t)sx * C + p % C);
                uint32_t sum = 0u;
                for (int k = 0; k < rows; ++k)
                    sum += src[(int64_t)fold(row0 + k, H, pad) * pitch];
                col16[g * rowbuf + p] = (uint16_t)sum;
            }
        }
        if (sp.vec && sp.real < WB) {
            // padded columns: the sums of the columns they mirror, or nothing
            const int np = WB - sp.real;
            const FastDiv by_np(np);
            if (pad != kPadNone)
                lds_barrier();
            for (int i = tid; i < ng * np; i += NT) {
                const int g = by_np(i), p = sp.real + (i - g * np);
                const int x = p / C, ch = p - x * C;
                col16[g * rowbuf + p] =
                    pad == kPadNone ? (uint16_t)0 : col16[g * rowbuf + mirror_col(x, sp.real / C, pad) * C + ch];
            }
        }
        lds_barrier();
        // running sums of every (subcell column, channel) for the coarse cells
        if ((s & 1) == 0) {
            subcell_sums_pairs<C>(col16, rowbuf, Kt * n, s, ng, fr0, cspart, DBG ? a.dbg_fine : nullptr,
                                  F.fine_base + (int64_t)(r * n + fr0) * ((int64_t)F.GC * n) + (int64_t)x0c * n,
                                  (int64_t)F.GC * n);
        } else {
            for (int j = tid; j < items; j += NT) {
                const int fc = j / C, ch = j - fc * C;
                uint32_t total = fr0 == 0 ? 0u : cspart[j];
                for (int g = 0; g < ng; ++g) {
                    const uint16_t* cp = col16 + g * rowbuf + fc * s * C + ch;
                    uint32_t S = 0;
                    for (int x = 0; x < s; ++x)
                        S += cp[x * C];
                    total += S;
                    if (DBG && a.dbg_fine)
                        a.dbg_fine[(F.fine_base + (int64_t)(r * n + fr0 + g) * ((int64_t)F.GC * n) +
                                    (int64_t)x0c * n + fc) * C + ch] = S;
                }
                cspart[j] = total;
            }
        }
        // releases of the complex cells' subcells, spread evenly over the
        // lanes (only complex cells draw noise, so a lane-per-subcell loop
        // would leave the lanes of simple cells idle): one item per (complex
        // cell, subgrid row, subcell column) re-reads the subcell's column
        // sums and releases its C channels
        const int ncx = (int)s_ncx;
        const int per_cx = ng * n;
        const FastDiv by_cx(per_cx), by_n(n);
        for (int it = tid; it < ncx * per_cx; it += NT) {
            const int q = by_cx(it);
            const int rem = it - q * per_cx;
            const int g = by_n(rem), jj = rem - g * n;
            const int kc = cxl[q];
            const int fc = kc * n + jj, fr = fr0 + g;
            uint32_t S[C];
            subcell_sums<C>(col16 + g * rowbuf + fc * s * C, s, S);
            const uint32_t id = (uint32_t)(r * n + fr) * (uint32_t)(F.GC * n) + (uint32_t)(x0c * n + fc);
            const double area = pad == kPadNone ? stat_area(F, r * b + fr * s, x0c * b + fc * s, s) : area_s;
            const uint64_t at = fg_base + ((uint64_t)cidx[kc] * nn + fr * n + jj) * C;
            uint8_t* vd = vgc + (fr * Kt * n + fc) * C;
            // one channel at a time (unrolled, the C draws would be live at once)
#pragma unroll 1
            for (int ch = 0; ch < C; ++ch) {
                uint32_t Sc = S[0];
#pragma unroll
                for (int k = 1; k < C; ++k)
                    Sc = ch == k ? S[k] : Sc;
                uint8_t pass;
                const float v = release<false>((double)Sc, area, inv_s, F.noise_fg, F.sigma_fg, F, id, ch, 1, pass);
                a.fg[at + ch] = v;
                if (a.clip_fg)
                    a.clip_fg[at + ch] = pass;
                vd[ch] = to_u8(v);
            }
        }
        lds_barrier();
    }

    // ---- simple cells: coarse sum = total of the n*n subcell sums ----
    for (int j = tid; j < Kt * C; j += NT) {
        const int kc = j / C, ch = j - kc * C;
        uint32_t S = 0;
        for (int jj = 0; jj < n; ++jj)
            S += cspart[(kc * n + jj) * C + ch];
        if (DBG && a.dbg_coarse)
            a.dbg_coarse[(F.cell_base + (int64_t)r * F.GC + x0c + kc) * C + ch] = S;
        if (!cflag[kc]) {
            const uint32_t id = (uint32_t)(r * F.GC + x0c + kc);
            uint8_t pass;
            const float v = release<false>((double)S, stat_area(F, r * b, (x0c + kc) * b, b), exact_inv_area(F, b),
                                    F.noise_bg, F.sigma_bg, F, id, ch, 0, pass);
            const uint64_t at = bg_base + (uint64_t)cidx[kc] * C + ch;
            a.bg[at] = v;
            if (a.clip_bg)
                a.clip_bg[at] = pass;
            vgs[kc * C + ch] = to_u8(v);
        }
    }
    if (out == nullptr)
        return;
    lds_barrier();

    // ---- fused reconstruction of the band's real pixels ----
    // The expanded row alternates between two LDS buffers, so one barrier per
    // subgrid row suffices: a buffer is rewritten two rows later, after every
    // lane has passed the barrier that follows its last read.
    const int real = sp.real;
    const FastDiv by_nstr(nstr);
    uint8_t* band_out = out + (int64_t)r * b * pitch + X0;
    for (int fr = 0; fr < n; ++fr) {
        uint8_t* exb = ex + (fr & 1) * (16 * nstr);
        expand_row_u8<C>(exb, Kt * n, n, s, fr, cflag, vgs, vgc);
        lds_barrier();
        const int row0 = r * b + fr * s;
        const int rows = min(s, H - row0);
        // items (row part, strip): the s_b rows of a strip are split over
        // `parts` lanes when the tile has fewer strips than lanes
        const int parts = max(1, min(rows, NT / nstr));
        const int per = (rows + parts - 1) / max(parts, 1);
        for (int it = tid; it < nstr * parts; it += NT) {
            const int part = by_nstr(it);
            const int st = it - part * nstr;
            const int k0 = part * per, k1 = min(rows, k0 + per);
            if (16 * st >= real)
                continue;
            if (real >= 16) {
                // the last strip ends with the real columns (the bytes it
                // shares with its neighbour are written twice, alike)
                const int po = min(16 * st, real - 16);
                const v4u v = lds16(exb + po);
                if (F.off32) {
                    const uint32_t off = (uint32_t)(fr * s) * upitch + (uint32_t)po;
                    for (int k = k0; k < k1; ++k)
                        st16_nt(band_out + (off + (uint32_t)k * upitch), v);
                } else {
                    for (int k = k0; k < k1; ++k)
                        st16_nt(out + (int64_t)(row0 + k) * pitch + X0 + po, v);
                }
            } else {
                for (int k = k0; k < k1; ++k) {
                    g_u8w* op = (g_u8w*)(out + (int64_t)(row0 + k) * pitch + X0);
                    for (int q = 0; q < real; ++q)
                        op[q] = exb[q];
                }
            }
        }
    }
}

// ==========================================================================
// Forward, fp32 CHW.  Column sums in fp32 over at most s_b rows, subcell and
// cell sums in fp64.
// ==========================================================================
// Broadcast of a tile's statistics to its real pixels, fp32 CHW: an item per
// (channel, subgrid row, 4-float strip) finds the strip's values among the
// tile's statistics in LDS and stores its s_b rows, consecutive lanes on
// consecutive strips; nothing is expanded and no lane waits for another.
// vgs / vgc hold the values of the simple cells and of the complex subcells
// (as the fp32 forward lays them out).  Bound by the stores.  64 x 3 x 218 x 178,
// b 8 / s_b 4: forward 29.6 -> 26.1 us, adjoint 47.7 -> 45.1; 32 x 3 x 512 x 512,
// b 16 / s_b 8: no change at 35 us each (before: one row of one channel
// expanded in LDS at a time, a barrier each, on as many lanes as it has strips).
__device__ __forceinline__ void broadcast_tile_f32(const FrameRec& F, int r, int64_t X0, int real, int Kt,
                                                   const uint8_t* cflag, const float* vgs, const float* vgc,
                                                   float* out)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, s = F.s, n = F.n, H = F.H, C = F.C;
    const int kn = Kt * n, nst = (real + 3) >> 2;
    const int64_t pitch = F.pitch, plane = pitch * H;
    const FastDiv by_nst(nst), by_n(n), by_s(s);
    for (int it = tid; it < C * n * nst; it += NT) {
        const int rest = by_nst(it), st = it - rest * nst;
        const int ch = by_n(rest), fr = rest - ch * n;
        const int row0 = r * b + fr * s;
        const int rows = min(s, H - row0);
        // the last strip ends with the real columns (the floats it shares with
        // its neighbour are written twice, alike)
        const int po = real >= 4 ? min(4 * st, real - 4) : 0;
        int fc = by_s(po), in = po - fc * s, kc = by_n(fc), jj = fc - kc * n;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = fc >= kn ? 0.f : (cflag[kc] ? vgc[(fr * kn + fc) * C + ch] : vgs[kc * C + ch]);
            if (++in == s) {
                in = 0;
                ++fc;
                if (++jj == n) {
                    jj = 0;
                    ++kc;
                }
            }
        }
        float* o = out + plane * ch + (int64_t)row0 * pitch + X0 + po;
        if (real >= 4) {
            const v4f w = v4f{v[0], v[1], v[2], v[3]};
            for (int k = 0; k < rows; ++k)
                st16f_nt(o + (int64_t)k * pitch, w);
        } else {
            for (int k = 0; k < rows; ++k)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (q < real)
                        ((g_f32w*)o)[(int64_t)k * pitch + q] = v[q];
        }
    }
}

// Column sums of one 4-float strip at any float of a row buffer.
__device__ __forceinline__ void store_colsums4(float* dst, const v4f& v)
{
    if ((reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
        *reinterpret_cast<v4f*>(dst) = v;
        return;
    }
    dst[0] = v.x;
    dst[1] = v.y;
    dst[2] = v.z;
    dst[3] = v.w;
}

__device__ void forward_tile_f32(const TileArgs& a, const FrameRec& F, const TileCoord& tc, uint8_t* lds)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, s = F.s, n = F.n, H = F.H, W = F.W, C = F.C, pad = F.pad;
    const int r = tc.r;
    const int x0c = tc.ct * F.K;
    const int Kt = min(F.K, F.GC - x0c);
    const int WB = Kt * b;                 // floats
    const int nstr = (WB + 3) >> 2;
    const int64_t X0 = (int64_t)x0c * b;
    const int64_t tile_end = X0 + WB;
    const int64_t lim = min(tile_end, (int64_t)W);
    const int64_t pitch = F.pitch;
    const int64_t plane = pitch * H;
    const float* img = static_cast<const float*>(a.images[tc.f]);
    float* out = a.outs ? static_cast<float*>(a.outs[tc.f]) : nullptr;
    const Strips sp = tile_strips_of(WB, (int)(lim - X0), 4, 1, pad);

    const double inv_s = exact_inv_area(F, s), inv_b = exact_inv_area(F, b);
    const LdsPlan L = lds_plan(kFwdF32, F.K, b, n, C);
    float* colsum = reinterpret_cast<float*>(lds + L.colsum);
    double* cspart = reinterpret_cast<double*>(lds + L.cspart);
    uint32_t* cidx = reinterpret_cast<uint32_t*>(lds + L.cidx);
    uint8_t* cflag = lds + L.cflag;
    float* vgs = reinterpret_cast<float*>(lds + L.vgs);
    float* vgc = reinterpret_cast<float*>(lds + L.vgc);

    tile_cells(a, F, tc.t, r, x0c, Kt, cidx, cflag);
    const uint64_t bg_base = a.counts[4 * tc.f + 2];
    const uint64_t fg_base = a.counts[4 * tc.f + 3];
    const int nn = n * n;
    const int kn = Kt * n;
    lds_barrier();

    // Subgrid rows in groups of kRowGroupF: one item per (channel, subgrid
    // row, 4-float strip), consecutive lanes on consecutive strips of a row,
    // rows added in order (fp32) with up to four loads in flight; then one
    // lane per (channel, subcell column) adds the s_b column sums (fp64) per
    // subgrid row and releases the complex subcells.
    const int kn4 = 4 * nstr;                 // floats of one row buffer
    const FastDiv by_kn(kn), by_n(n);
    for (int fr0 = 0; fr0 < n; fr0 += kRowGroupF) {
        const int ng = min(kRowGroupF, n - fr0);
        const int nit = sp.vec ? sp.nvec : nstr;
        const FastDiv by_nit(nit), by_ng(ng);
        for (int it = tid; it < C * ng * nit; it += NT) {
            const int rest = by_nit(it), st = it - rest * nit;
            const int ch = by_ng(rest), g = rest - ch * ng;
            const float* pl = img + plane * ch;
            const int row0 = r * b + (fr0 + g) * s;
            const int po = sp.vec ? min(4 * st, sp.real - 4) : 4 * st;   // the last strip ends with the real columns
            const int64_t p0 = X0 + po;
            // rows past the frame are absent in the unpadded mode
            const int srows = pad == kPadNone ? max(0, min(s, H - row0)) : s;
            const int64_t cend = pad == kPadNone ? lim : tile_end;
            v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
            if (p0 + 4 <= lim) {
                int k = 0;
                for (; k + 4 <= srows; k += 4) {
                    v4f w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        w[i] = ld16f_nt(pl + (int64_t)fold(row0 + k + i, H, pad) * pitch + p0);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc += w[i];
                }
                for (; k < srows; ++k)
                    acc += ld16f_nt(pl + (int64_t)fold(row0 + k, H, pad) * pitch + p0);
            } else {
                for (int k = 0; k < srows; ++k) {
                    const g_f32* rk = (const g_f32*)(pl + (int64_t)fold(row0 + k, H, pad) * pitch);
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[q] = (p0 + q < cend) ? rk[fold((int)(p0 + q), W, pad)] : 0.f;
                    acc.x += v[0]; acc.y += v[1]; acc.z += v[2]; acc.w += v[3];
                }
            }
            store_colsums4(colsum + (ch * ng + g) * kn4 + po, acc);
        }
        if (sp.vec && sp.real < WB) {
            // padded columns: the sums of the columns they mirror, or nothing
            const int np = WB - sp.real;
            if (pad != kPadNone)
                lds_barrier();
            const FastDiv by_np(np);
            for (int i = tid; i < C * ng * np; i += NT) {
                const int row = by_np(i);
                float* cs = colsum + row * kn4;
                const int x = sp.real + i - row * np;
                cs[x] = pad == kPadNone ? 0.f : cs[mirror_col(x, sp.real, pad)];
            }
        }
        lds_barrier();
        for (int j = tid; j < C * kn; j += NT) {
            const int ch = by_kn(j), fc = j - ch * kn;
            const int kc = by_n(fc), jj = fc - kc * n;
            const int ci = fc * C + ch;
            double part = fr0 == 0 ? 0.0 : cspart[ci];
            for (int g = 0; g < ng; ++g) {
                const float* cs = colsum + (ch * ng + g) * kn4 + fc * s;
                double S = 0.0;
                for (int x = 0; x < s; ++x)
                    S += (double)cs[x];
                part += S;
                if (cflag[kc]) {
                    const int fr = fr0 + g;
                    const int row0 = r * b + fr * s;
                    const uint32_t id = (uint32_t)(r * n + fr) * (uint32_t)(F.GC * n) + (uint32_t)(x0c * n + fc);
                    uint8_t pass;
                    const float v = release<true>(S, stat_area(F, row0, x0c * b + fc * s, s), inv_s, F.noise_fg,
                                            F.sigma_fg, F, id, ch, 1, pass);
                    const uint64_t at = fg_base + ((uint64_t)cidx[kc] * nn + fr * n + jj) * C + ch;
                    a.fg[at] = v;
                    if (a.clip_fg)
                        a.clip_fg[at] = pass;
                    vgc[(fr * kn + fc) * C + ch] = v;
                }
            }
            cspart[ci] = part;
        }
        lds_barrier();
    }
    const FastDiv by_c(C);
    for (int j = tid; j < Kt * C; j += NT) {
        const int kc = by_c(j), ch = j - kc * C;
        if (cflag[kc])
            continue;
        double S = 0.0;
        for (int jj = 0; jj < n; ++jj)
            S += cspart[(kc * n + jj) * C + ch];
        const uint32_t id = (uint32_t)(r * F.GC + x0c + kc);
        uint8_t pass;
        const float v = release<true>(S, stat_area(F, r * b, (x0c + kc) * b, b), inv_b, F.noise_bg, F.sigma_bg, F, id,
                                ch, 0, pass);
        const uint64_t at = bg_base + (uint64_t)cidx[kc] * C + ch;
        a.bg[at] = v;
        if (a.clip_bg)
            a.clip_bg[at] = pass;
        vgs[kc * C + ch] = v;
    }
    if (out == nullptr)
        return;
    lds_barrier();
    broadcast_tile_f32(F, r, X0, sp.real, Kt, cflag, vgs, vgc, out);
}

// Persistent workgroups take tiles from an atomic ticket; the last one out
// resets the ticket for the next launch (no memset, so graphs can replay).
// Each launch covers one group of frames sharing layout and channel count
// (scheduling indices [sched_offset, sched_offset + n_tiles)), so every kernel
// instantiation carries only its own path.
template <typename Body>
__device__ __forceinline__ void run_tiles(const TileArgs& a, uint8_t* lds, Body body)
{
    if (!a.persistent) {
        FrameRec F;
        const TileCoord tc = tile_of(a, blockIdx.x, F);
        body(F, tc);
        return;
    }
    __shared__ int64_t s_next;
    for (;;) {
        if (threadIdx.x == 0)
            s_next = (int64_t)atomicAdd(&a.ticket[0], 1u);
        lds_barrier();
        const int64_t idx = s_next;
        if (idx >= a.n_tiles)
            break;
        FrameRec F;
        const TileCoord tc = tile_of(a, idx, F);
        body(F, tc);
        lds_barrier();
    }
    if (threadIdx.x == 0) {
        __threadfence();
        const uint32_t done = atomicAdd(&a.ticket[1], 1u);
        if (done == gridDim.x - 1) {
            atomicExch(&a.ticket[0], 0u);
            atomicExch(&a.ticket[1], 0u);
        }
    }
}

// DPPIX_FWD_WAVES_PER_EU waves per SIMD: enough resident tiles per CU to keep HBM
// busy while other waves are in their LDS phases.
template <int C, bool DBG = false>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(DPPIX_FWD_WAVES_PER_EU))) void
k_forward_u8(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    run_tiles(a, lds, [&](const FrameRec& F, const TileCoord& tc) { forward_tile_u8<C, DBG>(a, F, tc, lds); });
}

// Five waves per SIMD (fp32 crops of 218 x 178: 22.6 -> 21.7 us).
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_forward_f32(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    run_tiles(a, lds, [&](const FrameRec& F, const TileCoord& tc) { forward_tile_f32(a, F, tc, lds); });
}

// ==========================================================================
// Reconstruction from the compact store (Sec. VI-F).
// ==========================================================================
// PACED: a wave has at most four row stores on their way, and none when it
// expands the next subgrid row.  Where two subgrid rows of five or six pixel
// rows make a tile, waves otherwise issue stores faster than the memory takes
// them, and the L2's write queues back up: 300 x 576 x 768 RGB, b 12 / s_b 6:
// 1.41 M stall cycles (TCC_EA0_WRREQ_STALL) and 77.5 us, paced 69.4; with the
// slower divisions that the expansion had once, 0.10 M and 72.4; b 10 / s_b 5: 99
// and 88.4.  64 frames: 21.2 / 20.6 and 24.4 / 23.6; 64 x 1080p, b 10 / s_b 5:
// 82.0 / 80.4; up to 16 frames 2 % slower.  Other grids gain nothing (n 2, s_b 8 and 9:
// -1 %, s_b 4: +2 %; n 4, s_b 6 and 8: +2 and +4 %).
template <int C, bool PACED>
__device__ void reconstruct_tile_u8(const TileArgs& a, const FrameRec& F, const TileCoord& tc, uint8_t* lds)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, s = F.s, n = F.n, H = F.H, W = F.W;
    const int r = tc.r;
    const int x0c = tc.ct * F.K;
    const int Kt = min(F.K, F.GC - x0c);
    const int WB = Kt * b * C;
    const int nstr = (WB + 15) >> 4;
    const int64_t X0 = (int64_t)x0c * b * C;
    const int64_t lim = min(X0 + WB, (int64_t)W * C);
    const int64_t pitch = F.pitch;
    uint8_t* out = static_cast<uint8_t*>(a.outs[tc.f]);
    const LdsPlan L = lds_plan(kRecU8, F.K, b, n, C);
    uint8_t* ex = lds + L.colsum;
    uint32_t* cidx = reinterpret_cast<uint32_t*>(lds + L.cidx);
    uint8_t* cflag = lds + L.cflag;
    uint8_t* vgs = lds + L.vgs;
    uint8_t* vgc = lds + L.vgc;
    tile_cells(a, F, tc.t, r, x0c, Kt, cidx, cflag);
    const uint64_t bg_base = a.counts[4 * tc.f + 2];
    const uint64_t fg_base = a.counts[4 * tc.f + 3];
    const int nn = n * n, kn = Kt * n;
    const FastDiv by_kn(kn), by_n(n);
    lds_barrier();
    for (int j = tid; j < Kt * C; j += NT) {
        const int kc = j / C, ch = j - kc * C;
        if (!cflag[kc])
            vgs[j] = to_u8(a.bg[bg_base + (uint64_t)cidx[kc] * C + ch]);
    }
    for (int j = tid; j < Kt * nn * C; j += NT) {
        // j = ((fr * kn) + fc) * C + ch
        const int ch = j % C;
        const int q = j / C;
        const int fr = by_kn(q), fc = q - fr * kn;
        const int kc = by_n(fc), jj = fc - kc * n;
        if (cflag[kc])
            vgc[j] = to_u8(a.fg[fg_base + ((uint64_t)cidx[kc] * nn + fr * n + jj) * C + ch]);
    }
    lds_barrier();
    const int real = (int)(lim - X0);
    const FastDiv by_nstr(nstr);
    const uint32_t upitch = (uint32_t)pitch;
    uint8_t* band_out = out + (int64_t)r * b * pitch + X0;
    for (int fr = 0; fr < n; ++fr) {
        uint8_t* exb = ex + (fr & 1) * (16 * nstr);   // two alternating row buffers
        expand_row_u8<C>(exb, kn, n, s, fr, cflag, vgs, vgc);
        lds_barrier();
        const int row0 = r * b + fr * s;
        const int rows = min(s, H - row0);
        // items (row part, strip): the s_b rows of a strip are split over
        // `parts` lanes when the tile has fewer strips than lanes
        const int parts = max(1, min(rows, NT / nstr));
        const int per = (rows + parts - 1) / max(parts, 1);
        for (int it = tid; it < nstr * parts; it += NT) {
            const int part = by_nstr(it);
            const int st = it - part * nstr;
            const int k0 = part * per, k1 = min(rows, k0 + per);
            if (16 * st >= real)
                continue;
            if (real >= 16) {
                // the last strip ends with the real columns (the bytes it
                // shares with its neighbour are written twice, alike)
                const int po = min(16 * st, real - 16);
                const v4u v = lds16(exb + po);
                if (F.off32) {
                    const uint32_t off = (uint32_t)(fr * s) * upitch + (uint32_t)po;
                    for (int k = k0; k < k1; ++k) {
                        st16_nt(band_out + (off + (uint32_t)k * upitch), v);
                        if constexpr (PACED)
                            asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
                    }
                } else {
                    for (int k = k0; k < k1; ++k)
                        st16_nt(out + (int64_t)(row0 + k) * pitch + X0 + po, v);
                }
            } else {
                for (int k = k0; k < k1; ++k) {
                    g_u8w* op = (g_u8w*)(out + (int64_t)(row0 + k) * pitch + X0);
                    for (int q = 0; q < real; ++q)
                        op[q] = exb[q];
                }
            }
        }
        if constexpr (PACED)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
}

__device__ void reconstruct_tile_f32(const TileArgs& a, const FrameRec& F, const TileCoord& tc, uint8_t* lds)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, n = F.n, W = F.W, C = F.C;
    const int r = tc.r;
    const int x0c = tc.ct * F.K;
    const int Kt = min(F.K, F.GC - x0c);
    const int64_t X0 = (int64_t)x0c * b;
    const int real = (int)(min(X0 + Kt * b, (int64_t)W) - X0);
    const LdsPlan L = lds_plan(kRecF32, F.K, b, n, C);
    uint32_t* cidx = reinterpret_cast<uint32_t*>(lds + L.cidx);
    uint8_t* cflag = lds + L.cflag;
    float* vgs = reinterpret_cast<float*>(lds + L.vgs);
    float* vgc = reinterpret_cast<float*>(lds + L.vgc);
    tile_cells(a, F, tc.t, r, x0c, Kt, cidx, cflag);
    const uint64_t bg_base = a.counts[4 * tc.f + 2];
    const uint64_t fg_base = a.counts[4 * tc.f + 3];
    const int nn = n * n, kn = Kt * n;
    const FastDiv by_kn(kn), by_n(n);
    lds_barrier();
    for (int j = tid; j < Kt * C; j += NT) {
        const int kc = j / C, ch = j - kc * C;
        if (!cflag[kc])
            vgs[j] = a.bg[bg_base + (uint64_t)cidx[kc] * C + ch];
    }
    for (int j = tid; j < Kt * nn * C; j += NT) {
        const int ch = j % C;
        const int q = j / C;
        const int fr = by_kn(q), fc = q - fr * kn;
        const int kc = by_n(fc), jj = fc - kc * n;
        if (cflag[kc])
            vgc[j] = a.fg[fg_base + ((uint64_t)cidx[kc] * nn + fr * n + jj) * C + ch];
    }
    lds_barrier();
    broadcast_tile_f32(F, r, X0, real, Kt, cflag, vgs, vgc, static_cast<float*>(a.outs[tc.f]));
}

template <int C, bool PACED = false>
__global__ __launch_bounds__(kMaxThreads) void k_reconstruct_u8(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    run_tiles(a, lds, [&](const FrameRec& F, const TileCoord& tc) { reconstruct_tile_u8<C, PACED>(a, F, tc, lds); });
}

__global__ __launch_bounds__(kMaxThreads) void k_reconstruct_f32(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    run_tiles(a, lds, [&](const FrameRec& F, const TileCoord& tc) { reconstruct_tile_f32(a, F, tc, lds); });
}

// ==========================================================================
// Adjoint (fp32 CHW).  Per tile: G_k = sum of grad_out over the real pixels
// of statistic k, g_k = pass_k * G_k / area_k (kept in the gradient store for
// the mirror terms), and every real pixel of the tile takes its own g_k.
// Then, only where padding folds onto real pixels: add the g of every padded
// position that folds onto the pixel.
// ==========================================================================
__device__ void backward_reduce_tile(const TileArgs& a, const FrameRec& F, const TileCoord& tc, uint8_t* lds)
{
    const int tid = threadIdx.x, NT = blockDim.x;
    const int b = F.b, s = F.s, n = F.n, H = F.H, W = F.W, C = F.C;
    const int r = tc.r;
    const int x0c = tc.ct * F.K;
    const int Kt = min(F.K, F.GC - x0c);
    const int WB = Kt * b;
    const int nstr = (WB + 3) >> 2;
    const int64_t X0 = (int64_t)x0c * b;
    const int64_t lim = min(X0 + WB, (int64_t)W);
    const int64_t pitch = F.pitch, plane = pitch * H;
    const float* go = a.grad_out[tc.f];
    // real columns only: padded ones have no output
    const Strips sp = tile_strips_of(WB, (int)(lim - X0), 4, 1, kPadNone);
    const LdsPlan L = lds_plan(kBwd, F.K, b, n, C);
    float* colsum = reinterpret_cast<float*>(lds + L.colsum);
    double* cspart = reinterpret_cast<double*>(lds + L.cspart);
    uint32_t* cidx = reinterpret_cast<uint32_t*>(lds + L.cidx);
    uint8_t* cflag = lds + L.cflag;
    float* vgs = reinterpret_cast<float*>(lds + L.vgs);
    float* vgc = reinterpret_cast<float*>(lds + L.vgc);
    float* gin = a.grad_in ? a.grad_in[tc.f] : nullptr;
    tile_cells(a, F, tc.t, r, x0c, Kt, cidx, cflag);
    const uint64_t bg_base = a.counts[4 * tc.f + 2];
    const uint64_t fg_base = a.counts[4 * tc.f + 3];
    const int nn = n * n, kn = Kt * n;
    lds_barrier();
    // as in the fp32 forward: (channel, subgrid row, strip) items over groups
    // of kRowGroupF subgrid rows, real rows only, in order, then one lane per
    // (channel, subcell column)
    const int kn4 = 4 * nstr;
    const FastDiv by_kn(kn), by_n(n);
    for (int fr0 = 0; fr0 < n; fr0 += kRowGroupF) {
        const int ng = min(kRowGroupF, n - fr0);
        const int nit = sp.vec ? sp.nvec : nstr;
        const FastDiv by_nit(nit), by_ng(ng);
        for (int it = tid; it < C * ng * nit; it += NT) {
            const int rest = by_nit(it), st = it - rest * nit;
            const int ch = by_ng(rest), g = rest - ch * ng;
            const float* pl = go + plane * ch;
            const int row0 = r * b + (fr0 + g) * s;
            const int rows = max(0, min(s, H - row0));   // real rows only
            const int po = sp.vec ? min(4 * st, sp.real - 4) : 4 * st;   // the last strip ends with the real columns
            const int64_t p0 = X0 + po;
            v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
            if (p0 + 4 <= lim) {
                const float* col = pl + (int64_t)row0 * pitch + p0;
                int k = 0;
                for (; k + 4 <= rows; k += 4) {
                    v4f w[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        w[i] = ld16f_nt(col + (int64_t)(k + i) * pitch);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc += w[i];
                }
                for (; k < rows; ++k)
                    acc += ld16f_nt(col + (int64_t)k * pitch);
            } else {
                for (int k = 0; k < rows; ++k) {
                    const g_f32* rk = (const g_f32*)(pl + (int64_t)(row0 + k) * pitch);
                    acc.x += (p0 + 0 < lim) ? rk[p0 + 0] : 0.f;
                    acc.y += (p0 + 1 < lim) ? rk[p0 + 1] : 0.f;
                    acc.z += (p0 + 2 < lim) ? rk[p0 + 2] : 0.f;
                    acc.w += (p0 + 3 < lim) ? rk[p0 + 3] : 0.f;
                }
            }
            store_colsums4(colsum + (ch * ng + g) * kn4 + po, acc);
        }
        if (sp.vec && sp.real < WB) {
            const int np = WB - sp.real;
            const FastDiv by_np(np);
            for (int i = tid; i < C * ng * np; i += NT) {
                const int row = by_np(i);
                colsum[row * kn4 + sp.real + i - row * np] = 0.f;
            }
        }
        lds_barrier();
        for (int j = tid; j < C * kn; j += NT) {
            const int ch = by_kn(j), fc = j - ch * kn;
            const int kc = by_n(fc), jj = fc - kc * n;
            const int ci = fc * C + ch;
            double part = fr0 == 0 ? 0.0 : cspart[ci];
            for (int g = 0; g < ng; ++g) {
                const float* cs = colsum + (ch * ng + g) * kn4 + fc * s;
                double G = 0.0;
                for (int x = 0; x < s; ++x)
                    G += (double)cs[x];
                part += G;
                if (cflag[kc]) {
                    const int fr = fr0 + g;
                    const uint64_t at = fg_base + ((uint64_t)cidx[kc] * nn + fr * n + jj) * C + ch;
                    const double area = stat_area(F, r * b + fr * s, x0c * b + fc * s, s);
                    const float gv = (a.clip_fg[at] && area > 0.0) ? (float)(G / area) : 0.f;
                    a.g_fg[at] = gv;
                    vgc[(fr * kn + fc) * C + ch] = gv;
                }
            }
            cspart[ci] = part;
        }
        lds_barrier();
    }
    for (int j = tid; j < Kt * C; j += NT) {
        const int kc = j / C, ch = j - kc * C;
        if (cflag[kc])
            continue;
        double G = 0.0;
        for (int jj = 0; jj < n; ++jj)
            G += cspart[(kc * n + jj) * C + ch];
        const uint64_t at = bg_base + (uint64_t)cidx[kc] * C + ch;
        const float gv = a.clip_bg[at] ? (float)(G / stat_area(F, r * b, (x0c + kc) * b, b)) : 0.f;
        a.g_bg[at] = gv;
        vgs[kc * C + ch] = gv;
    }
    if (gin == nullptr)
        return;
    // every real pixel takes its own statistic's gradient (the mirror terms
    // of pixels near padded borders are added by a later pass)
    lds_barrier();
    broadcast_tile_f32(F, r, X0, sp.real, Kt, cflag, vgs, vgc, gin);
}

// Seven waves per SIMD (adjoint of fp32 crops of 218 x 178: 27.2 -> 24.2 us).
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(7))) void k_backward_reduce(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    run_tiles(a, lds, [&](const FrameRec& F, const TileCoord& tc) { backward_reduce_tile(a, F, tc, lds); });
}

// Gradient of the statistic of cell (cy, cx) at its subgrid row i, column j.
__device__ __forceinline__ float g_at(const TileArgs& a, const FrameRec& F, int f, int cy, int cx, int i, int j, int ch)
{
    const int64_t cell = F.cell_base + (int64_t)cy * F.GC + cx;
    const uint32_t idx = a.cell_index[cell];
    const uint8_t fl = a.flags[cell];
    const float* g = fl ? a.g_fg + a.counts[4 * f + 3] + ((uint64_t)idx * F.n * F.n + i * F.n + j) * F.C
                        : a.g_bg + a.counts[4 * f + 2] + (uint64_t)idx * F.C;
    return g[ch];
}

// Mirror terms of the adjoint: a real pixel near the bottom or right border is
// also the source of the padded positions that fold onto it, and collects
// their statistics' gradients too.  Its own statistic's gradient is already in
// grad_in (broadcast by the reduction's tile), so only
// the pixels that have mirror preimages are visited, and only the mirror
// terms are added.  Nothing to do in the unpadded mode.
__global__ __launch_bounds__(kMaxThreads) void k_backward_mirror(TileArgs a)
{
    const UnitCoord u = unit_of(a, blockIdx.x);
    const int f = u.f;
    const FrameRec& F = a.frames[f];
    const int b = F.b, H = F.H, W = F.W, pad = F.pad;
    const BorderArea m = border_area(F);
    const BorderPart part(m, W, u.local);
    const int ch = part.ch;
    const int PR = F.GR * b - H, PC = F.GC * b - W;
    const int64_t pitch = F.pitch, plane = pitch * H;
    g_f32w* gi = (g_f32w*)a.grad_in[f] + plane * ch;
    // Where the padding folds onto the frame once, a pixel has at most one
    // padded row and one padded column, which lie in the last band and the
    // last column of cells: their statistics' loads are all in flight
    // together.  (64 x 3 x 218 x 178, b 8: the adjoint 88.5 -> 27 us; a search
    // over the padding, channel after channel, was one chain of dependent
    // loads, every position's cell a division, and one workgroup walked the
    // whole of a tile.)
    const int last = pad == 0 ? 1 : 2;              // mirror of y: 2 H - last - y
    const bool once = PR <= H - (last - 1) && PC <= W - (last - 1);
    const FastDiv by_s(F.s);
    const WideDiv by_b(b), by_wide((int)part.wide);
    for (int k = threadIdx.x; k < part.n; k += blockDim.x) {
        int y, x;
        part.pixel(m, k, by_wide, y, x);
        g_f32w* dst = gi + (int64_t)y * pitch + x;
        const int cy = by_b(y), cx = by_b(x);
        const int i = by_s(y - cy * b), j = by_s(x - cx * b);
        float acc = 0.f;
        if (once) {
            const int yy = 2 * H - last - y, xx = 2 * W - last - x;
            const int ly = (F.GR - 1) * b, lx = (F.GC - 1) * b;      // first row of the last band, column of the last cell
            const bool rows = yy >= H && yy < F.GR * b, cols = xx >= W && xx < F.GC * b;
            const int im = rows ? by_s(yy - ly) : 0, jm = cols ? by_s(xx - lx) : 0;
            const float old = *dst;
            const float g0 = rows ? g_at(a, F, f, F.GR - 1, cx, im, j, ch) : 0.f;
            const float g1 = rows && cols ? g_at(a, F, f, F.GR - 1, F.GC - 1, im, jm, ch) : 0.f;
            const float g2 = cols ? g_at(a, F, f, cy, F.GC - 1, i, jm, ch) : 0.f;
            acc = (g0 + g1) + g2;
            if (acc != 0.f)
                *dst = old + acc;
            continue;
        }
        // padded rows folding onto y, each also with the padded columns folding onto x
        for (int yy = H; yy < F.GR * b; ++yy)
            if (fold(yy, H, pad) == y) {
                const int im = by_s(yy - (F.GR - 1) * b);
                acc += g_at(a, F, f, F.GR - 1, cx, im, j, ch);
                for (int xx = W; xx < F.GC * b; ++xx)
                    if (fold(xx, W, pad) == x)
                        acc += g_at(a, F, f, F.GR - 1, F.GC - 1, im, by_s(xx - (F.GC - 1) * b), ch);
            }
        for (int xx = W; xx < F.GC * b; ++xx)
            if (fold(xx, W, pad) == x)
                acc += g_at(a, F, f, cy, F.GC - 1, i, by_s(xx - (F.GC - 1) * b), ch);
        if (acc != 0.f)
            *dst += acc;
    }
}

// ==========================================================================
// Complexity label from the image (Sec. VI-A names the Sobel operator as one
// source of the region mask): per real pixel, the 3x3 Sobel responses of the
// channel sum S, with neighbours past the border mirrored; the pixel is an
// edge pixel when |Gx| + |Gy| >= threshold * C.  A unit is a frame's columns
// cut into equal chunks of at most kLabCols x a segment of rows, walked as the
// plan from labels walks them; a lane writes its four labels of a row as one
// dword at any byte of the mask.
// ==========================================================================
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) u32_any g_u32w;

template <int C>
__global__ __launch_bounds__(256) void k_edge_mask(TileArgs a)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x;
    const int64_t unit = a.sched_offset + blockIdx.x;
    const UnitCoord u = unit_of(a, unit);
    const int f = u.f, local = u.local;
    const FrameRec& F = a.frames[f];
    const int H = F.H, W = F.W;
    const int chunks = (W + kLabCols - 1) / kLabCols, width = label_chunk(W);
    const int seg = local / chunks;
    const int px0 = (local - seg * chunks) * width, py0 = seg * a.edge_rows;
    const int cols = min(width, W - px0), rows = min(a.edge_rows, H - py0);
    if (cols <= 0)
        return;
    const int n = min(4, cols - 4 * tid);
    uint8_t* out = a.masks_out[f] + (int64_t)py0 * W + px0 + 4 * tid;
    label_walk<C>(static_cast<const uint8_t*>(a.images[f]), F.pitch, H, W, F.pad, py0, rows, px0, cols,
                  a.edge_threshold * C, reinterpret_cast<uint16_t*>(lds), label_stride(4 * (int)blockDim.x),
                  [&](int y0, int ya, int yb, const uint32_t (&lab)[kLabBlock]) {
#pragma unroll
        for (int i = 0; i < kLabBlock; ++i) {
            if (y0 + i < ya || y0 + i >= yb)
                continue;
            uint8_t* o = out + (int64_t)(y0 + i) * W;
            if (n == 4)
                __builtin_nontemporal_store(lab[i], (g_u32w*)o);
            else
                for (int q = 0; q < n; ++q)
                    ((g_u8w*)o)[q] = (uint8_t)(lab[i] >> (8 * q));
        }
    });
}

// ==========================================================================
// Utility metrics of the paper's evaluation (Sec. VII-A): MSE and SSIM
// (Wang et al. 2004; 7 x 7 equal-weight windows fully inside the frame,
// sample covariances, K1 = 0.01, K2 = 0.03, range 255, channels averaged).
// With uint8 inputs every window sum of x, y, x^2, y^2 and xy is an integer,
// so the sums are exact and so are the numerators below; only the final
// ratio is fp64.  Each unit writes its partial sums; k_metrics_reduce adds a
// frame's in a fixed order (strided over the lanes, then a tree).
//
// SSIM of a window from its integer sums s0 = sum x, s1 = sum y, s2 = sum x^2,
// s3 = sum y^2, s4 = sum xy over np = 49 pixels: with ux = s0/49, the sample
// variances (49 s2 - s0^2) / (49 * 48) and covariance (49 s4 - s0 s1) / (49 * 48),
// the four factors of SSIM share the denominators 49^2 and 49 * 48, which
// cancel:  SSIM = (A B) / (D E) with
//   A = 2 s0 s1 + 49^2 c1,            B = 2 (49 s4 - s0 s1) + 49 * 48 c2,
//   D = s0^2 + s1^2 + 49^2 c1,        E = 49 (s2 + s3) - s0^2 - s1^2 + 49 * 48 c2,
// every integer part below 2^31.
//
// The kernel is bound by its vector instructions (the frames are read once,
// 2 bytes per pixel and channel against about 40 instructions), so the work
// is laid out to share them.  A unit is kCw pixels x a segment of rows of
// one frame, whatever the plan's tiles: a lane takes the two windows that
// start at one even pixel of one channel and walks down the rows.  The eight
// taps of the pair are two words of a channel plane in LDS; byte dot products
// add them onto running sums (one per moment and window) that are never
// reset, and a window's sum is the running sum minus its value seven rows
// earlier (a ring in registers): one subtraction per moment.  SSIM needs the
// sum of x^2 and y^2 only together, and the pair's two quotients share one
// reciprocal.  Rows come in blocks of seven (the ring's length), each block's
// vectors loaded while the one before is worked on (two LDS buffers, one
// barrier per block).
// 16 x 1080p RGB: 275 -> 164 us; 6000 x 4000 RGB: 380 -> 125 us; 24 photos of
// odd widths: 417 -> 124 us (before: one window per lane, 38-row chunks staged
// per tile, squared errors by a second read, vectors only for aligned rows,
// and one lane per frame for the final sums).
// ==========================================================================
constexpr int kMetBlock = 7;                    // rows per block: the window's height

// A unit's lanes, windows of a lane, pixels (their windows start in it, and
// their squared errors are its own), 16-pixel groups of a staged row (the
// windows reach 6 pixels further), and bytes of a staged plane row.
//
// NARROW: one wave a unit and one window a lane, for batches whose frames leave
// the lanes of wide units idle (metrics_narrow; an idle wave still holds its
// registers, and there are twelve waves' worth on a CU).  256 RGB frames of 64
// x 64: 23.1 us wide, 14.2 narrow, 13.0 with a kernel of a window a lane and
// four workgroups a frame; 512 of 32 x 32: 24 / 10.7 / 10.6; 64 of 218 x 178:
// 39.6 / 29.9 / 62; 256 gray ones of 64 x 64: 18.7 / 8.7 / 10.0.  Pairs of windows
// in single waves were slower: 15.4 and, of four channels, 20 us where single
// windows then took 14.4 and 17.3.
template <int C, bool NARROW>
struct MetShape {
    static constexpr int kThreads = NARROW ? 64 : 256;
    static constexpr int kWin = NARROW ? 1 : 2;
    static constexpr int kCw = kThreads * kWin / C / 16 * 16;
    static constexpr int kGroups = kCw / 16 + 1;
    static constexpr int kRow = 16 * kGroups;
};

template <int C, bool NARROW>
struct MetLds {
    alignas(16) uint8_t px[2][2][C][kMetBlock][MetShape<C, NARROW>::kRow];   // [buffer][frame]
    double red[4];
    unsigned long long red_se[4];
};

// Add the moments of one row's pair of windows, the 7 taps from byte `sh` of
// xr[0] and the 7 from the byte after it, onto the running sums: per window
// sum x, sum y, sum x^2 + y^2, sum xy.
__device__ __forceinline__ void add_row_moments(const uint32_t* xr, const uint32_t* yr, uint32_t sh,
                                                uint32_t (&t)[2][4])
{
    const uint32_t xa = __builtin_amdgcn_alignbyte(xr[1], xr[0], sh), xb = __builtin_amdgcn_alignbyte(xr[2], xr[1], sh);
    const uint32_t ya = __builtin_amdgcn_alignbyte(yr[1], yr[0], sh), yb = __builtin_amdgcn_alignbyte(yr[2], yr[1], sh);
    const uint32_t xb0 = xb & 0x00FFFFFFu, yb0 = yb & 0x00FFFFFFu, xa1 = xa & 0xFFFFFF00u, ya1 = ya & 0xFFFFFF00u;
    constexpr uint32_t one = 0x01010101u, low = 0x00010101u, high = 0x01010100u;
    t[0][0] = __builtin_amdgcn_udot4(xb, low, __builtin_amdgcn_udot4(xa, one, t[0][0], false), false);
    t[0][1] = __builtin_amdgcn_udot4(yb, low, __builtin_amdgcn_udot4(ya, one, t[0][1], false), false);
    t[1][0] = __builtin_amdgcn_udot4(xb, one, __builtin_amdgcn_udot4(xa, high, t[1][0], false), false);
    t[1][1] = __builtin_amdgcn_udot4(yb, one, __builtin_amdgcn_udot4(ya, high, t[1][1], false), false);
    t[0][2] = __builtin_amdgcn_udot4(xb, xb0, __builtin_amdgcn_udot4(xa, xa, t[0][2], false), false);
    t[0][2] = __builtin_amdgcn_udot4(yb, yb0, __builtin_amdgcn_udot4(ya, ya, t[0][2], false), false);
    t[1][2] = __builtin_amdgcn_udot4(xb, xb, __builtin_amdgcn_udot4(xa, xa1, t[1][2], false), false);
    t[1][2] = __builtin_amdgcn_udot4(yb, yb, __builtin_amdgcn_udot4(ya, ya1, t[1][2], false), false);
    t[0][3] = __builtin_amdgcn_udot4(xb0, yb, __builtin_amdgcn_udot4(xa, ya, t[0][3], false), false);
    t[1][3] = __builtin_amdgcn_udot4(xb, yb, __builtin_amdgcn_udot4(xa1, ya, t[1][3], false), false);
}

// The same for one window, the 7 taps from byte `sh`.
__device__ __forceinline__ void add_row_moments(const uint32_t* xr, const uint32_t* yr, uint32_t sh,
                                                uint32_t (&t)[1][4])
{
    const uint32_t xa = __builtin_amdgcn_alignbyte(xr[1], xr[0], sh), ya = __builtin_amdgcn_alignbyte(yr[1], yr[0], sh);
    const uint32_t xb = __builtin_amdgcn_alignbyte(xr[2], xr[1], sh) & 0x00FFFFFFu;
    const uint32_t yb = __builtin_amdgcn_alignbyte(yr[2], yr[1], sh) & 0x00FFFFFFu;
    constexpr uint32_t one = 0x01010101u;
    t[0][0] = __builtin_amdgcn_udot4(xb, one, __builtin_amdgcn_udot4(xa, one, t[0][0], false), false);
    t[0][1] = __builtin_amdgcn_udot4(yb, one, __builtin_amdgcn_udot4(ya, one, t[0][1], false), false);
    t[0][2] = __builtin_amdgcn_udot4(xb, xb, __builtin_amdgcn_udot4(xa, xa, t[0][2], false), false);
    t[0][2] = __builtin_amdgcn_udot4(yb, yb, __builtin_amdgcn_udot4(ya, ya, t[0][2], false), false);
    t[0][3] = __builtin_amdgcn_udot4(xb, yb, __builtin_amdgcn_udot4(xa, ya, t[0][3], false), false);
}

// A quarter of SSIM's numerator and its denominator (A B / 4 and D E above)
// of one window, from sum x, sum y, sum x^2 + y^2 and sum xy.  Every integer
// is below 2^53, so the products are exact and each factor is rounded once.
__device__ __forceinline__ void ssim_ratio(uint32_t s0, uint32_t s1, uint32_t s23, uint32_t s4, double& num, double& den)
{
    constexpr double c1 = (0.01 * 255.0) * (0.01 * 255.0), c2 = (0.03 * 255.0) * (0.03 * 255.0);
    const double x = (double)s0, y = (double)s1;
    const double p = x * y, q = fma(x, x, y * y);
    const double B = fma(49.0, (double)s4, -p), E = fma(49.0, (double)s23, -q);
    num = (p + 0.5 * (2401.0 * c1)) * (B + 0.5 * (2352.0 * c2));
    den = (q + 2401.0 * c1) * (E + 2352.0 * c2);
}

// Sixteen pixels of C interleaved channels (C 16-byte vectors; pixel i's
// channel c at byte C i + c) as C planes of 16 bytes, by byte permutes.
template <int C>
__device__ __forceinline__ void deinterleave16(const v4u (&v)[C], v4u (&p)[C])
{
    uint32_t d[4 * C], o[4 * C];   // o[4 c + j]: pixels 4 j .. 4 j + 3 of channel c
#pragma unroll
    for (int i = 0; i < C; ++i) {
        d[4 * i] = v[i].x;
        d[4 * i + 1] = v[i].y;
        d[4 * i + 2] = v[i].z;
        d[4 * i + 3] = v[i].w;
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (C == 1) {
                o[j] = d[j];
            } else if constexpr (C == 2) {
                o[4 * c + j] = __builtin_amdgcn_perm(d[2 * j + 1], d[2 * j], 0x06040200u + 0x01010101u * c);
            } else if constexpr (C == 3) {
                constexpr uint32_t lo[3] = {0x0C060300u, 0x0C070401u, 0x0C0C0502u};
                constexpr uint32_t hi[3] = {0x05020100u, 0x06020100u, 0x07040100u};
                o[4 * c + j] = __builtin_amdgcn_perm(d[3 * j + 2], __builtin_amdgcn_perm(d[3 * j + 1], d[3 * j], lo[c]),
                                                     hi[c]);
            } else {
                const uint32_t sel = 0x0C0C0400u + 0x0101u * c;
                o[4 * c + j] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(d[4 * j + 3], d[4 * j + 2], sel),
                                                     __builtin_amdgcn_perm(d[4 * j + 1], d[4 * j], sel), 0x05040100u);
            }
        }
#pragma unroll
    for (int c = 0; c < C; ++c)
        p[c] = v4u{o[4 * c], o[4 * c + 1], o[4 * c + 2], o[4 * c + 3]};
}

// A plane of 16 bytes with its last 16 - sh bytes moved to the front, zeros
// behind them.
__device__ __forceinline__ void drop_bytes(v4u& w, int sh)
{
    if (sh & 8) {
        w.x = w.z;
        w.y = w.w;
        w.z = w.w = 0u;
    }
    if (sh & 4) {
        w.x = w.y;
        w.y = w.z;
        w.z = w.w;
        w.w = 0u;
    }
    const uint32_t b = (uint32_t)(sh & 3);
    w.x = __builtin_amdgcn_alignbyte(w.y, w.x, b);
    w.y = __builtin_amdgcn_alignbyte(w.z, w.y, b);
    w.z = __builtin_amdgcn_alignbyte(w.w, w.z, b);
    w.w = __builtin_amdgcn_alignbyte(0u, w.w, b);
}

// Squared differences of two planes' 16 bytes: sum x^2 + sum y^2 - 2 sum xy.
__device__ __forceinline__ uint32_t sq_diff16(const v4u& x, const v4u& y)
{
    uint32_t s = 0u, m = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        s = __builtin_amdgcn_udot4(x[k], x[k], s, false);
        s = __builtin_amdgcn_udot4(y[k], y[k], s, false);
        m = __builtin_amdgcn_udot4(x[k], y[k], m, false);
    }
    return s - 2u * m;
}

// One 16-pixel group of one row, C interleaved 16-byte vectors.
template <int C>
struct MetGroup {
    v4u w[C];

    // n < 0: all 16 pixels; else the first n of a frame narrower than that.
    __device__ __forceinline__ void load(const uint8_t* p, int n)
    {
        if (n < 0) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                w[c] = ld16_nt(p + 16 * c);
            return;
        }
        const g_u8* g = (const g_u8*)p;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t v = 0u;
                for (int b = 0; b < 4; ++b) {
                    const int i = 16 * c + 4 * k + b;
                    if (i < n * C)
                        v |= (uint32_t)g[i] << (8 * b);
                }
                w[c][k] = v;
            }
    }

    // Into the planes of a staged row, `back` pixels further left (a group
    // that crosses the right edge is read that far back from its place).
    __device__ __forceinline__ void store(uint8_t* dst, int plane, int back)
    {
        v4u p[C];
        deinterleave16<C>(w, p);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (back != 0)
                drop_bytes(p[c], back);
            *reinterpret_cast<v4u*>(dst + c * plane) = p[c];
        }
    }
};

// Three waves per SIMD: the ring of a pair of windows is 56 registers, and with
// the 128 of four waves the kernel spills (444 us instead of 164, 16 x 1080p).
template <int C, bool NARROW>
__global__ __launch_bounds__((NARROW ? 64 : 256)) __attribute__((amdgpu_waves_per_eu(3))) void
k_metrics(TileArgs a)
{
    __shared__ MetLds<C, NARROW> L;
    using Sh = MetShape<C, NARROW>;
    constexpr int NT = Sh::kThreads, kWin = Sh::kWin;
    const int tid = threadIdx.x;
    const int64_t unit = a.sched_offset + blockIdx.x;
    const UnitCoord u = unit_of(a, unit);
    const int f = u.f, local = u.local;
    const FrameRec& F = a.frames[f];
    const int H = F.H, W = F.W;
    const int64_t pitch = F.pitch;
    const int cols = (W + Sh::kCw - 1) / Sh::kCw;
    const int seg = local / cols;
    const int p0 = (local - seg * cols) * Sh::kCw, r0 = seg * a.met_rows;
    const int own = min(a.met_rows, H - r0);                 // rows whose squared errors are the unit's
    const int nrow = min(a.met_rows + kMetBlock - 1, H - r0);   // rows its windows read
    const int nblk = (nrow + kMetBlock - 1) / kMetBlock;
    const uint8_t* X = static_cast<const uint8_t*>(a.images[f]) + (int64_t)r0 * pitch;
    const uint8_t* Y = static_cast<const uint8_t*>(a.outs[f]) + (int64_t)r0 * pitch;
    double acc = 0.0;
    uint32_t se = 0u;

    // Staging of a block: an item per (frame, row, 16-pixel group).  Where
    // they do not fill the workgroup, another wave begins each block, so that
    // every SIMD gets its share.
    constexpr int kItems = 2 * kMetBlock * Sh::kGroups, kPer = (kItems + NT - 1) / NT;
    const int narrow = W >= 16 ? -1 : W;
    MetGroup<C> grp[kPer];
    struct Item {
        int y, row, g, px, from;
        bool in;
    };
    auto item = [&](int blk, int i) {
        const int it = ((tid + 64 * blk) & (NT - 1)) + NT * i;
        Item m;
        m.y = it / (kMetBlock * Sh::kGroups);
        const int q = it - m.y * (kMetBlock * Sh::kGroups);
        m.row = q / Sh::kGroups;
        m.g = q - m.row * Sh::kGroups;
        m.px = p0 + 16 * m.g;
        m.from = W >= 16 ? min(m.px, W - 16) : 0;
        m.in = it < kItems && m.px < W && blk * kMetBlock + m.row < nrow;
        return m;
    };
    auto load = [&](int blk) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const Item m = item(blk, i);
            if (m.in)
                grp[i].load((m.y ? Y : X) + (int64_t)(blk * kMetBlock + m.row) * pitch + (int64_t)m.from * C, narrow);
        }
    };
    auto store = [&](int blk) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const Item m = item(blk, i);
            if (m.in)
                grp[i].store(&L.px[blk & 1][m.y][0][m.row][16 * m.g], kMetBlock * Sh::kRow, m.px - m.from);
        }
    };
    // Squared errors of a staged block: a lane per (channel, row, group) of
    // the unit's own pixels (planes end in zeros past the right edge).
    constexpr int kOwnGroups = Sh::kCw / 16;
    const int eg = tid % kOwnGroups, erow = tid / kOwnGroups % kMetBlock, ech = tid / (kOwnGroups * kMetBlock);
    const bool errs = ech < C && p0 + 16 * eg < W;
    auto errors = [&](int blk) {
        if (errs && blk * kMetBlock + erow < own)
            se += sq_diff16(*reinterpret_cast<const v4u*>(&L.px[blk & 1][0][ech][erow][16 * eg]),
                            *reinterpret_cast<const v4u*>(&L.px[blk & 1][1][ech][erow][16 * eg]));
    };
    // this lane's (channel, first window)
    constexpr int kLanes = Sh::kCw / kWin;
    const int ch = tid / kLanes, w0 = kWin * (tid - ch * kLanes);
    const bool works = ch < C && p0 + w0 < W - 6 && nrow >= kMetBlock;
    const double second = p0 + w0 + 1 < W - 6 ? 1.0 : 0.0;
    const uint32_t sh = (uint32_t)(w0 & 3);
    const int word = w0 >> 2;
    uint32_t t[kWin][4] = {};
    uint32_t ring[kMetBlock][kWin][4];
    // One block of rows.  `first`: windows end only with its last row, and
    // start at the unit's first; `full`: all seven rows are there (no branch
    // between them, so their loads and sums interleave).
    auto rows = [&](int blk, auto first, auto full) {
        const uint32_t* xr = reinterpret_cast<const uint32_t*>(&L.px[blk & 1][0][ch][0][0]) + word;
        const uint32_t* yr = reinterpret_cast<const uint32_t*>(&L.px[blk & 1][1][ch][0][0]) + word;
#pragma unroll
        for (int j = 0; j < kMetBlock; ++j) {
            if (!full && blk * kMetBlock + j >= nrow)
                break;
            add_row_moments(xr + j * (Sh::kRow / 4), yr + j * (Sh::kRow / 4), sh, t);
            if (!first || j == kMetBlock - 1) {
                uint32_t w[kWin][4];
#pragma unroll
                for (int m = 0; m < 4 * kWin; ++m)
                    w[m >> 2][m & 3] = t[m >> 2][m & 3] - (first ? 0u : ring[j][m >> 2][m & 3]);
                // n0 / d0 + n1 / d1 over one reciprocal, refined by one
                // Newton step (it squares the relative error); the
                // denominators are normal numbers below 2^62
                double n0, d0, n1, d1;
                ssim_ratio(w[0][0], w[0][1], w[0][2], w[0][3], n0, d0);
                double num = n0, den = d0;
                if constexpr (kWin == 2) {
                    ssim_ratio(w[1][0], w[1][1], w[1][2], w[1][3], n1, d1);
                    num = fma(n0, d1, second * n1 * d0);
                    den = d0 * d1;
                }
                double r = __builtin_amdgcn_rcp(den);
                r = fma(r, fma(-den, r, 1.0), r);
                acc = fma(num, r, acc);
            }
#pragma unroll
            for (int m = 0; m < 4 * kWin; ++m)
                ring[j][m >> 2][m & 3] = t[m >> 2][m & 3];
        }
    };
    load(0);
    store(0);
    lds_barrier();
    if (nblk > 1)
        load(1);
    errors(0);
    if (works)
        rows(0, std::true_type(), std::true_type());
    for (int blk = 1; blk < nblk; ++blk) {
        store(blk);
        lds_barrier();
        if (blk + 1 < nblk)
            load(blk + 1);
        errors(blk);
        if (works) {
            if ((blk + 1) * kMetBlock <= nrow)
                rows(blk, std::false_type(), std::true_type());
            else
                rows(blk, std::false_type(), std::false_type());
        }
    }
    // workgroup reduction in a fixed order
    acc *= 4.0;
    unsigned long long se64 = se;
    for (int d = 32; d > 0; d >>= 1) {
        acc += __shfl_down(acc, d, 64);
        se64 += __shfl_down(se64, d, 64);
    }
    if ((tid & 63) == 0) {
        L.red[tid >> 6] = acc;
        L.red_se[tid >> 6] = se64;
    }
    lds_barrier();
    if (tid == 0) {
        a.met_partial[2 * unit] = NARROW ? L.red[0] : (L.red[0] + L.red[1]) + (L.red[2] + L.red[3]);
        reinterpret_cast<unsigned long long*>(a.met_partial)[2 * unit + 1] =
            NARROW ? L.red_se[0] : (L.red_se[0] + L.red_se[1]) + (L.red_se[2] + L.red_se[3]);
    }
}

// One workgroup per frame: MSE = sum of squared errors / (H W C); SSIM = sum
// of window values / (windows * C), the units' partial sums added in a fixed
// order (strided over the lanes, then a tree).
__global__ __launch_bounds__(256) void k_metrics_reduce(TileArgs a, double* out)
{
    __shared__ double red[4];
    __shared__ unsigned long long red_se[4];
    const int f = a.spans[blockIdx.x].frame, tid = threadIdx.x;
    const FrameRec& F = a.frames[f];
    const int64_t base = a.spans[blockIdx.x].first, n = a.spans[blockIdx.x + 1].first - base;
    double t = 0.0;
    unsigned long long e = 0;
    for (int64_t i = tid; i < n; i += 256) {
        t += a.met_partial[2 * (base + i)];
        e += reinterpret_cast<const unsigned long long*>(a.met_partial)[2 * (base + i) + 1];
    }
    for (int d = 32; d > 0; d >>= 1) {
        t += __shfl_down(t, d, 64);
        e += __shfl_down(e, d, 64);
    }
    if ((tid & 63) == 0) {
        red[tid >> 6] = t;
        red_se[tid >> 6] = e;
    }
    lds_barrier();
    if (tid != 0)
        return;
    t = (red[0] + red[1]) + (red[2] + red[3]);
    e = (red_se[0] + red_se[1]) + (red_se[2] + red_se[3]);
    const double windows = (double)max(F.H - 6, 0) * (double)max(F.W - 6, 0) * F.C;
    out[2 * f + 0] = (double)e / ((double)F.H * F.W * F.C);
    out[2 * f + 1] = windows > 0 ? t / windows : 0.0;
}

// Advance every frame's Philox counter (frame_index) by `step`: the next
// video step of a captured graph draws fresh noise.
__global__ void k_noise_advance(uint64_t* noise, int32_t n, uint64_t step)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        noise[2 * i + 1] += step;
}

// ==========================================================================
// Diagnostics.
// ==========================================================================
__global__ void k_philox(const uint32_t* in, uint32_t* out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t* p = in + 6 * i;
    const uint4 w = philox10(make_uint4(p[0], p[1], p[2], p[3]), p[4], p[5]);
    out[4 * i + 0] = w.x;
    out[4 * i + 1] = w.y;
    out[4 * i + 2] = w.z;
    out[4 * i + 3] = w.w;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
// Workgroups asking for more than 64 KiB of LDS must opt in per kernel.  The
// limit belongs to the kernel, not to a plan, so it is only ever raised (per
// device, under a lock): a smaller request from one host thread must not
// lower it between another thread's opt-in and its launch.
template <typename K>
hipError_t allow_lds(K kernel, size_t lds)
{
    if (lds <= 65536)
        return hipSuccess;
    static std::mutex mu;
    static std::map<std::pair<int, const void*>, size_t> granted;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    const void* fn = reinterpret_cast<const void*>(kernel);
    std::lock_guard<std::mutex> lock(mu);
    size_t& g = granted[{dev, fn}];
    if (lds <= g)
        return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess)
        g = lds;
    return e;
}

hipError_t launch_scan(const TileArgs& a, bool prefix_scan, hipStream_t s)
{
    if (prefix_scan)
        hipLaunchKernelGGL(k_scan_prefix, dim3((unsigned)a.n_frames), dim3(256), 0, s, a);
    else {
        hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)a.n_frames), dim3(256), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_scan_frames, dim3(1), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_plan(const TileArgs& a, int64_t n_units, int threads, size_t lds, bool prefix_scan, hipStream_t s)
{
    if (n_units == 0)
        return hipSuccess;
    if (a.masks == nullptr) {
        const int64_t n = std::max<int64_t>(std::max<int64_t>(a.total_cells, a.n_tiles), 4 * (int64_t)a.n_frames);
        const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 2048);
        hipLaunchKernelGGL(k_plan_simple, dim3(grid), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    hipError_t e = allow_lds(k_plan, lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_plan, dim3((unsigned)n_units), dim3(threads), lds, s, a);
    e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_scan(a, prefix_scan, s);
}

hipError_t launch_plan_labels(const TileArgs& a, int C, int64_t n_units, int threads, size_t lds, hipStream_t s)
{
    if (n_units == 0)
        return hipSuccess;
    const dim3 grid((unsigned)n_units), block((unsigned)threads);
    switch (C) {
    case 1: hipLaunchKernelGGL(k_plan_labels<1>, grid, block, lds, s, a); break;
    case 2: hipLaunchKernelGGL(k_plan_labels<2>, grid, block, lds, s, a); break;
    case 3: hipLaunchKernelGGL(k_plan_labels<3>, grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL(k_plan_labels<4>, grid, block, lds, s, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_store_index(const TileArgs& a, bool prefix_scan, hipStream_t s)
{
    if (a.n_tiles == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_tile_count, dim3((unsigned)((a.n_tiles + 255) / 256)), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    return launch_scan(a, prefix_scan, s);
}

template <typename K>
hipError_t launch_tiles(K kernel, const TileArgs& a, int threads, size_t lds, int grid, hipStream_t s)
{
    if (a.n_tiles == 0)
        return hipSuccess;
    hipError_t e = allow_lds(kernel, lds);
    if (e != hipSuccess)
        return e;
    const unsigned g = a.persistent ? (unsigned)grid : (unsigned)a.n_tiles;
    hipLaunchKernelGGL(kernel, dim3(g), dim3(threads), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_forward(const TileArgs& a, int layout, int C, int threads, size_t lds, int grid, hipStream_t s)
{
    if (layout == 1)
        return launch_tiles(k_forward_f32, a, threads, lds, grid, s);
    if (a.dbg_coarse != nullptr || a.dbg_fine != nullptr) {
        switch (C) {
        case 1: return launch_tiles(k_forward_u8<1, true>, a, threads, lds, grid, s);
        case 2: return launch_tiles(k_forward_u8<2, true>, a, threads, lds, grid, s);
        case 3: return launch_tiles(k_forward_u8<3, true>, a, threads, lds, grid, s);
        default: return launch_tiles(k_forward_u8<4, true>, a, threads, lds, grid, s);
        }
    }
    switch (C) {
    case 1: return launch_tiles(k_forward_u8<1>, a, threads, lds, grid, s);
    case 2: return launch_tiles(k_forward_u8<2>, a, threads, lds, grid, s);
    case 3: return launch_tiles(k_forward_u8<3>, a, threads, lds, grid, s);
    default: return launch_tiles(k_forward_u8<4>, a, threads, lds, grid, s);
    }
}

hipError_t launch_reconstruct(const TileArgs& a, int layout, int C, bool paced, int threads, size_t lds, int grid,
                              hipStream_t s)
{
    if (layout == 1)
        return launch_tiles(k_reconstruct_f32, a, threads, lds, grid, s);
    if (paced && C == 3)
        return launch_tiles(k_reconstruct_u8<3, true>, a, threads, lds, grid, s);
    switch (C) {
    case 1: return launch_tiles(k_reconstruct_u8<1>, a, threads, lds, grid, s);
    case 2: return launch_tiles(k_reconstruct_u8<2>, a, threads, lds, grid, s);
    case 3: return launch_tiles(k_reconstruct_u8<3>, a, threads, lds, grid, s);
    default: return launch_tiles(k_reconstruct_u8<4>, a, threads, lds, grid, s);
    }
}

hipError_t launch_backward_reduce(const TileArgs& a, int threads, size_t lds, int grid, hipStream_t s)
{
    return launch_tiles(k_backward_reduce, a, threads, lds, grid, s);
}

hipError_t launch_backward_mirror(const TileArgs& a, int64_t n_units, int threads, hipStream_t s)
{
    hipLaunchKernelGGL(k_backward_mirror, dim3((unsigned)n_units), dim3(threads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_edge_mask(const TileArgs& a, int C, int64_t n_units, int threads, size_t lds, hipStream_t s)
{
    if (n_units == 0)
        return hipSuccess;
    const dim3 grid((unsigned)n_units), block((unsigned)threads);
    switch (C) {
    case 1: hipLaunchKernelGGL(k_edge_mask<1>, grid, block, lds, s, a); break;
    case 2: hipLaunchKernelGGL(k_edge_mask<2>, grid, block, lds, s, a); break;
    case 3: hipLaunchKernelGGL(k_edge_mask<3>, grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL(k_edge_mask<4>, grid, block, lds, s, a); break;
    }
    return hipGetLastError();
}

template <int C>
hipError_t launch_metrics_c(const TileArgs& a, bool narrow, int64_t n_units, hipStream_t s)
{
    const dim3 grid((unsigned)n_units);
    if (narrow)
        hipLaunchKernelGGL((k_metrics<C, true>), grid, dim3(MetShape<C, true>::kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((k_metrics<C, false>), grid, dim3(MetShape<C, false>::kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_metrics(const TileArgs& a, int C, bool narrow, int64_t n_units, hipStream_t s)
{
    if (n_units == 0)
        return hipSuccess;
    switch (C) {
    case 1: return launch_metrics_c<1>(a, narrow, n_units, s);
    case 2: return launch_metrics_c<2>(a, narrow, n_units, s);
    case 3: return launch_metrics_c<3>(a, narrow, n_units, s);
    default: return launch_metrics_c<4>(a, narrow, n_units, s);
    }
}

int metrics_unit_pixels(int C, bool narrow)
{
    switch (C) {
    case 1: return narrow ? MetShape<1, true>::kCw : MetShape<1, false>::kCw;
    case 2: return narrow ? MetShape<2, true>::kCw : MetShape<2, false>::kCw;
    case 3: return narrow ? MetShape<3, true>::kCw : MetShape<3, false>::kCw;
    default: return narrow ? MetShape<4, true>::kCw : MetShape<4, false>::kCw;
    }
}

hipError_t launch_metrics_reduce(const TileArgs& a, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_metrics_reduce, dim3((unsigned)a.n_frames), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

hipError_t launch_noise_advance(uint64_t* noise, int32_t n, uint64_t step, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_noise_advance, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, noise, n, step);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t* in, uint32_t* out, int64_t n, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

hipError_t occupancy_forward(int layout, int C, int threads, size_t lds, int* blocks_per_cu)
{
    const void* k;
    if (layout == 1)
        k = reinterpret_cast<const void*>(k_forward_f32);
    else if (C == 1)
        k = reinterpret_cast<const void*>(k_forward_u8<1>);
    else if (C == 2)
        k = reinterpret_cast<const void*>(k_forward_u8<2>);
    else if (C == 3)
        k = reinterpret_cast<const void*>(k_forward_u8<3>);
    else
        k = reinterpret_cast<const void*>(k_forward_u8<4>);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, threads, lds);
}

}  // namespace dppix
