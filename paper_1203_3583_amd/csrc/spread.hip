// Spreading on gfx950: the "interpolation" half of the non-uniform FFT the
// paper evaluates Eq. (9) with (Sec. 2).  Each binned point carries
// c_j = u1_j exp(i phi_j) and adds c_j psi(l_x - g_x) psi(l_y - g_y) to the w x w
// fine cells around its position g (periodic), where psi is the
// exponential-of-semicircle kernel psi(z) = exp(beta (sqrt(1 - (2z/w)^2) - 1)).
//
// One workgroup owns one tile of the fine grid.  Its bin lists every point whose
// footprint touches the tile, so the workgroup accumulates whole footprints
// into an LDS tile padded by w-1 cells on each side (no clipping), then writes
// only its own cells -- every fine cell of a tile some record reaches is written
// exactly once with plain stores, no global atomics and no separate clear of the
// fine grid.  Where the plan asks for it, a tile no record reaches is not written at
// all: the binning flags it 0 and the column pass reads its cells as zeros
// (geometries whose frequencies cover part of the fine grid leave most tiles so).
//
// Kernel values.  psi at the w cells of a footprint is a polynomial in the
// point's cell offset f (es_poly.h, FP64 Chebyshev interpolants, within 1e-7 of
// psi at w = 7); psi is even, so the cells i and w-1-i share the even and odd
// parts of one polynomial: about w + 3 FMAs per pair of cells instead of an
// exp and a sqrt per cell.
//
// Accumulation is in fixed point with LDS integer atomics: on gfx950 an LDS
// float atomic add runs about one lane at a time, the integer ones at full LDS
// rate.  A term t is made an integer by y = fma(a, k, 1.5 * 2^23): for
// |t| < 2^22 the float y lies in [2^23, 2^24), where floats are the integers,
// so the FMA rounds the exact product to the nearest integer (ties to even:
// unbiased, which matters because a bias per term would add up coherently over
// ~1e9 terms at the lowest modes) and the bit pattern of y is
// 0x4B400000 + round(t).  One 64-bit integer add of a constant then removes the
// 0x4B400000 offsets.  Per tile, M = max(|Re c_j|, |Im c_j|) over its points
// bounds every term's parts.  A tile of at most 1023 records gives no cell more
// than 1023 terms; its terms are scaled to below 2^21 (rounding step 2^-21 M)
// and packed.  Larger tiles count the footprints starting in each cell: K = w^2
// times the most of them bounds the terms any cell receives; terms are scaled
// to below 2^22 (rounding step 2^-22 M), and
//   packed (K <= 511): no cell sum leaves int32 (511 (2^22 + 1/2) < 2^31, and
//            1023 (2^21 + 1/2) < 2^31), so one 64-bit word holds Re + 2^32 Im:
//            a single ds_add_u64 adds both parts of a term (the carry of the low
//            half into the high half is undone exactly at unpacking);
//   split:   denser tiles, and grids so small that the padded tile folds onto
//            itself, keep separate 64-bit sums of Re and Im, accumulated in two
//            sweeps over the same LDS array, with 42-bit terms (term42: the
//            rounding remainder of each term kept as a second 20-bit piece).
// One rounding step for every term of a tile costs a tile whose weight sits in a
// few records (a bright point among weak ones) more than the others: their
// rounding error is set by the bright record's amplitude, not by their own.
// Such tiles (nonzero parts averaging 4 or more octaves below the largest) take
// the split sums as well.  Every decision of a tile comes from maxima and integer
// counts, and integer addition is associative, so the spread is bitwise
// deterministic and independent of the order the binning left the records in.
//
// Crowded tiles.  A tile far above the mean load of a resident workgroup (the
// binning's scan decides, from the record counts) is cut into slices of
// consecutive records, each taken by its own workgroup.  The slices share one
// scale -- the largest |u1| among all the tile's records -- and the split sums,
// write their integer sums to a partial buffer, and the last slice to finish
// adds them (exactly) and writes the tile.
//
// Bank conflicts.  A wave's 64 lanes add the same footprint offset to 64
// different points, so lane l touches base_l + const; LDS serves a quarter wave
// at a time, conflict-free when the 16 bases are distinct modulo 16 cells.
// Random bases put about three lanes on the busiest residue, and in dense
// regions whole quarter waves can hit one cell, so the records of a tile are
// counting-sorted by that residue in LDS and dealt out column-wise: lane i of a
// quarter wave takes sorted entry i * ceil(n/16) + q, so a quarter wave draws
// one entry from each sixteenth of the sorted list -- distinct residues unless
// a residue class is larger than n/16.  Only tiles with a handful of records
// skip the sort and add from registers.  Measured on gfx950, ds_add_u64 runs at
// ~10 lanes/clk/CU conflict-free and ~6 with random addresses.
//
// The fine grid is stored in panels of `panel` adjacent columns: element
// (gx, gy) lives at ((gx / panel) * nfy + gy) * panel + gx % panel, so that the
// first FFT pass reads a panel of columns as one contiguous block.
#include "asf_internal.h"
#include "es_poly.h"

namespace asf {
namespace {

constexpr int kTileXMax = 64;
constexpr int kTileYMax = 32;
constexpr int kThreads = 512;
constexpr int kBatch = 2;                 // records per thread held in registers, sorted and dealt at a time
constexpr int kChunk = kBatch * kThreads;
constexpr int kScanA = 4;                 // records per thread in flight in the first pass over a larger tile
constexpr int kWavesPerSimd = 6;          // three 512-thread workgroups per CU (LDS allows three)

template <int W>
struct TileGeom {
    static constexpr int PAD = W - 1;
    // LDS row pitch (cells), = 2 mod 16: the write-out reads 16 lanes as 8 rows x 2
    // adjacent columns, which then fall in 16 distinct bank pairs
    static constexpr int PITCH = (kTileXMax + 2 * PAD - 2 + 15) / 16 * 16 + 2;
    static constexpr int ROWS = kTileYMax + 2 * PAD;
    static constexpr int CELLS = PITCH * ROWS;
};

// psi at the w footprint cells for offset f in [-1/2, 1/2]
template <int W>
__device__ inline void es_values(float f, float (&v)[W]) {
    constexpr int D = es_poly_degree(W);
    const float u = f * f;
#pragma unroll
    for (int i = 0; i < (W + 1) / 2; ++i) {
        float e = kEsPoly[W - 2][i][D & ~1];
#pragma unroll
        for (int k = (D & ~1) - 2; k >= 0; k -= 2) e = __builtin_fmaf(e, u, kEsPoly[W - 2][i][k]);
        if (2 * i == W - 1) {
            v[i] = e;
        } else {
            constexpr int DO = (D - 1) | 1;   // highest odd power
            float o = kEsPoly[W - 2][i][DO];
#pragma unroll
            for (int k = DO - 2; k >= 1; k -= 2) o = __builtin_fmaf(o, u, kEsPoly[W - 2][i][k]);
            v[i] = __builtin_fmaf(f, o, e);
            v[W - 1 - i] = __builtin_fmaf(-f, o, e);
        }
    }
}

constexpr float kMagic = 12582912.f;             // 1.5 * 2^23
constexpr unsigned kMagicBits = 0x4B400000u;      // bit pattern of kMagic
constexpr unsigned long long kMagic1 = kMagicBits;
constexpr unsigned long long kMagic2 = ((unsigned long long)kMagicBits << 32) | kMagicBits;

// round(a k) as a 64-bit two's-complement integer, for |a k| < 2^22
__device__ inline unsigned long long term1(float a, float k) {
    return (unsigned long long)__float_as_uint(__builtin_fmaf(a, k, kMagic)) - kMagic1;
}

// round(re) + 2^32 round(im) modulo 2^64, for |re|, |im| < 2^22
__device__ inline unsigned long long term(float ar, float ai, float k) {
    const float yr = __builtin_fmaf(ar, k, kMagic);
    const float yi = __builtin_fmaf(ai, k, kMagic);
    return (((unsigned long long)__float_as_uint(yi) << 32) | __float_as_uint(yr)) - kMagic2;
}

// round(a k 2^20) as a 64-bit integer to within one unit, for |a k| < 2^22 (the
// split sums of crowded or high-dynamic-range tiles): round(a k) from the FMA above,
// then the remainder a k - round(a k) (|.| <= 1/2, formed exactly by a second FMA and
// rounded once to FP32) scaled by 2^20 and rounded the same way.  Both roundings are
// to nearest even, so the terms stay unbiased.
__device__ inline unsigned long long term42(float a, float k) {
    const float y = __builtin_fmaf(a, k, kMagic);
    const float h = y - kMagic;
    const float r = __builtin_fmaf(a, k, -h);
    const float z = __builtin_fmaf(r, 0x1p20f, kMagic);
    const long long hi = (int)(__float_as_uint(y) - kMagicBits);
    const long long lo = (int)(__float_as_uint(z) - kMagicBits);
    return (unsigned long long)(hi * (1ll << 20) + lo);
}

__device__ inline void unpack2(unsigned long long v, int &re, int &im) {
    re = (int)(unsigned)(v & 0xffffffffull);
    im = (int)(unsigned)((v - (unsigned long long)(long long)re) >> 32);
}

// padded start position of a point in this tile, or false if it does not touch it
__device__ inline bool local_start(uint32_t cell, int x0, int y0, int pad, int hix, int hiy,
                                   int nfx, int nfy, int &px, int &py) {
    px = (int)(cell & 0xffffu) - x0 + pad;
    if (px < 0) px += nfx;
    else if (px > hix) px -= nfx;
    py = (int)(cell >> 16) - y0 + pad;
    if (py < 0) py += nfy;
    else if (py > hiy) py -= nfy;
    return px >= 0 && px <= hix && py >= 0 && py <= hiy;
}

// The records of one batch: slots base + tid + k kThreads for k < kBatch, as loaded.
// Every load is issued unconditionally (slots past s1 are clamped to s1 - 1, a record
// of the same tile, and later discarded), so that all of a thread's loads are in flight
// together instead of each waiting behind a branch, and nothing here depends on their
// values: they stay in flight until load_field asks for the indices.  base < s1;
// offsets are 32-bit from the batch's uniform base.
struct Batch {
    uint2 key[kBatch];      // (cell, point index)
    float2 fr[kBatch], ph[kBatch];
};

__device__ inline void load_records(Batch &r, const Binned &b, uint32_t base, uint32_t s1) {
    const uint2 *key = b.key + base;
    const float2 *rec = reinterpret_cast<const float2 *>(b.rec + base);
    const uint32_t last = s1 - 1u - base;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
        const uint32_t s = min(threadIdx.x + k * kThreads, last);
        r.key[k] = key[s];
        r.fr[k] = rec[2u * s];
        r.ph[k] = rec[2u * s + 1u];
    }
}

// u1 at the batch's points (n >= 1, below 2^30)
__device__ inline void load_field(float2 (&u)[kBatch], const Batch &r, const float2 *__restrict__ u1, uint32_t n) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) u[k] = u1[min(r.key[k].y, n - 1u)];
}

__device__ inline float2 times_phase(float2 u, float2 ph) {
    return make_float2(u.x * ph.x - u.y * ph.y, u.x * ph.y + u.y * ph.x);
}

template <int W, int PITCH, bool PACKED>
__device__ __forceinline__ void accumulate(unsigned long long *row, float4 d) {
    float kx[W], ky[W];
    es_values<W>(d.z, kx);
    es_values<W>(d.w, ky);
#pragma unroll
    for (int jy = 0; jy < W; ++jy) {
        const float ar = d.x * ky[jy], ai = d.y * ky[jy];
#pragma unroll
        for (int i = 0; i < W; ++i)
            atomicAdd(row + jy * PITCH + i, PACKED ? term(ar, ai, kx[i]) : term42(ar, kx[i]));
    }
}

// Tiles with more records than this deal them out by start residue (see the
// file comment); the few lighter ones add their footprints straight from
// registers, where the sort would cost more than the conflicts it removes.
// (Measured on the 2048^2 cap: dealing every tile with more than 64 records
// takes the spread from 0.159 to 0.144 ms; a threshold of 1024 left most of its
// tiles conflicted.)
constexpr uint32_t kDealRecords = 64;
// Tiles of at most this many records skip the start histogram and pack their
// cells with terms below 2^21: no cell sum can leave int32.
constexpr uint32_t kFewRecords = 1023;

// The tile's own cells are read back and written out in panel order: thread tid
// handles cells tid + k nt; with nt a multiple of panel * tile_y it keeps its row
// ly and column offset lx, and successive k step col_step = nt / tile_y columns
// (col_step nfy elements in the fine grid's panel layout).
struct TileCells {
    int lx, ly, col_step;
    size_t grid, grid_step;
};

__device__ inline TileCells tile_cells(const SpreadParams &p, int x0, int y0, int nt) {
    const int tid = threadIdx.x;
    const int C = 1 << p.log_panel;
    const int c = tid & (C - 1);
    const int rest = tid >> p.log_panel;
    TileCells m;
    m.ly = rest & ((1 << p.log_tile_y) - 1);
    m.lx = ((rest >> p.log_tile_y) << p.log_panel) + c;
    m.col_step = nt >> p.log_tile_y;
    m.grid = (((size_t)((x0 + m.lx) >> p.log_panel) * p.nfy + y0 + m.ly) << p.log_panel) + c;
    m.grid_step = (size_t)m.col_step * p.nfy;
    return m;
}

// The tile's own cells as FP32 into the fine grid.
template <int W, int PITCH>
__device__ inline void write_tile(const unsigned long long *acc, float2 *__restrict__ fine,
                                  const SpreadParams &p, int x0, int y0, int ncell, int nt, bool packed,
                                  int sweep, float unscale) {
    constexpr int PAD = W - 1;
    const TileCells m = tile_cells(p, x0, y0, nt);
    const unsigned long long *src = acc + (m.ly + PAD) * PITCH + m.lx + PAD;
    float2 *dst = fine + m.grid;
    for (int k = 0; k < ncell / nt; ++k) {
        const unsigned long long v = src[k * m.col_step];
        float2 *d = dst + k * m.grid_step;
        if (packed) {
            int sr, si;
            unpack2(v, sr, si);
            *d = make_float2((float)sr * unscale, (float)si * unscale);
        } else {
            // split tiles: sweep 0 writes the real part, sweep 1 the imaginary part
            reinterpret_cast<float *>(d)[sweep] = (float)(long long)v * unscale;
        }
    }
}

// A slice of a cut tile: its integer sums (one sweep's part) in write-out order.
template <int W, int PITCH>
__device__ inline void write_partial(const unsigned long long *acc, unsigned long long *__restrict__ part,
                                     const SpreadParams &p, int ncell, int nt) {
    constexpr int PAD = W - 1;
    const TileCells m = tile_cells(p, 0, 0, nt);
    const unsigned long long *src = acc + (m.ly + PAD) * PITCH + m.lx + PAD;
    for (int k = 0; k < ncell / nt; ++k) part[k * nt + threadIdx.x] = src[k * m.col_step];
}

// The last slice of a cut tile to finish adds the slices' integer sums (exact: the
// result does not depend on how the records were dealt to slices, nor on which
// slice ends last) and writes the tile.  part: [slices][2][ncell], Re then Im.
// The tile's cells are kCombineCells per thread (ncell = 2048 = 4 nt on the grids
// that cut tiles); each step loads kCombineSlices slices' sums of all of them, 32
// loads in flight.
constexpr int kCombineCells = 4;
constexpr int kCombineSlices = 4;
static_assert(kTileXMax * kTileYMax == kCombineCells * kThreads, "cut tiles are full 64 x 32 tiles");

__device__ inline void combine_tile(const unsigned long long *part, uint32_t nsl, float2 *__restrict__ fine,
                                    const SpreadParams &p, int x0, int y0, int ncell, int nt, float unscale) {
    const TileCells m = tile_cells(p, x0, y0, nt);
    unsigned long long re[kCombineCells] = {}, im[kCombineCells] = {};
    const unsigned long long *src = part + threadIdx.x;
    for (uint32_t q = 0; q < nsl; q += kCombineSlices) {
        unsigned long long v[kCombineSlices][2][kCombineCells];
#pragma unroll
        for (int h = 0; h < kCombineSlices; ++h) {
            const uint32_t qh = min(q + h, nsl - 1u);   // past the last slice: reloaded, added as zero
#pragma unroll
            for (int k = 0; k < kCombineCells; ++k) {
                v[h][0][k] = src[(size_t)(2 * qh) * ncell + k * nt];
                v[h][1][k] = src[(size_t)(2 * qh + 1) * ncell + k * nt];
            }
        }
#pragma unroll
        for (int h = 0; h < kCombineSlices; ++h) {
            const unsigned long long keep = q + h < nsl ? ~0ull : 0ull;
#pragma unroll
            for (int k = 0; k < kCombineCells; ++k) {
                re[k] += v[h][0][k] & keep;
                im[k] += v[h][1][k] & keep;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kCombineCells; ++k)
        fine[m.grid + k * m.grid_step] = make_float2((float)(long long)re[k] * unscale, (float)(long long)im[k] * unscale);
}

// Wave-wide reductions by lane permutations on the vector ALU (DPP): within each
// row of 16 lanes, exchanges with lane ^ 1 and lane ^ 2, then the half-row and row
// mirrors leave every lane with its row's result; four lane reads combine the
// rows.  A few cycles per step, where shuffles routed through the LDS crossbar
// take a round trip each.
__device__ inline unsigned dpp_row_max(unsigned v) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad [1,0,3,2]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad [2,3,0,1]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row half mirror
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row mirror
    return v;
}

__device__ inline unsigned dpp_row_sum(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);
    return v;
}

// inclusive prefix sum within each row of 16 lanes (row shifts by 1, 2, 4, 8;
// lanes shifted in from outside the row read 0)
__device__ inline unsigned dpp_row_prefix(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
    return v;
}

// (the whole wave must be active; the result is uniform)
__device__ inline unsigned wave_max(unsigned v) {
    v = dpp_row_max(v);
    return max(max((unsigned)__builtin_amdgcn_readlane((int)v, 0), (unsigned)__builtin_amdgcn_readlane((int)v, 16)),
               max((unsigned)__builtin_amdgcn_readlane((int)v, 32), (unsigned)__builtin_amdgcn_readlane((int)v, 48)));
}

__device__ inline unsigned wave_sum(unsigned v) {
    v = dpp_row_sum(v);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 0) + (unsigned)__builtin_amdgcn_readlane((int)v, 16) +
           (unsigned)__builtin_amdgcn_readlane((int)v, 32) + (unsigned)__builtin_amdgcn_readlane((int)v, 48);
}

// A tile whose weight sits in a few of its records: the exponents of its nonzero
// parts (max(|Re c|, |Im c|) per record) average 4 or more below the largest one,
// E.  The packed sums round every term to 2^-21 M (or 2^-22 M), M the largest part,
// which costs the other records a relative error set by M rather than by their own
// size: about 1.5e-6 for a tile of random phases and amplitudes, 2e-5 for one
// bright point among 500 points 1e4 times weaker.  Such tiles take the split sums
// with 42-bit terms.  (Zero records add exact zeros and do not count.)  The
// statistic is a sum of integer exponents, so this decision, like the tile's
// others (maxima and counts), does not depend on the order the binning left the
// records in.
__device__ inline bool high_dynamic_range(unsigned ebig, unsigned long long nnz, unsigned long long esum) {
    return nnz > 0ull && ebig * nnz - esum >= 4ull * nnz;
}

// Exponent bound of the terms of a split tile: each record adds at most one term
// to a cell, so a cell sum of nrec terms below 2^(emax + 20) (term42) stays below
// 2^62 when emax + 20 + log2(nrec) <= 62.
__device__ inline int split_emax(uint32_t nrec) {
    int lg = 0;
    while (lg < 32 && (1u << lg) < nrec) ++lg;
    return min(22, 42 - lg);
}

// What a workgroup knows of its tile (uniform), and its LDS.  Its three ways through a
// tile -- small (one batch of records, kept in registers), large (several batches) and
// cut_slice -- are separate code with packed and split sums separate again: in one body
// with the next batch fetched ahead 29 to 49 of the 80 registers that six waves per SIMD
// leave were spilled, the batch in flight among them, which waits for it.  Apart, 20 are
// at w = 7 (8 to 16 below, 37 and 60 at w = 8 and 9), some of them reloaded in the batch
// loops; without a batch fetched ahead none were from w = 3 on, and the kernel was slower.
// Bound by latency (the chain of dependent loads per tile: slots, keys, field) and by the
// 49 LDS atomics per record, which the next batch's loads overlap: 2048^2 cap (8192 small
// tiles) 126.5 -> 114.8 us, 4096^2 relief (large) 501 -> 474, 1024^2 at w = 9 with split
// sums 84.3 -> 48.3; since the tiles are taken in order of size (the binning's tile_order)
// 105, 342 and 40 us.  The cap's records, field and cells are 300 MB, 59 us at the rate of
// a large copy.
template <int W>
struct Tile {
    using G = TileGeom<W>;
    static constexpr int PAD = G::PAD, PITCH = G::PITCH;
    static constexpr int SWMAX = (kTileXMax + PAD) * (kTileYMax + PAD);
    static constexpr int SDAT = (kChunk + 16) > (SWMAX + 3) / 4 ? (kChunk + 16) : (SWMAX + 3) / 4;

    struct Lds {
        __align__(16) unsigned long long acc[G::CELLS];
        __align__(16) float4 sdat[SDAT];   // dealt records (Re c, Im c, fx, fy); before that the start histogram
        int sbase[kChunk + 16];            // their padded start cell
        unsigned rcount[16];               // records per start residue
        unsigned sbig, smost;              // block maxima
        unsigned long long snnz, sesum;    // nonzero records, sum of their exponents
        unsigned slast;
    };

    const SpreadParams &p;
    Lds &l;
    const float2 *u1;
    float2 *fine;
    uint32_t n;            // source points
    int x0, y0;            // first cell
    bool fold_x, fold_y;   // the grid is narrower than the padded tile

    __device__ __forceinline__ int swx() const { return (1 << p.log_tile_x) + PAD; }   // start positions per axis
    __device__ __forceinline__ int swy() const { return (1 << p.log_tile_y) + PAD; }
    __device__ __forceinline__ int ncell() const { return 1 << (p.log_tile_x + p.log_tile_y); }
    __device__ __forceinline__ int *starts() const { return reinterpret_cast<int *>(l.sdat); }

    __device__ __forceinline__ void clear_acc() const {
        uint4 *a4 = reinterpret_cast<uint4 *>(l.acc);
        for (int i = threadIdx.x; i < G::CELLS / 2; i += kThreads) a4[i] = make_uint4(0u, 0u, 0u, 0u);
    }

    __device__ __forceinline__ void clear_lds(bool count_starts) const {
        clear_acc();
        if (count_starts)
            for (int i = threadIdx.x; i < swx() * swy(); i += kThreads) starts()[i] = 0;
        if (threadIdx.x < 16) l.rcount[threadIdx.x] = 0u;
        if (threadIdx.x == 0) {
            l.sbig = l.smost = 0u;
            l.snnz = l.sesum = 0ull;
        }
    }

    // padded start position of a record (if it is one), or false where it does not touch the tile
    __device__ __forceinline__ bool start_of(bool in, uint2 key, int &px, int &py) const {
        return in && key.y < n && local_start(key.x, x0, y0, PAD, swx() - 1, swy() - 1, p.nfx, p.nfy, px, py);
    }

    // This thread's share of the tile's statistics: the largest |Re c| or |Im c|, the
    // nonzero parts and the sum of their exponents, and (count_starts) the footprint
    // starts per position.
    struct Tally {
        float big = 0.f;
        unsigned nnz = 0u, esum = 0u;
    };
    __device__ __forceinline__ void tally(Tally &s, float2 c, int px, int py, bool count_starts) const {
        const float part = fmaxf(fabsf(c.x), fabsf(c.y));
        s.big = fmaxf(s.big, part);
        // branch-free: a zero part adds exponent 0 and no count
        s.nnz += part > 0.f ? 1u : 0u;
        s.esum += __float_as_uint(part) >> 23;
        if (count_starts) atomicAdd(&starts()[py * swx() + px], 1);
    }

    // block maximum (non-negative floats order like their bit patterns) and the
    // exponent statistics: wave sums in 32 bits (a wave holds an eighth of the
    // tile's records; tiles of 2^24 or more records skip the statistic), 64-bit
    // sums across the block
    __device__ __forceinline__ void reduce(const Tally &s, bool exponents) const {
        const unsigned wbig = wave_max(__float_as_uint(s.big));
        const unsigned wnnz = wave_sum(s.nnz), wesum = wave_sum(s.esum);
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&l.sbig, wbig);
            if (exponents && wnnz) {
                atomicAdd(&l.snnz, (unsigned long long)wnnz);
                atomicAdd(&l.sesum, (unsigned long long)wesum);
            }
        }
        __syncthreads();   // sbig, snnz, sesum and starts[] complete
    }

    // Most footprint starts in one cell (every thread calls this).
    __device__ __forceinline__ unsigned most_starts() const {
        unsigned most = 0u;
        for (int i = threadIdx.x; i < swx() * swy(); i += kThreads) most = max(most, (unsigned)starts()[i]);
        most = wave_max(most);
        if ((threadIdx.x & 63) == 0) atomicMax(&l.smost, most);
        __syncthreads();
        return l.smost;
    }

    // Exponent of the scale that brings the tile's terms below 2^emax.
    __device__ __forceinline__ int scale_exponent(int emax) const {
        const float big = __uint_as_float(l.sbig);
        int e = 0;
        if (big > 0.f) {
            int em;
            frexpf(big * (1.f + 0x1p-18f), &em);   // margin for rounding in c and psi
            e = emax - em;
        }
        return max(-120, min(e, 120));
    }

    // One batch's records, each (Re c, Im c, fx, fy) with its padded start cell (-1:
    // none), sorted by start residue and dealt (see the file comment): returns how many
    // records there are; slot s of the deal holds one where dealt(s, total).
    __device__ __forceinline__ unsigned deal(const float4 (&rec)[kBatch], const int (&rb)[kBatch]) const {
        const int lane = threadIdx.x & 63;
        int rres[kBatch];
        unsigned rrank[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            rres[q] = rb[q] & 15;
            rrank[q] = rb[q] >= 0 ? atomicAdd(&l.rcount[rres[q]], 1u) : 0u;   // rank within class
        }
        __syncthreads();   // residue counts complete
        // exclusive prefix of the 16 counts, held by lanes 0..15 of every wave
        const unsigned cnt = lane < 16 ? l.rcount[lane] : 0u;
        const unsigned inc = dpp_row_prefix(cnt);
        const unsigned total = (unsigned)__builtin_amdgcn_readlane((int)inc, 15);
        const unsigned excl = inc - cnt;
        const unsigned n16 = (total + 15u) >> 4;
        const float inv16 = n16 ? 1.f / (float)n16 : 0.f;
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            // sorted position, then the column-wise deal: position srt goes
            // to slot (srt mod n16) * 16 + srt / n16 (the quotient is exact:
            // the float estimate of (srt + 1/2) / n16 is >= 1/128 from an
            // integer)
            const unsigned srt = rrank[q] + __shfl(excl, rres[q]);
            if (rb[q] < 0) continue;
            const unsigned quo = (unsigned)(((float)srt + 0.5f) * inv16);
            const unsigned slot = (srt - quo * n16) * 16u + quo;
            l.sdat[slot] = rec[q];
            l.sbase[slot] = rb[q];
        }
        __syncthreads();   // records dealt; counts read by everyone
        if (threadIdx.x < 16) l.rcount[threadIdx.x] = 0u;
        return total;
    }

    // Add the footprint of deal slot s.
    template <bool PACKED>
    __device__ __forceinline__ void add_slot(unsigned s, unsigned total) const {
        const unsigned n16 = (total + 15u) >> 4;
        if ((s >> 4) < n16 && (s & 15u) * n16 + (s >> 4) < total)
            accumulate<W, PITCH, PACKED>(l.acc + l.sbase[s], l.sdat[s]);
    }

    // The tile's own cells into the fine grid (sweep's part of them unless packed).
    __device__ __forceinline__ void write_out(bool packed, int sweep, float unscale) const {
        if (!fold_x && !fold_y) {
            write_tile<W, PITCH>(l.acc, fine, p, x0, y0, ncell(), kThreads, packed, sweep, unscale);
            return;
        }
        // grids narrower than the padded tile: fold the wrapped halo back in
        const int tsx = 1 << p.log_tile_x, tsy = 1 << p.log_tile_y, C = 1 << p.log_panel;
        const int ext_x = tsx + 2 * PAD, ext_y = tsy + 2 * PAD;
        for (int i = threadIdx.x; i < tsx * tsy; i += kThreads) {
            const int c = i & (C - 1);
            const int rest = i >> p.log_panel;
            const int ly = rest & (tsy - 1);
            const int lx = ((rest >> p.log_tile_y) << p.log_panel) + c;
            unsigned long long v = 0ull;
            for (int oy = ly + PAD - 2 * p.nfy; oy < ext_y; oy += p.nfy) {
                if (oy < 0 || (!fold_y && oy != ly + PAD)) continue;
                for (int ox = lx + PAD - 2 * p.nfx; ox < ext_x; ox += p.nfx) {
                    if (ox < 0 || (!fold_x && ox != lx + PAD)) continue;
                    v += l.acc[oy * PITCH + ox];
                }
            }
            float2 *dst = fine + ((((size_t)((x0 + lx) >> p.log_panel) * p.nfy + y0 + ly) << p.log_panel) + c);
            if (packed) {
                int sr, si;
                unpack2(v, sr, si);
                *dst = make_float2((float)sr * unscale, (float)si * unscale);
            } else {
                reinterpret_cast<float *>(dst)[sweep] = (float)(long long)v * unscale;
            }
        }
    }

    // A tile of at most one batch of records, not cut: they stay in registers throughout.
    __device__ __forceinline__ void small(const Binned &b, uint32_t s0, uint32_t s1) const {
        const uint32_t nrec = s1 - s0;
        // a tile of few records needs no start histogram: no cell receives more than
        // nrec terms (unless the grid folds the padded tile onto itself: split sums)
        const bool few = nrec <= kFewRecords && !fold_x && !fold_y;
        // the records' loads are in flight while the LDS is cleared, the field's while
        // the workgroup waits for that
        Batch r;
        float2 uf[kBatch];
        if (nrec) load_records(r, b, s0, s1);
        clear_lds(!few);
        if (nrec) load_field(uf, r, u1, n);
        __syncthreads();
        float4 rec[kBatch];   // Re c, Im c, offsets
        int rb[kBatch];
        Tally s;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            int px, py;
            rb[k] = -1;
            rec[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (nrec && start_of(threadIdx.x + k * kThreads < nrec, r.key[k], px, py)) {
                rb[k] = py * PITCH + px;
                const float2 c = times_phase(uf[k], r.ph[k]);
                rec[k] = make_float4(c.x, c.y, r.fr[k].x, r.fr[k].y);
                tally(s, c, px, py, !few);
            }
        }
        reduce(s, true);
        bool packed = true;   // kFewRecords (2^21 + 1/2) < 2^31
        int emax = 21;        // terms are bounded by 2^emax
        if (!few) {
            // 511 (2^22 + 1/2) < 2^31; grids folding the tile onto itself sum several cells
            packed = most_starts() * (unsigned)(W * W) <= 511u && !fold_x && !fold_y;
            emax = 22;
        }
        // a few records dominating the tile: the others would be rounded on the dominant
        // ones' grid, so the tile takes the split sums with 42-bit terms
        if (high_dynamic_range(l.sbig >> 23, l.snnz, l.sesum)) packed = false;
        if (!packed) emax = split_emax(nrec);
        const int e = scale_exponent(emax);
        const float scale = ldexpf(1.f, e);
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            rec[k].x *= scale;
            rec[k].y *= scale;
        }
        if (packed) {
            add_batch<true>(nrec, rec, rb);
            __syncthreads();
            write_out(true, 0, ldexpf(1.f, -e));
            return;
        }
        // two sweeps, real then imaginary parts; split sums carry 20 more fractional bits
#pragma unroll 1
        for (int sweep = 0; sweep < 2; ++sweep) {
            if (sweep) {
                __syncthreads();
                clear_acc();
#pragma unroll
                for (int k = 0; k < kBatch; ++k) rec[k].x = rec[k].y;
                __syncthreads();
            }
            add_batch<false>(nrec, rec, rb);
            __syncthreads();
            write_out(false, sweep, ldexpf(1.f, -e - 20));
        }
    }

    // One batch's footprints (scaled records): dealt, or straight from registers where
    // there are few (at most one per thread).
    template <bool PACKED>
    __device__ __forceinline__ void add_batch(uint32_t nrec, const float4 (&rec)[kBatch], const int (&rb)[kBatch]) const {
        static_assert(kDealRecords <= kThreads, "one record per thread below");
        if (nrec <= kDealRecords) {
            if (rb[0] >= 0) accumulate<W, PITCH, PACKED>(l.acc + rb[0], rec[0]);
            return;
        }
        const unsigned total = deal(rec, rb);
#pragma unroll 1
        for (int q = 0; q < kBatch; ++q) add_slot<PACKED>(threadIdx.x + q * kThreads, total);
    }

    // The batches of a larger tile or of a long slice, one after the other: each batch's
    // records are fetched while the one before is accumulated (its keys, offsets and
    // phases before the first half of the accumulation, its field, which needs the keys,
    // before the second).  r and uf hold the first batch, in flight.
    template <bool PACKED>
    __device__ __forceinline__ void add_batches(const Binned &b, uint32_t s0, uint32_t s1, Batch &r,
                                                float2 (&uf)[kBatch], float scale, int sweep) const {
        for (uint32_t at = s0; at < s1; at += kChunk) {
            float4 rec[kBatch];
            int rb[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                int px, py;
                const float2 c = times_phase(uf[k], r.ph[k]);
                const float cr = c.x * scale, ci = c.y * scale;
                rec[k] = make_float4(PACKED || sweep == 0 ? cr : ci, ci, r.fr[k].x, r.fr[k].y);
                rb[k] = start_of(at + threadIdx.x + k * kThreads < s1, r.key[k], px, py) ? py * PITCH + px : -1;
            }
            const unsigned total = deal(rec, rb);
            const uint32_t next = at + kChunk;
            if (next < s1) load_records(r, b, next, s1);
            add_slot<PACKED>(threadIdx.x, total);
            if (next < s1) load_field(uf, r, u1, n);
            add_slot<PACKED>(threadIdx.x + kThreads, total);
            __syncthreads();   // staging reused by the next batch
        }
    }

    // A tile of more than one batch of records: a first pass over them for the scale and
    // the footprint starts, then the batches.
    __device__ __forceinline__ void large(const Binned &b, uint32_t s0, uint32_t s1) const {
        clear_lds(true);
        __syncthreads();
        Tally s;
        // keys, phases and field only, kScanA records per thread in flight
        for (uint32_t base = s0; base < s1; base += kScanA * kThreads) {
            const uint2 *key = b.key + base;
            const float2 *rec = reinterpret_cast<const float2 *>(b.rec + base);
            const uint32_t last = s1 - 1u - base;
            uint2 kv[kScanA];
            float2 ph[kScanA], u[kScanA];
#pragma unroll
            for (int k = 0; k < kScanA; ++k) {
                const uint32_t i = min(threadIdx.x + k * kThreads, last);
                kv[k] = key[i];
                ph[k] = rec[2u * i + 1u];
            }
#pragma unroll
            for (int k = 0; k < kScanA; ++k) u[k] = u1[min(kv[k].y, n - 1u)];
#pragma unroll
            for (int k = 0; k < kScanA; ++k) {
                int px, py;
                if (start_of(threadIdx.x + k * kThreads <= last, kv[k], px, py))
                    tally(s, times_phase(u[k], ph[k]), px, py, true);
            }
        }
        // the first batch again, in flight while the workgroup settles the scale
        Batch r;
        float2 uf[kBatch];
        load_records(r, b, s0, s1);
        load_field(uf, r, u1, n);
        reduce(s, true);
        const bool packed = most_starts() * (unsigned)(W * W) <= 511u && !fold_x && !fold_y &&
                            s1 - s0 < (1u << 24) && !high_dynamic_range(l.sbig >> 23, l.snnz, l.sesum);
        const int e = scale_exponent(packed ? 22 : split_emax(s1 - s0));
        const float scale = ldexpf(1.f, e);
        if (packed) {
            add_batches<true>(b, s0, s1, r, uf, scale, 0);
            write_out(true, 0, ldexpf(1.f, -e));
            return;
        }
#pragma unroll 1
        for (int sweep = 0; sweep < 2; ++sweep) {
            if (sweep) next_sweep(b, s0, s1, r, uf);
            add_batches<false>(b, s0, s1, r, uf, scale, sweep);
            write_out(false, sweep, ldexpf(1.f, -e - 20));
        }
    }

    // Between the sweeps of split sums: clear them, fetch the first batch again.
    __device__ __forceinline__ void next_sweep(const Binned &b, uint32_t s0, uint32_t s1, Batch &r,
                                               float2 (&uf)[kBatch]) const {
        __syncthreads();
        clear_acc();
        uint32_t from = s0;
        asm volatile("" : "+s"(from));   // its addresses are formed here, not kept from the first load
        load_records(r, b, from, s1);
        load_field(uf, r, u1, n);
        __syncthreads();
    }

    // Slice [s0, s1) of cut tile t.  The slices of a tile all take the split sums with
    // 42-bit terms at one scale, set by the largest |u1| among all the tile's records
    // (|exp(i phi)| = 1 bounds |Re c| and |Im c| by it): every term is then the same
    // integer whichever slice adds it, and the slices' sums add up exactly to the whole
    // tile's.  A slice of one batch (the usual length) keeps its records in registers,
    // loaded while the pass over the whole tile runs.
    __device__ __forceinline__ void cut_slice(const Binned &b, int t, uint32_t s0, uint32_t s1, uint32_t slice,
                                              uint32_t nsl, uint32_t slot) const {
        const bool one = s1 - s0 <= (uint32_t)kChunk;
        Batch r;
        float2 uf[kBatch];
        if (s0 < s1) load_records(r, b, s0, s1);   // (a slice may be empty)
        clear_lds(false);
        if (s0 < s1) load_field(uf, r, u1, n);
        __syncthreads();
        float4 rec[kBatch];
        int rb[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            int px, py;
            rb[k] = -1;
            rec[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (start_of(s0 + threadIdx.x + k * kThreads < s1, r.key[k], px, py)) {
                rb[k] = py * PITCH + px;
                const float2 c = times_phase(uf[k], r.ph[k]);
                rec[k] = make_float4(c.x, c.y, r.fr[k].x, r.fr[k].y);
            }
        }
        Tally s;
        uint32_t a0, a1;
        tile_slots(b, t, a0, a1);
        constexpr int kScan = 8;   // records per thread in flight
        for (uint32_t i = a0 + threadIdx.x; i < a1; i += kScan * kThreads) {
            uint32_t j[kScan];
            float2 u[kScan];
#pragma unroll
            for (int q = 0; q < kScan; ++q) j[q] = b.key[min(i + q * kThreads, a1 - 1u)].y;
#pragma unroll
            for (int q = 0; q < kScan; ++q) u[q] = u1[min(j[q], n - 1u)];
#pragma unroll
            for (int q = 0; q < kScan; ++q)
                if (i + q * kThreads < a1 && j[q] < n) s.big = fmaxf(s.big, sqrtf(u[q].x * u[q].x + u[q].y * u[q].y));
        }
        reduce(s, false);
        const int e = scale_exponent(split_emax(a1 - a0));
        const float scale = ldexpf(1.f, e), unscale = ldexpf(1.f, -e - 20);
        // slices are only made on grids that do not fold
        unsigned long long *part = b.partial + (size_t)(2 * (slot + slice)) * ncell();
        if (one) {
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                rec[k].x *= scale;
                rec[k].y *= scale;
            }
#pragma unroll 1
            for (int sweep = 0; sweep < 2; ++sweep) {
                if (sweep) {
                    __syncthreads();
                    clear_acc();
#pragma unroll
                    for (int k = 0; k < kBatch; ++k) rec[k].x = rec[k].y;
                    __syncthreads();
                }
                add_batch<false>(s1 - s0, rec, rb);
                __syncthreads();
                write_partial<W, PITCH>(l.acc, part + (size_t)sweep * ncell(), p, ncell(), kThreads);
            }
        } else {
            load_records(r, b, s0, s1);
            load_field(uf, r, u1, n);
#pragma unroll 1
            for (int sweep = 0; sweep < 2; ++sweep) {
                if (sweep) next_sweep(b, s0, s1, r, uf);
                add_batches<false>(b, s0, s1, r, uf, scale, sweep);
                write_partial<W, PITCH>(l.acc, part + (size_t)sweep * ncell(), p, ncell(), kThreads);
            }
        }
        // partial sums stored: make them visible device-wide, then count the slice in;
        // the last of the tile's slices (whichever it is) reads all partials back
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) l.slast = atomicAdd(&b.combine[slot], 1u) == nsl - 1;
        __syncthreads();
        if (l.slast) {
            __threadfence();
            combine_tile(b.partial + (size_t)2 * slot * ncell(), nsl, fine, p, x0, y0, ncell(), kThreads, unscale);
            if (threadIdx.x == 0) b.combine[slot] = 0u;   // ready for the next launch
        }
    }
};

template <int W>
__global__ void __launch_bounds__(kThreads, kWavesPerSimd) spread_kernel(SpreadParams p, Binned b,
                                                          const float2 *__restrict__ u1,
                                                          float2 *__restrict__ fine) {
    __shared__ typename Tile<W>::Lds lds;
    // this workgroup's tile, and its slice of the records if the tile is cut
    int t;
    uint32_t slice, nsl, slot, s0, s1;
    // (tiles no record reaches may be left unwritten: the column pass then reads their cells
    // as zeros)
    if (!work_item(b, p.ntx * p.nty, p.ordered, p.skip_dead, t, slice, nsl, slot, s0, s1)) return;
    constexpr int PAD = TileGeom<W>::PAD;
    const int tsx = 1 << p.log_tile_x, tsy = 1 << p.log_tile_y;
    const int ty = t >> p.log_ntx, tx = t & ((1 << p.log_ntx) - 1);
    const Tile<W> tile{p, lds, u1, fine, (uint32_t)p.n, tx << p.log_tile_x, ty << p.log_tile_y,
                       p.nfx < tsx + 2 * PAD, p.nfy < tsy + 2 * PAD};
    if (nsl > 1) tile.cut_slice(b, t, s0, s1, slice, nsl, slot);
    else if (s1 - s0 <= (uint32_t)kChunk) tile.small(b, s0, s1);
    else tile.large(b, s0, s1);
}

template <int W>
hipError_t launch_w(const SpreadParams &p, const Binned &b, const float2 *u1, float2 *fine,
                    hipStream_t s) {
    const int groups = p.ntx * p.nty + (p.split ? kSplitSlots : 0);
    hipLaunchKernelGGL(spread_kernel<W>, dim3(groups), dim3(kThreads), 0, s, p, b, u1, fine);
    return hipGetLastError();
}

// Interpolation, the adjoint of spreading (the type-2 direction): every point
// gathers its w x w footprint of the fine grid with the same kernel weights,
//   g_j = conj(exp(i phi_j)) sum_l psi(l_x - g_x) psi(l_y - g_y) F[l],
// the conjugate pre-phase being the adjoint of the pre-phase multiply.  One
// workgroup per tile copies into LDS the cells the footprints of the tile's own
// points reach (the tile plus w-1 cells right and below, periodic).  A point is
// handled in the tile that holds its first footprint cell and skipped in the
// other bins that list it, so each point is written once, with a plain store:
// no atomics, and FP32 sums in registers.  Only footprint cells enter the sums:
// every one lies in a tile whose bin lists the point, so cells of tiles no record
// reaches (which the column pass may leave unwritten) are copied but never used.
constexpr int kInterpThreads = 256;

template <int W>
__global__ void __launch_bounds__(kInterpThreads) interp_kernel(SpreadParams p, Binned b,
                                                                const float2 *__restrict__ fine,
                                                                float2 *__restrict__ g1) {
    constexpr int RP = kTileXMax + W - 1;   // LDS row pitch (cells)
    __shared__ float2 reg[(kTileYMax + W - 1) * RP];
    // this workgroup's tile, and its slice of the records if the tile is cut (no
    // combining: every point is written by the one workgroup that holds its record)
    int t;
    uint32_t slice, nsl, slot, s0, s1;
    // (without points to gather for, the region is not needed)
    if (!work_item(b, p.ntx * p.nty, p.ordered, true, t, slice, nsl, slot, s0, s1) || s0 == s1) return;
    const int tsx = 1 << p.log_tile_x, tsy = 1 << p.log_tile_y;
    const int rx = tsx + W - 1, ry = tsy + W - 1;
    const int ty = t >> p.log_ntx, tx = t & ((1 << p.log_ntx) - 1);
    const int x0 = tx << p.log_tile_x, y0 = ty << p.log_tile_y;
    constexpr int nt = kInterpThreads;
    const int tid = threadIdx.x;
    // copy the region in the fine grid's panel order (C adjacent columns per row,
    // rows of a panel contiguous), so consecutive lanes read consecutive elements
    const int C = 1 << p.log_panel;
    const int rxp = (rx + C - 1) & ~(C - 1);
    const float inv_ry = 1.f / (float)ry;
    // The whole region's loads in flight before their LDS writes (rounded up to panels it may
    // take a second turn): the copy is one wait instead of two.  2048^2 cap: six per thread
    // 86.4 us, eight 85.0, all eleven 82.2 (66 are its bytes); 1024^2 at w = 9 33.9 and 33.1.
    constexpr int kRegionLoads = (RP * (kTileYMax + W - 1) + nt - 1) / nt;
    for (int i0 = tid; i0 < rxp * ry; i0 += kRegionLoads * nt) {
        float2 v[kRegionLoads];
        int at[kRegionLoads];
#pragma unroll
        for (int q = 0; q < kRegionLoads; ++q) {
            const int i = i0 + q * nt;
            const int c = i & (C - 1);
            const int rest = i >> p.log_panel;
            const int qx = (int)(((float)rest + 0.5f) * inv_ry);   // rest / ry, exact for rest < 2^20
            const int yy = rest - qx * ry;
            const int xx = qx * C + c;
            at[q] = (i < rxp * ry && xx < rx) ? yy * RP + xx : -1;
            int gx = x0 + xx, gy = y0 + yy;
            if (gx >= p.nfx) gx -= p.nfx;
            if (gy >= p.nfy) gy -= p.nfy;
            v[q] = at[q] >= 0 ? fine[(((size_t)(gx >> p.log_panel) * p.nfy + gy) << p.log_panel) + (gx & (C - 1))]
                              : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int q = 0; q < kRegionLoads; ++q)
            if (at[q] >= 0) reg[at[q]] = v[q];
    }
    __syncthreads();
    // two records per thread and iteration: their key and record loads all go out
    // together (slots past s1 clamped to s1 - 1 and discarded)
    for (uint32_t sb = s0 + tid; sb < s1; sb += 2 * nt) {
        uint2 kv[2];   // (cell, point index)
        float4 rv[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t s = min(sb + q * nt, s1 - 1u);
            kv[q] = b.key[s];
            rv[q] = b.rec[s];
        }
        bool home[2];
        int px[2], py[2];
        uint32_t j[2];
        float2 fr[2], ph[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            px[q] = (int)(kv[q].x & 0xffffu) - x0;
            py[q] = (int)(kv[q].x >> 16) - y0;
            // a point is handled in its home tile only (and past s1 nowhere)
            home[q] = sb + q * nt < s1 && px[q] >= 0 && px[q] < tsx && py[q] >= 0 && py[q] < tsy;
            j[q] = home[q] ? kv[q].y : 0u;
            fr[q] = make_float2(rv[q].x, rv[q].y);
            ph[q] = make_float2(rv[q].z, rv[q].w);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (!home[q]) continue;
            float kx[W], ky[W];
            es_values<W>(fr[q].x, kx);
            es_values<W>(fr[q].y, ky);
            const float2 *row = reg + py[q] * RP + px[q];
            float ar = 0.f, ai = 0.f;
#pragma unroll
            for (int jy = 0; jy < W; ++jy) {
                float sr = 0.f, si = 0.f;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const float2 v = row[jy * RP + i];
                    sr = __builtin_fmaf(kx[i], v.x, sr);
                    si = __builtin_fmaf(kx[i], v.y, si);
                }
                ar = __builtin_fmaf(ky[jy], sr, ar);
                ai = __builtin_fmaf(ky[jy], si, ai);
            }
            // times conj(exp(i phi))
            g1[j[q]] = make_float2(ar * ph[q].x + ai * ph[q].y, ai * ph[q].x - ar * ph[q].y);
        }
    }
}

template <int W>
hipError_t launch_interp_w(const SpreadParams &p, const Binned &b, const float2 *fine, float2 *g1,
                           hipStream_t s) {
    const int groups = p.ntx * p.nty + (p.split ? kSplitSlots : 0);
    hipLaunchKernelGGL(interp_kernel<W>, dim3(groups), dim3(kInterpThreads), 0, s, p, b, fine, g1);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_spread(const SpreadParams &p, const Binned &b, const float2 *u1, float2 *fine,
                         hipStream_t s) {
    if ((1 << p.log_tile_x) > kTileXMax || (1 << p.log_tile_y) > kTileYMax) return hipErrorInvalidValue;
    if ((1 << p.log_tile_x) % 16 != 0) return hipErrorInvalidValue;   // start residues need 16 | tile_x
    switch (p.w) {
        case 2: return launch_w<2>(p, b, u1, fine, s);
        case 3: return launch_w<3>(p, b, u1, fine, s);
        case 4: return launch_w<4>(p, b, u1, fine, s);
        case 5: return launch_w<5>(p, b, u1, fine, s);
        case 6: return launch_w<6>(p, b, u1, fine, s);
        case 7: return launch_w<7>(p, b, u1, fine, s);
        case 8: return launch_w<8>(p, b, u1, fine, s);
        case 9: return launch_w<9>(p, b, u1, fine, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_interp(const SpreadParams &p, const Binned &b, const float2 *fine, float2 *g1,
                         hipStream_t s) {
    if ((1 << p.log_tile_x) > kTileXMax || (1 << p.log_tile_y) > kTileYMax) return hipErrorInvalidValue;
    switch (p.w) {
        case 2: return launch_interp_w<2>(p, b, fine, g1, s);
        case 3: return launch_interp_w<3>(p, b, fine, g1, s);
        case 4: return launch_interp_w<4>(p, b, fine, g1, s);
        case 5: return launch_interp_w<5>(p, b, fine, g1, s);
        case 6: return launch_interp_w<6>(p, b, fine, g1, s);
        case 7: return launch_interp_w<7>(p, b, fine, g1, s);
        case 8: return launch_interp_w<8>(p, b, fine, g1, s);
        case 9: return launch_interp_w<9>(p, b, fine, g1, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace asf
