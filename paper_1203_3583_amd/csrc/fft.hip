// Uniform FFT on gfx950: the "uniform FFT" half of the non-uniform FFT the
// paper evaluates Eq. (9) with (Sec. 2), plus the deconvolution, crop and
// destination phase of Eq. (8) fused into the last pass.
//
// A 2D forward DFT (exp(-i) sign) of the nfx x nfy fine grid is done in two
// passes, each pruned to the modes the destination grid keeps:
//   pass 1: every fine-grid column (length nfy; where the plan leaves the tiles no
//           record reaches unwritten, their cells read as zeros without a load, and
//           a panel of columns with no such tile writes zeros without a transform),
//           keep the my centred modes,
//           write them to mid in the fine grid's panel layout (panels of C
//           adjacent columns, element (lx, ky) at ((lx / C) my + ky) C + lx % C),
//           so that each workgroup writes one contiguous block;
//   pass 2: every mid row (length nfx), gathered from the panels (C elements at
//           a time; the 16 / C rows that share a 128-byte line run on one XCD,
//           whose L2 serves the line to all of them), keep the mx centred
//           modes, multiply by
//           Dx[ix] Dy[iy] (1/psi-hat, the destination chirp of Eq. (6)/(7) and
//           the prefactor exp(i k z0)/(i lambda z0)) and write u2[iy][ix].
// The transforms of a workgroup are the engine's (fft_engine.h).
#include "asf_internal.h"
#include "fft_engine.h"

namespace asf {
namespace {

// With flags (tiles no record reaches, left unwritten): the flags of the tile column
// holding fine-grid column x0, one byte per tile row, into LDS.  Returns whether
// flags are in use.
__device__ __forceinline__ bool live_rows(const LiveTiles &lt, int x0, uint8_t *lrow) {
    if (!lt.flag) return false;
    const uint8_t *col = lt.flag + (x0 >> lt.log_tile_x);
    for (int i = threadIdx.x; i < lt.nty; i += blockDim.x) lrow[i] = col[(size_t)i * lt.ntx];
    __syncthreads();
    return true;
}

// With flags: whether the tile column holding fine-grid column x0 has a flagged tile
// (the same answer in every thread).  The columns of one with none are zeros: the
// column passes skip them, and the row passes neither read nor write them in mid.
__device__ __forceinline__ bool column_needed(const LiveTiles &lt, int x0) {
    return !lt.flag || lt.col[x0 >> lt.log_tile_x] != 0;
}

// With flags: the tile columns' flags, one byte per tile column, into LDS.  Returns
// whether flags are in use.
__device__ __forceinline__ bool live_cols(const LiveTiles &lt, uint8_t *lcol) {
    if (!lt.flag) return false;
    for (int i = threadIdx.x; i < lt.ntx; i += blockDim.x) lcol[i] = lt.col[i];
    __syncthreads();
    return true;
}

// A thread's inputs: element q + r LT / R for r < R (q = at(a), negative: none) through
// in.get<R>(q, r), every load in flight together.  Where the binning's flags are in use
// (in.sparse, uniform) the flags of all of them are read before the first load: one LDS
// round trip, not one per load.  ZERO: the middle half of each transform is zeros.
template <class S, int A, int R, bool ZERO, class In, class At>
__device__ __forceinline__ void load_inputs(const In &in, float2 (&x)[A][R], At at) {
    const float2 zero = make_float2(0.f, 0.f);
    const auto inside = [](int r) { return !(ZERO && R >= 4 && r >= R / 4 && r < 3 * R / 4); };
    if (in.sparse) {
        bool need[A][R];
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) need[a][r] = at(a) >= 0 && in.need(at(a) + r * (S::LT / R));
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) x[a][r] = need[a][r] ? in.template get<R>(at(a), r) : zero;
    } else {
#pragma unroll
        for (int a = 0; a < A; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) x[a][r] = inside(r) && at(a) >= 0 ? in.template get<R>(at(a), r) : zero;
    }
}

// The workgroup's BATCH transforms: inputs through in, the outputs (PRUNE: the kept
// ones only) through out.  ZERO: the inputs of the middle half of each transform are
// zeros (the adjoint's padding) and not asked for.
template <class S, bool SPLIT, bool PRUNE, bool ZERO, class In, class Out>
__device__ __forceinline__ void transform(float2 *lds, const float2 *tw, const float2 *w16, float *scratch,
                                          const In &in, const Out &out) {
    using F = First<S>;
    float2 x[F::N][F::R];
    load_inputs<S, F::N, F::R, ZERO>(in, x, [](int a) { return F::at(a); });
    transform_loaded<S, SPLIT, PRUNE>(lds, tw, w16, scratch, x, out);
}

// Pass 1: a workgroup transforms one panel of BATCH adjacent fine-grid columns.  mid's
// panels hold MP >= BATCH columns: the MP / BATCH workgroups that fill one panel (each
// writing its columns' pieces of the panel's lines) run on one XCD when xcd_pair is set,
// so that its L2 merges the pieces before they reach HBM.
template <class S>
struct ColsIn {
    const float2 *src;
    const uint8_t *lrow;
    int log_tile_y;
    bool sparse;
    __device__ __forceinline__ bool need(int E) const { return lrow[(E / S::B) >> log_tile_y] != 0; }
    template <int R>
    __device__ __forceinline__ float2 get(int q, int r) const {
        return at_offset(src, 8u * ((unsigned)q + r * (S::LT / R)));
    }
};

template <class S, int MP>
struct ColsOut {
    using Pre = NoPre;
    float2 *dst;
    __device__ __forceinline__ Pre pre(int, int) const { return {}; }
    // output l + i L / 4 is mode row l + L / 4 (i = 0) or l (i = 3)
    __device__ __forceinline__ void put(int E, int i, float2 v, Pre) const {
        const unsigned ky = (unsigned)E / S::B + (i == 0 ? S::L / 4 : 0);
        put_offset(dst, 8u * (ky * MP + (unsigned)E % S::B), v);
    }
};

template <int LOGL, int BATCH, int NT, bool SPLIT, int MP>
__global__ void __launch_bounds__(NT) fft_pass1_kernel(const float2 *__restrict__ fine,
                                                       float2 *__restrict__ mid,
                                                       const float2 *__restrict__ tw,
                                                       const float2 *__restrict__ w16, LiveTiles lt,
                                                       int xcd_pair) {
    using S = Shape<LOGL, BATCH, NT>;
    static_assert(MP % BATCH == 0, "mid panels hold whole column batches");
    extern __shared__ float2 lds[];
    __shared__ float scratch[NT / 64 * BATCH];
    __shared__ uint8_t lrow[kMaxTileRows];
    int pc = blockIdx.x;
    if (MP > BATCH && xcd_pair) {
        constexpr int G = MP / BATCH;
        const int xcd = pc & 7, slot = pc >> 3;
        pc = ((slot / G) * 8 + xcd) * G + slot % G;
    }
    if (!column_needed(lt, pc * BATCH)) return;
    const bool sparse = live_rows(lt, pc * BATCH, lrow);
    const float2 *src = fine + (size_t)pc * S::LT;
    constexpr int MY = S::L / 2;   // the kept modes (the fine grid is twice the destination)
    const int x0 = pc * BATCH;
    const ColsOut<S, MP> out{mid + (size_t)(x0 / MP) * MY * MP + x0 % MP};
    transform<S, SPLIT, true, false>(
        lds, tw, w16, scratch, ColsIn<S>{src, lrow, lt.log_tile_y, sparse}, out);
}

// Pass 2: a workgroup transforms BATCH rows of mid; fused deconvolution and
// destination phase (mx = L / 2).
template <class S>
struct RowsIn {
    const float2 *mid;   // this workgroup's first row
    const uint8_t *lcol;
    unsigned my;
    int log_panel, log_tile_x;
    bool sparse;
    __device__ __forceinline__ bool need(int E) const { return lcol[(E / S::B) >> log_tile_x] != 0; }
    __device__ __forceinline__ unsigned index(unsigned E) const {
        const unsigned lx = E / S::B;
        // (24-bit factors: at most 16384 columns and 8192 rows)
        return ((__umul24(lx >> log_panel, my) + E % S::B) << log_panel) + (lx & ((1u << log_panel) - 1u));
    }
    template <int R>
    __device__ __forceinline__ float2 get(int q, int r) const {
        // panels hold at most 16 columns: steps of a multiple of 16 columns are linear
        if constexpr (S::L / R % 16 == 0) return at_offset(mid, 8u * (index(q) + r * (S::L / R) * my));
        else return at_offset(mid, 8u * index(q + r * (S::LT / R)));
    }
};

template <class S>
struct RowsOut {
    struct Pre {
        float2 d, old;
    };
    float2 *u2;   // this workgroup's first row
    const float2 *dx, *dy;
    int accumulate;
    static constexpr int MX = S::L / 2;
    // output l + i L / 4 is mode column l + L / 4 (i = 0) or l (i = 3)
    static __device__ __forceinline__ unsigned column(int E, int i) { return (unsigned)E / S::B + (i == 0 ? S::L / 4 : 0); }
    static __device__ __forceinline__ unsigned at(int E, int i) { return 8u * ((unsigned)E % S::B * MX + column(E, i)); }
    __device__ __forceinline__ Pre pre(int E, int i) const {
        return {at_offset(dx, 8u * column(E, i)), accumulate ? at_offset(u2, at(E, i)) : make_float2(0.f, 0.f)};
    }
    __device__ __forceinline__ void put(int E, int i, float2 v, Pre p) const {
        const float2 r = cmul(cmul(v, p.d), dy[E % S::B]);
        put_offset(u2, at(E, i), make_float2(p.old.x + r.x, p.old.y + r.y));
    }
};

template <int LOGL, int BATCH, int NT, bool SPLIT>
__global__ void __launch_bounds__(NT) fft_pass2_kernel(const float2 *__restrict__ mid,
                                                       float2 *__restrict__ u2,
                                                       const float2 *__restrict__ tw,
                                                       const float2 *__restrict__ w16,
                                                       const float2 *__restrict__ dx,
                                                       const float2 *__restrict__ dy, int my,
                                                       int log_panel, int xcd_group, int accumulate,
                                                       LiveTiles lt) {
    using S = Shape<LOGL, BATCH, NT>;
    extern __shared__ float2 lds[];
    __shared__ float scratch[NT / 64 * BATCH];
    __shared__ uint8_t lcol[kMaxTileCols];
    // workgroups are dealt to the 8 XCDs round-robin: give the xcd_group
    // workgroups whose rows share lines of mid consecutive slots on one XCD
    int grp = blockIdx.x;
    if (xcd_group > 1) {
        const int xcd = grp & 7, slot = grp >> 3;
        grp = ((slot / xcd_group) * 8 + xcd) * xcd_group + slot % xcd_group;
    }
    const int row0 = grp * BATCH;
    const bool sparse = live_cols(lt, lcol);
    // columns the column pass skipped are zeros, not loaded
    transform<S, SPLIT, true, false>(
        lds, tw, w16, scratch,
        RowsIn<S>{mid + ((size_t)row0 << log_panel), lcol, (unsigned)my, log_panel, lt.log_tile_x, sparse},
        RowsOut<S>{u2 + (size_t)row0 * (S::L / 2), dx, dy + row0, accumulate});
}

// ---- adjoint (type-2 direction) -------------------------------------------------
// The adjoint of the forward's two pruned passes: the kept modes, zero-padded
// to the fine grid, go through the unnormalised inverse-direction (exp(+i)) DFT,
// rows first, then columns.  exp(+i) transforms reuse the exp(-i) stages as
// conj(DFT(conj(x))): values are conjugated as they are loaded and stored.
// Mode m of a length-L transform sits at index m mod L; destination pixel ix
// is mode ix - mx/2.

// Adjoint pass 2: a workgroup takes BATCH rows of g2, multiplies by
// conj(Dx[ix] Dy[iy]) (the adjoint of the fused deconvolution and phase),
// zero-pads to nfx and writes the transformed rows to mid (my x nfx, row-major; with
// flags, not the columns the column pass skips).
// Kept mode of element l0 + r L / R (l0 < L / R), or -1 where the padding is: modes
// 0 .. L/4 - 1 sit in the first quarter, -L/4 .. -1 in the last.
template <class S, int R>
__device__ __forceinline__ int kept_mode(int l0, int r) {
    if constexpr (R >= 4) return l0 + r * (S::L / R) + (r < R / 4 ? S::L / 4 : -(3 * S::L / 4));
    else return r == 0 ? (l0 < S::L / 4 ? l0 + S::L / 4 : -1) : (l0 >= S::L / 4 ? l0 - S::L / 4 : -1);
}

template <class S>
struct AdjRowsIn {
    const float2 *g2;   // this workgroup's first row
    const float2 *dx, *dy;
    static constexpr bool sparse = false;   // g2 is all there
    __device__ __forceinline__ bool need(int) const { return true; }
    template <int R>
    __device__ __forceinline__ float2 get(int q, int r) const {
        const int ix = kept_mode<S, R>(q / S::B, r), row = q % S::B;
        if (R < 4 && ix < 0) return make_float2(0.f, 0.f);
        // conj(g conj(Dx Dy)) = conj(g) Dx Dy
        const float2 gv = at_offset(g2, 8u * (unsigned)(row * (S::L / 2) + ix));
        return cmul(cmul(make_float2(gv.x, -gv.y), at_offset(dx, 8u * (unsigned)ix)), dy[row]);
    }
};

template <class S>
struct AdjRowsOut {
    using Pre = NoPre;
    float2 *dst;
    const uint8_t *lcol;
    int log_tile_x;
    bool sparse;   // only the flagged tile columns are written
    __device__ __forceinline__ Pre pre(int, int) const { return {}; }
    __device__ __forceinline__ void put(int E, int i, float2 v, Pre) const {
        const unsigned l = (unsigned)E / S::B + i * (S::L / 4);
        if (!sparse || lcol[l >> log_tile_x])
            put_offset(dst, 8u * ((unsigned)E % S::B * S::L + l), make_float2(v.x, -v.y));
    }
};

template <int LOGL, int BATCH, int NT, bool SPLIT>
__global__ void __launch_bounds__(NT) fft_adj_rows_kernel(const float2 *__restrict__ g2,
                                                          float2 *__restrict__ mid,
                                                          const float2 *__restrict__ tw,
                                                          const float2 *__restrict__ w16,
                                                          const float2 *__restrict__ dx,
                                                          const float2 *__restrict__ dy, LiveTiles lt) {
    using S = Shape<LOGL, BATCH, NT>;
    extern __shared__ float2 lds[];
    __shared__ float scratch[NT / 64 * BATCH];
    __shared__ uint8_t lcol[kMaxTileCols];
    const int row0 = blockIdx.x * BATCH;
    const bool sparse = live_cols(lt, lcol);
    transform<S, SPLIT, false, true>(
        lds, tw, w16, scratch, AdjRowsIn<S>{g2 + (size_t)row0 * (S::L / 2), dx, dy + row0},
        AdjRowsOut<S>{mid + (size_t)row0 * S::L, lcol, lt.log_tile_x, sparse});
}

// Adjoint pass 1: a workgroup takes BATCH adjacent columns of mid (the my kept
// rows), zero-pads to nfy and writes the transformed columns to the fine grid
// in its panel layout (panels of FP columns: FP = BATCH, or 1, column-major; with the
// binning's flags, only the cells of tiles some record reaches, which are all that the
// interpolation uses).  The 16 / BATCH panels that share 128-byte lines of mid rows
// run on one XCD.
template <class S>
struct AdjColsIn {
    const float2 *src;
    unsigned nfx;
    static constexpr bool sparse = false;   // the panel's columns are all there
    __device__ __forceinline__ bool need(int) const { return true; }
    template <int R>
    __device__ __forceinline__ float2 get(int q, int r) const {
        const int ky = kept_mode<S, R>(q / S::B, r);
        if (R < 4 && ky < 0) return make_float2(0.f, 0.f);
        const float2 v = at_offset(src, 8u * ((unsigned)ky * nfx + (unsigned)q % S::B));
        return make_float2(v.x, -v.y);
    }
};

template <class S, int FP>
struct AdjColsOut {
    using Pre = NoPre;
    float2 *dst;
    const uint8_t *lrow;
    int log_tile_y;
    bool sparse;   // only the cells of flagged tiles are written
    __device__ __forceinline__ Pre pre(int, int) const { return {}; }
    __device__ __forceinline__ void put(int E, int i, float2 v, Pre) const {
        const unsigned l = (unsigned)E / S::B + i * (S::L / 4);
        if (sparse && !lrow[l >> log_tile_y]) return;
        const unsigned at = FP == S::B ? (unsigned)E + i * (S::LT / 4) : (unsigned)E % S::B * S::L + l;
        put_offset(dst, 8u * at, make_float2(v.x, -v.y));
    }
};

template <int LOGL, int BATCH, int NT, bool SPLIT, int FP>
__global__ void __launch_bounds__(NT) fft_adj_cols_kernel(const float2 *__restrict__ mid,
                                                          float2 *__restrict__ fine,
                                                          const float2 *__restrict__ tw,
                                                          const float2 *__restrict__ w16,
                                                          int nfx, int xcd_group, LiveTiles lt) {
    using S = Shape<LOGL, BATCH, NT>;
    static_assert(FP == BATCH || FP == 1, "narrower fine-grid panels are single columns");
    extern __shared__ float2 lds[];
    __shared__ float scratch[NT / 64 * BATCH];
    __shared__ uint8_t lrow[kMaxTileRows];
    int pc = blockIdx.x;
    if (xcd_group > 1) {
        const int xcd = pc & 7, slot = pc >> 3;
        pc = ((slot / xcd_group) * 8 + xcd) * xcd_group + slot % xcd_group;
    }
    // with flags: a panel no record reaches is not needed at all, and in the others
    // only the cells of tiles some record reaches are stored
    if (!column_needed(lt, pc * BATCH)) return;
    const bool sparse = live_rows(lt, pc * BATCH, lrow);
    transform<S, SPLIT, false, true>(
        lds, tw, w16, scratch, AdjColsIn<S>{mid + pc * BATCH, (unsigned)nfx},
        AdjColsOut<S, FP>{fine + (size_t)pc * S::LT, lrow, lt.log_tile_y, sparse});
}

// Kernels needing more than 64 KB of dynamic LDS must say so once per size.
hipError_t allow_lds(const void *kernel, size_t lds, size_t &enabled) {
    if (lds > 65536 && lds > enabled) {
        hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        enabled = lds;
    }
    return hipSuccess;
}

// Threads per workgroup for BATCH transforms of length 2^LOGL: one wave per
// 16-instance block up to 8 waves, then several blocks per wave, except that several
// columns in 68 KB of LDS (two workgroups per CU) take 16 waves (2048 x 2048 fine grid,
// column pass 15.3 -> 14.5 us; the adjoint's of 4096 x 4096 55.3 -> 52.9; one 4096-
// or 8192-point column in 16 waves is slower, 53.8 -> 64.1 and 88 -> 98 us).  The split
// FP16 stages need more registers than the second workgroup of 16 waves leaves them (the
// adjoint's columns of 4096 x 4096: 75.4 us in 16 waves, 57.0 in 8).  No more threads than
// the radix-8 first stage has instances.
template <int LOGL, int BATCH, bool COLUMNS, bool SPLIT>
constexpr int threads_for() {
    constexpr int total = BATCH << LOGL, blocks = total / 256;
    constexpr int nt = blocks <= 8 ? 64 * blocks : COLUMNS && !SPLIT && BATCH > 1 && blocks >= 32 ? 1024 : 512;
    constexpr int cap = LOGL % 4 == 3 && total / 8 >= 64 ? total / 8 : nt;
    return nt < cap ? nt : cap;
}

template <int LOGL, int BATCH, bool SPLIT, int MP = BATCH>
hipError_t launch1(const float2 *fine, float2 *mid, const float2 *tw, const float2 *w16, int nfx, int my,
                   const LiveTiles &lt, hipStream_t s) {
    constexpr int NT = threads_for<LOGL, BATCH, true, SPLIT>();
    constexpr size_t lds = Shape<LOGL, BATCH, NT>::SIZE * sizeof(float2);
    static thread_local size_t enabled = 0;
    auto k = fft_pass1_kernel<LOGL, BATCH, NT, SPLIT, MP>;
    hipError_t e = allow_lds((const void *)k, lds, enabled);
    if (e != hipSuccess) return e;
    if (my != (1 << LOGL) / 2) return hipErrorInvalidValue;
    const int groups = nfx / BATCH;
    const int xcd_pair = (MP > BATCH && groups % (8 * (MP / BATCH)) == 0) ? 1 : 0;
    hipLaunchKernelGGL(k, dim3(groups), dim3(NT), lds, s, fine, mid, tw, w16, lt, xcd_pair);
    return hipGetLastError();
}

template <int LOGL, int BATCH, bool SPLIT>
hipError_t launch2(const float2 *mid, float2 *u2, const float2 *tw, const float2 *w16, const float2 *dx,
                   const float2 *dy, int mx, int my, int log_panel, int accumulate, const LiveTiles &lt,
                   hipStream_t s) {
    constexpr int NT = threads_for<LOGL, BATCH, false, SPLIT>();
    constexpr size_t lds = Shape<LOGL, BATCH, NT>::SIZE * sizeof(float2);
    static thread_local size_t enabled = 0;
    auto k = fft_pass2_kernel<LOGL, BATCH, NT, SPLIT>;
    hipError_t e = allow_lds((const void *)k, lds, enabled);
    if (e != hipSuccess) return e;
    if (mx != (1 << LOGL) / 2) return hipErrorInvalidValue;
    const int groups = my / BATCH;
    const int rows_per_line = 16 >> log_panel;   // rows of mid that share a 128-byte line
    const int g = rows_per_line > BATCH ? rows_per_line / BATCH : 1;
    const int xcd_group = (g > 1 && groups % (8 * g) == 0) ? g : 1;
    hipLaunchKernelGGL(k, dim3(groups), dim3(NT), lds, s, mid, u2, tw, w16, dx, dy, my, log_panel, xcd_group,
                       accumulate, lt);
    return hipGetLastError();
}

template <int LOGL, int BATCH, bool SPLIT>
hipError_t launch_adj2(const float2 *g2, float2 *mid, const float2 *tw, const float2 *w16,
                       const float2 *dx, const float2 *dy, int mx, int my, const LiveTiles &lt,
                       hipStream_t s) {
    constexpr int NT = threads_for<LOGL, BATCH, false, SPLIT>();
    constexpr size_t lds = Shape<LOGL, BATCH, NT>::SIZE * sizeof(float2);
    static thread_local size_t enabled = 0;
    auto k = fft_adj_rows_kernel<LOGL, BATCH, NT, SPLIT>;
    hipError_t e = allow_lds((const void *)k, lds, enabled);
    if (e != hipSuccess) return e;
    if (mx != (1 << LOGL) / 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3(my / BATCH), dim3(NT), lds, s, g2, mid, tw, w16, dx, dy, lt);
    return hipGetLastError();
}

template <int LOGL, int BATCH, bool SPLIT, int FP = BATCH>
hipError_t launch_adj1(const float2 *mid, float2 *fine, const float2 *tw, const float2 *w16,
                       int nfx, int my, const LiveTiles &lt, hipStream_t s) {
    constexpr int NT = threads_for<LOGL, BATCH, true, SPLIT>();
    constexpr size_t lds = Shape<LOGL, BATCH, NT>::SIZE * sizeof(float2);
    static thread_local size_t enabled = 0;
    auto k = fft_adj_cols_kernel<LOGL, BATCH, NT, SPLIT, FP>;
    hipError_t e = allow_lds((const void *)k, lds, enabled);
    if (e != hipSuccess) return e;
    if (my != (1 << LOGL) / 2) return hipErrorInvalidValue;
    const int groups = nfx / BATCH;
    const int g = BATCH < 16 ? 16 / BATCH : 1;   // panels per 128-byte line of a mid row
    const int xcd_group = (g > 1 && groups % (8 * g) == 0) ? g : 1;
    hipLaunchKernelGGL(k, dim3(groups), dim3(NT), lds, s, mid, fine, tw, w16, nfx, xcd_group, lt);
    return hipGetLastError();
}

template <bool SPLIT>
hipError_t dispatch_adj2(int len, const float2 *g2, float2 *mid, const float2 *tw, const float2 *w16,
                         const float2 *dx, const float2 *dy, int mx, int my, const LiveTiles &lt, hipStream_t s) {
    switch (__builtin_ctz(len)) {
        case 5: return launch_adj2<5, 8, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 6: return launch_adj2<6, 4, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 7: return launch_adj2<7, 2, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 8: return launch_adj2<8, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 9: return launch_adj2<9, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 10: return launch_adj2<10, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 11: return launch_adj2<11, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 12: return launch_adj2<12, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 13: return launch_adj2<13, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        case 14: return launch_adj2<14, 1, SPLIT>(g2, mid, tw, w16, dx, dy, mx, my, lt, s);
        default: return hipErrorInvalidValue;
    }
}

template <bool SPLIT>
hipError_t dispatch_adj1(int len, const float2 *mid, float2 *fine, const float2 *tw,
                         const float2 *w16, int nfx, int my, const LiveTiles &lt, hipStream_t s) {
    switch (__builtin_ctz(len)) {
        case 5: return launch_adj1<5, 16, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 6: return launch_adj1<6, 16, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 7: return launch_adj1<7, 16, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 8: return launch_adj1<8, 16, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 9: return launch_adj1<9, 16, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 10: return launch_adj1<10, 8, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 11: return launch_adj1<11, 4, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 12: return launch_adj1<12, 2, SPLIT, 1>(mid, fine, tw, w16, nfx, my, lt, s);
        case 13: return launch_adj1<13, 1, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        case 14: return launch_adj1<14, 1, SPLIT>(mid, fine, tw, w16, nfx, my, lt, s);
        default: return hipErrorInvalidValue;
    }
}

// Batch sizes used per length (the same as fft_batch_pass1/2): pass 1 holds up to
// 68 KB of LDS -- 16 columns up to 512 points, then 8, 4, and one column from 4096
// up.  At 4096 and 8192 mid keeps panels of two and four columns (fft_mid_panel),
// each filled by that many one-column workgroups on one XCD: the row pass gathers
// 16- and 32-byte pieces of mid's lines instead of 8 (15 us less at the 4096^2 fine
// grid, 35 us at 8192^2, where pass 1 pays 15 us of it back) while pass 1 keeps one
// column per workgroup.  The adjoint's column pass takes two columns at 4096 and
// stores them column-major.  Pass 2 takes enough rows for one wave when they are
// shorter than 256, two rows at 2048 and 4096 points -- neighbouring rows share every
// piece of a mid panel, so that a 128-byte line fetched from L2 gives 32 bytes instead of
// 16 at 4096 points (2048^2 cap 41.5 -> 34.0 us, 1024^2 11.7 -> 10.0) -- and one row
// otherwise (two 8192-point rows leave one workgroup per CU: 111 -> 114 us at the 4096^2
// relief; four at 512 and 1024 points take longer, too few workgroups).
template <bool SPLIT>
hipError_t dispatch1(const FftShape &sh, const float2 *fine, float2 *mid, const float2 *tw,
                     const float2 *w16, int nfx, int my, const LiveTiles &lt, hipStream_t s) {
    const int log = __builtin_ctz(sh.L);
    switch (log) {
        case 5: return launch1<5, 16, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 6: return launch1<6, 16, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 7: return launch1<7, 16, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 8: return launch1<8, 16, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 9: return launch1<9, 16, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 10: return launch1<10, 8, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 11: return launch1<11, 4, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        case 12: return launch1<12, 1, SPLIT, 2>(fine, mid, tw, w16, nfx, my, lt, s);
        case 13: return launch1<13, 1, SPLIT, 4>(fine, mid, tw, w16, nfx, my, lt, s);
        case 14: return launch1<14, 1, SPLIT>(fine, mid, tw, w16, nfx, my, lt, s);
        default: return hipErrorInvalidValue;
    }
}

template <bool SPLIT>
hipError_t dispatch2(const FftShape &sh, int log_panel, const float2 *mid, float2 *u2, const float2 *tw,
                     const float2 *w16, const float2 *dx, const float2 *dy, int mx, int my,
                     int accumulate, const LiveTiles &lt, hipStream_t s) {
    const int log = __builtin_ctz(sh.L);
    switch (log) {
        case 5: return launch2<5, 8, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 6: return launch2<6, 4, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 7: return launch2<7, 2, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 8: return launch2<8, 1, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 9: return launch2<9, 1, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 10: return launch2<10, 1, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 11: return launch2<11, 2, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 12: return launch2<12, 2, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 13: return launch2<13, 1, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        case 14: return launch2<14, 1, SPLIT>(mid, u2, tw, w16, dx, dy, mx, my, log_panel, accumulate, lt, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int fft_batch_pass1(int len) {
    const int log = __builtin_ctz(len);
    return log <= 9 ? 16 : log == 10 ? 8 : log == 11 ? 4 : 1;
}

int fft_mid_panel(int len) {
    const int log = __builtin_ctz(len);
    return log == 12 ? 2 : log == 13 ? 4 : fft_batch_pass1(len);
}

int fft_batch_pass2(int len) {
    const int log = __builtin_ctz(len);
    return log == 5 ? 8 : log == 6 ? 4 : log == 7 || log == 11 || log == 12 ? 2 : 1;
}

size_t fft_lds_bytes(int len, int batch) {
    const int total = len * batch, lq = total / 16;
    const int ps = lq > 16 ? __builtin_ctz(lq) : 4;
    return (size_t)(total + (total >> ps) * 16) * sizeof(float2);
}

int fft_max_lds_bytes() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 65536;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 65536;
    return v;
}

hipError_t launch_fft_pass1(const FftShape &sh, int split16, const float2 *fine, float2 *mid,
                            const float2 *tw, const float2 *w16, int nfx, int my, const LiveTiles &lt,
                            hipStream_t s) {
    if (lt.flag && (lt.nty > kMaxTileRows || lt.nty <= 0)) return hipErrorInvalidValue;
    if (split16) return dispatch1<true>(sh, fine, mid, tw, w16, nfx, my, lt, s);
    return dispatch1<false>(sh, fine, mid, tw, w16, nfx, my, lt, s);
}

hipError_t launch_fft_pass2(const FftShape &sh, int log_panel, int split16, const float2 *mid,
                            float2 *u2, const float2 *tw, const float2 *w16, const float2 *dx,
                            const float2 *dy, int mx, int my, int accumulate, const LiveTiles &lt,
                            hipStream_t s) {
    if (lt.flag && (lt.ntx > kMaxTileCols || lt.ntx <= 0)) return hipErrorInvalidValue;
    if (split16) return dispatch2<true>(sh, log_panel, mid, u2, tw, w16, dx, dy, mx, my, accumulate, lt, s);
    return dispatch2<false>(sh, log_panel, mid, u2, tw, w16, dx, dy, mx, my, accumulate, lt, s);
}

hipError_t launch_fft_adj_rows(int len, int split16, const float2 *g2, float2 *mid, const float2 *tw,
                               const float2 *w16, const float2 *dx, const float2 *dy, int mx, int my,
                               const LiveTiles &lt, hipStream_t s) {
    if (lt.flag && (lt.ntx > kMaxTileCols || lt.ntx <= 0)) return hipErrorInvalidValue;
    if (split16) return dispatch_adj2<true>(len, g2, mid, tw, w16, dx, dy, mx, my, lt, s);
    return dispatch_adj2<false>(len, g2, mid, tw, w16, dx, dy, mx, my, lt, s);
}

hipError_t launch_fft_adj_cols(int len, int split16, const float2 *mid, float2 *fine,
                               const float2 *tw, const float2 *w16, int nfx, int my, const LiveTiles &lt,
                               hipStream_t s) {
    if (lt.flag && (lt.nty > kMaxTileRows || lt.nty <= 0)) return hipErrorInvalidValue;
    if (split16) return dispatch_adj1<true>(len, mid, fine, tw, w16, nfx, my, lt, s);
    return dispatch_adj1<false>(len, mid, fine, tw, w16, nfx, my, lt, s);
}

}  // namespace asf
