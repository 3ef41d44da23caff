// The FFT engine of a workgroup on gfx950, shared by the two-dimensional passes and the
// line path.
//
// A workgroup holds `batch` whole transforms in LDS, interleaved: element e of
// transform c is element E = e batch + c of one array of length L batch, so that the
// workgroup's transforms run as one Stockham transform of that length whose first
// span is batch instead of 1 (every offset is a multiple of batch; neighbouring lanes
// hold neighbouring columns of a panel, which is how the panels are stored).  Each
// length L = r0 * 16^a (compile-time constants, so every index is a shift or a
// constant offset) runs as one radix-r0 stage (r0 in {1,2,4,8}) on the vector ALU,
// then a radix-16 stages, each a 16-point DFT of 16 transform instances per wave and
// block.  The first stage takes its inputs from global memory straight into
// registers and the last one stores the kept outputs straight to global memory: the
// data crosses LDS once per stage but the last.  Two engines run the 16-point DFTs:
//   FP32 (vector ALU): 4 x 4 -- a 4-point DFT over the four inputs a lane
//     holds, twiddles W16^(g k1), a transpose of the block's four 16-lane rows
//     by lane swaps, a second 4-point DFT (about 50 operations per lane);
//   split FP16 (matrix cores): the 16-point DFT as one small GEMM
//     [Re Y; Im Y] (32 x 16) = W16 (32 x 32 real form of the DFT matrix) x [Re X; Im X] (32 x 16)
//     with FP16 hi+lo split products (v_mfma_f32_16x16x32_f16: W_hi X_hi +
//     W_hi X_lo + W_lo X_hi, FP32 accumulation).  Each transform is scaled once, at
//     load, by a power of two that brings its largest |Re|, |Im| to at most 1: a
//     transform of length L grows values by at most L <= 16384 < 65504, and values
//     below 2^-3 of the largest, whose low halves are subnormal, keep 2^-25 of it.
//     (With one scale for the workgroup's transforms a row 2^14 times dimmer than its
//     neighbour was 1e-3 to 3e-3 off, with its own 2e-7; both take the same time.)
// On gfx950 the FP32 matrix rate equals the FP32 vector rate, and a dense
// 16-point DFT costs about six times the operations of the 4 x 4 network, so
// FP32 products stay on the vector ALU.
// Twiddles are applied in FP32 on the vector ALU before each stage's DFT, from
// FP64-computed tables laid out [k][lane group][4] so that a lane fetches its
// four twiddles with two 16-byte loads.
//
// Lane layout of one 16-instance block (wave64): lane = 16 g + jj holds instance
// jj's inputs r = g, g+4, g+8, g+12 and, after the DFT, its outputs
// p = g, g+4, g+8, g+12 (for the GEMM the DFT matrix rows are permuted so that
// the 16 x 16 accumulator's rows 4g..4g+3 are those outputs, and the K index of
// both operands is permuted the same way, (r, re/im) <-> K slot, which the
// contraction does not see).
#pragma once

#include <hip/hip_runtime.h>
#include <type_traits>

namespace asf {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Compile-time shape of a workgroup's BATCH transforms of length 2^LOGL, run by NT
// threads (see the file comment: E = e BATCH + c).
template <int LOGL, int BATCH, int NT>
struct Shape {
    static constexpr int L = 1 << LOGL;
    static constexpr int N16 = LOGL / 4;          // radix-16 stages
    static constexpr int R0 = 1 << (LOGL % 4);    // first (vector ALU) radix
    static constexpr int LT = L * BATCH;          // elements in LDS
    static constexpr int LQ = LT / 16;            // instances of a radix-16 stage
    static constexpr int PS = LQ > 16 ? __builtin_ctz(LQ) : 4;   // one pad of 16 per 2^PS elements
    static constexpr int SIZE = LT + (LT >> PS) * 16;             // LDS elements with the padding
    static constexpr int BLOCKS = LQ / 16;        // 16-instance blocks of a radix-16 stage
    static constexpr int BPW = BLOCKS / (NT / 64);                // per wave
    static constexpr int B = BATCH, T = NT;
    static_assert(BLOCKS % (NT / 64) == 0 && BPW >= 1, "blocks must divide among waves");
    static_assert((BATCH & (BATCH - 1)) == 0, "a power of two of transforms");
    // span (in E) of radix-16 stage s
    static constexpr int span(int s) { return BATCH * R0 << (4 * s); }
};

// LDS position of element e: low 4 bits XOR-swizzled by bits 4..7, plus 16 slots
// of padding every 2^PS elements (keeps a half-wave's accesses on distinct banks).
template <int PS>
__device__ __forceinline__ int lds_pos(int e) {
    return (e ^ ((e >> 4) & 15)) + ((e >> PS) << 4);
}

// 16-point DFTs on the vector ALU in FP32, as 4 x 4 (r = g + 4 i,
// p = k1 + 4 k2):
//   Y[k1 + 4 k2] = sum_g W4^(g k2) W16^(g k1) sum_i x[g + 4 i] W4^(i k1).
// A lane holds x[g + 4 i] for i = 0..3, so the inner 4-point DFT and the twiddle
// W16^(g k1) (g is the lane's row of 16 lanes) stay in its registers; a 4 x 4
// transpose of (row, register) -- two v_permlane32_swap and two
// v_permlane16_swap per real component -- gives row k1 the values of all four
// g, and the outer 4-point DFT leaves Y[g + 4 k2] in register k2 of row g: the
// layout the matrix-core engine produces.  About 50 VALU operations per lane and
// block, where the same DFT as a GEMM takes 16 FP32 MFMAs of 32 cycles.
struct Dft16Valu {
    float2 w1, w2, w3;   // W16^g, W16^2g, W16^3g for this lane's row g
    __device__ __forceinline__ void init(const float2 *w16, int g, int) {
        w1 = w16[g & 15];
        w2 = w16[(2 * g) & 15];
        w3 = w16[(3 * g) & 15];
    }
    // forward 4-point DFT (W4 = -i) in place
    static __device__ __forceinline__ void dft4(float2 (&v)[4]) {
        const float2 a0 = make_float2(v[0].x + v[2].x, v[0].y + v[2].y);
        const float2 a1 = make_float2(v[0].x - v[2].x, v[0].y - v[2].y);
        const float2 a2 = make_float2(v[1].x + v[3].x, v[1].y + v[3].y);
        const float2 a3 = make_float2(v[1].x - v[3].x, v[1].y - v[3].y);
        v[0] = make_float2(a0.x + a2.x, a0.y + a2.y);
        v[2] = make_float2(a0.x - a2.x, a0.y - a2.y);
        v[1] = make_float2(a1.x + a3.y, a1.y - a3.x);   // a1 - i a3
        v[3] = make_float2(a1.x - a3.y, a1.y + a3.x);   // a1 + i a3
    }
    // (row, register) transpose of one real component over the wave's four rows
    static __device__ __forceinline__ void transpose4(float &r0, float &r1, float &r2, float &r3) {
        auto s02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(r0), __float_as_uint(r2), false, false);
        auto s13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(r1), __float_as_uint(r3), false, false);
        auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
        auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
        r0 = __uint_as_float(s01[0]);
        r1 = __uint_as_float(s01[1]);
        r2 = __uint_as_float(s23[0]);
        r3 = __uint_as_float(s23[1]);
    }
    __device__ __forceinline__ void run(float2 (&v)[4]) const {
        dft4(v);
        v[1] = cmul(v[1], w1);
        v[2] = cmul(v[2], w2);
        v[3] = cmul(v[3], w3);
        transpose4(v[0].x, v[1].x, v[2].x, v[3].x);
        transpose4(v[0].y, v[1].y, v[2].y, v[3].y);
        dft4(v);
    }
};

struct Dft16Split16 {
    v8h re_hi, re_lo, im_hi, im_lo;
    __device__ __forceinline__ void init(const float2 *w16, int g, int jj) {
        const int p = (jj >> 2) + 4 * (jj & 3);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = g + 4 * (e >> 1);
            const float2 w = w16[(p * r) & 15];
            const float a = (e & 1) ? -w.y : w.x;
            const float b = (e & 1) ? w.x : w.y;
            const _Float16 ah = (_Float16)a, bh = (_Float16)b;
            re_hi[e] = ah;
            re_lo[e] = (_Float16)(a - (float)ah);
            im_hi[e] = bh;
            im_lo[e] = (_Float16)(b - (float)bh);
        }
    }
    // inputs already scaled into FP16 range
    __device__ __forceinline__ void run(float2 (&v)[4]) const {
        v8h bh, bl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v2f x = {v[i].x, v[i].y};
            const v2h h = __builtin_convertvector(x, v2h);
            const v2f r = x - __builtin_convertvector(h, v2f);
            const v2h l = __builtin_convertvector(r, v2h);
            bh[2 * i] = h.x;
            bh[2 * i + 1] = h.y;
            bl[2 * i] = l.x;
            bl[2 * i + 1] = l.y;
        }
        v4f accr = {0.f, 0.f, 0.f, 0.f}, acci = {0.f, 0.f, 0.f, 0.f};
        accr = __builtin_amdgcn_mfma_f32_16x16x32_f16(re_lo, bh, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f32_16x16x32_f16(im_lo, bh, acci, 0, 0, 0);
        accr = __builtin_amdgcn_mfma_f32_16x16x32_f16(re_hi, bl, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f32_16x16x32_f16(im_hi, bl, acci, 0, 0, 0);
        accr = __builtin_amdgcn_mfma_f32_16x16x32_f16(re_hi, bh, accr, 0, 0, 0);
        acci = __builtin_amdgcn_mfma_f32_16x16x32_f16(im_hi, bh, acci, 0, 0, 0);
        // the products are read here, in the block that issued them: where the first read
        // of the accumulators is left behind a branch (the flag of the adjoint rows' stores),
        // the compiler puts no wait states on the taken path and the read returned stale
        // values (without this, rows of 32, 64, 256, 512 and 1024 points read the sums two to
        // four instructions after the last product, past an s_cbranch)
        asm volatile("" : "+v"(accr), "+v"(acci));
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = make_float2(accr[i], acci[i]);
    }
};

// R-point DFTs (R = 2, 4, 8) of the first stage, in place.
__device__ __forceinline__ void dft_small(float2 (&x)[2]) {
    const float2 a = x[0], b = x[1];
    x[0] = make_float2(a.x + b.x, a.y + b.y);
    x[1] = make_float2(a.x - b.x, a.y - b.y);
}
__device__ __forceinline__ void dft_small(float2 (&x)[4]) { Dft16Valu::dft4(x); }
__device__ __forceinline__ void dft_small(float2 (&x)[8]) {
    float2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    Dft16Valu::dft4(e);
    Dft16Valu::dft4(o);
    // times W8^k = exp(-2 pi i k / 8)
    constexpr float c = 0.70710678118654752440f;
    const float2 t1 = make_float2((o[1].x + o[1].y) * c, (o[1].y - o[1].x) * c);
    const float2 t2 = make_float2(o[2].y, -o[2].x);
    const float2 t3 = make_float2((o[3].y - o[3].x) * c, -(o[3].x + o[3].y) * c);
    const float2 t[4] = {o[0], t1, t2, t3};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = make_float2(e[k].x + t[k].x, e[k].y + t[k].y);
        x[k + 4] = make_float2(e[k].x - t[k].x, e[k].y - t[k].y);
    }
}

// This lane's instance of block b of its wave.
template <class S>
__device__ __forceinline__ int instance(int b) {
    return ((int)(threadIdx.x >> 6) * S::BPW + b) * 16 + (int)(threadIdx.x & 15);
}

// This lane's twiddles of radix-16 stage ST (table entry (k, g, i) =
// exp(-2 pi i (g + 4 i) k / (16 NS)), NS = R0 16^ST): two 16-byte loads per block.  A
// stage's twiddles are fetched during the previous stage, before its last barrier, so
// that their latency hides behind the barrier instead of stalling the stage.
template <class S, int ST>
__device__ __forceinline__ void load_twiddles(const float4 *__restrict__ tw, float4 (&t)[S::BPW][2]) {
    constexpr int NS = S::span(ST) / S::B;
    if constexpr (NS > 1) {
        // tables are stored only for stages with NS > 1, in stage order, 16 NS entries each
        constexpr int first = S::R0 > 1 ? 0 : 1;
        constexpr int offset = [] {
            int off = 0;
            for (int s = first; s < ST; ++s) off += 16 * (S::R0 << (4 * s));
            return off;
        }();
        const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int b = 0; b < S::BPW; ++b) {
            const int k = (instance<S>(b) & (S::span(ST) - 1)) / S::B;
            const float4 *p = tw + (offset + k * 16 + g * 4) / 2;
            t[b][0] = p[0];
            t[b][1] = p[1];
        }
    }
}

// Inputs of radix-16 stage ST from LDS, times its twiddles, through the 16-point DFTs.
template <class S, int ST, class Engine>
__device__ __forceinline__ void stage_read_run(const float2 *lds, const float4 (&t)[S::BPW][2],
                                               float2 (&v)[S::BPW][4], const Engine &eng) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int b = 0; b < S::BPW; ++b) {
        const int q = instance<S>(b);
        if constexpr (S::LQ >= 64) {
            // q + 4 i LQ changes neither bits 4..7 of q nor q mod 2^PS: the swizzled
            // positions of the four inputs are one base plus constant offsets
            const float2 *src = lds + lds_pos<S::PS>(q + g * S::LQ);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[b][i] = src[i * (4 * S::LQ + 64)];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[b][i] = lds[lds_pos<S::PS>(q + (g + 4 * i) * S::LQ)];
        }
        if constexpr (S::span(ST) / S::B > 1) {
            v[b][0] = cmul(v[b][0], make_float2(t[b][0].x, t[b][0].y));
            v[b][1] = cmul(v[b][1], make_float2(t[b][0].z, t[b][0].w));
            v[b][2] = cmul(v[b][2], make_float2(t[b][1].x, t[b][1].y));
            v[b][3] = cmul(v[b][3], make_float2(t[b][1].z, t[b][1].w));
        }
        eng.run(v[b]);
    }
}

// Outputs of radix-16 stage ST (not the last) to their Stockham positions in LDS.
template <class S, int ST>
__device__ __forceinline__ void stage_write(float2 *lds, const float2 (&v)[S::BPW][4]) {
    constexpr int NS = S::span(ST);
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int b = 0; b < S::BPW; ++b) {
        const int q = instance<S>(b);
        const int k = q & (NS - 1);
        const int base = (q - k) * 16 + k;   // (q / NS) * 16 NS + k
        if constexpr (NS >= 64) {
            // 4 i NS leaves bits 4..7 alone, and the 16 NS outputs of an instance group lie
            // within one padding period (16 NS <= LQ = 2^PS): constant offsets
            static_assert(16 * NS <= S::LQ, "not the last stage");
            float2 *dst = lds + lds_pos<S::PS>(base + g * NS);
#pragma unroll
            for (int i = 0; i < 4; ++i) dst[i * 4 * NS] = v[b][i];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) lds[lds_pos<S::PS>(base + (g + 4 * i) * NS)] = v[b][i];
        }
    }
}

// Radix-16 stages ST .. N16-1 (twiddles tcur already in registers).  The last one hands
// its outputs, element E + i LT / 4 with E < LT / 4, to out.put(E, i, value,
// out.pre(E, i)), the pre loads going out before the stage's LDS reads; with PRUNE only
// the outer quarters' (i = 0 and 3: the kept centred modes).
template <class S, int ST, bool PRUNE, class Engine, class Out>
__device__ __forceinline__ void stages_from(float2 *lds, const float4 *tw, const Engine &eng,
                                            const float4 (&tcur)[S::BPW][2], const Out &out, float unscale) {
    float2 v[S::BPW][4];
    if constexpr (ST + 1 < S::N16) {
        stage_read_run<S, ST>(lds, tcur, v, eng);
        float4 tnext[S::BPW][2];
        load_twiddles<S, ST + 1>(tw, tnext);
        __syncthreads();
        stage_write<S, ST>(lds, v);
        __syncthreads();
        stages_from<S, ST + 1, PRUNE>(lds, tw, eng, tnext, out, unscale);
    } else {
        // span LQ: output p = g + 4 i of instance q is element q + p LQ
        const int g = (threadIdx.x & 63) >> 4;
        constexpr int STEP = PRUNE ? 3 : 1;
        typename Out::Pre pre[S::BPW][4];
#pragma unroll
        for (int b = 0; b < S::BPW; ++b)
#pragma unroll
            for (int i = 0; i < 4; i += STEP) pre[b][i] = out.pre(instance<S>(b) + g * S::LQ, i);
        stage_read_run<S, ST>(lds, tcur, v, eng);
#pragma unroll
        for (int b = 0; b < S::BPW; ++b)
#pragma unroll
            for (int i = 0; i < 4; i += STEP)
                out.put(instance<S>(b) + g * S::LQ, i, make_float2(v[b][i].x * unscale, v[b][i].y * unscale),
                        pre[b][i]);
    }
}

// The largest v over a workgroup's lanes of the same transform: lane l of a wave holds
// elements of transform l mod B, first-stage inputs and last-stage outputs alike (every
// instance index and offset is a multiple of B plus the lane).
template <int B>
__device__ __forceinline__ float transform_max(float v, float *scratch) {
    static_assert(B <= 16, "16 lanes of a block");
#pragma unroll
    for (int off = 32; off >= B; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    if ((threadIdx.x & 63) < B) scratch[(threadIdx.x >> 6) * B + (threadIdx.x & 63)] = v;
    __syncthreads();
    float s = 0.f;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s = fmaxf(s, scratch[i * B + (threadIdx.x & (B - 1))]);
    return s;
}

// power of two 2^e with max_abs * 2^-e <= 1 (1 for zero data)
__device__ __forceinline__ int range_exponent(float max_abs) {
    int e = 0;
    if (max_abs > 0.f) frexpf(max_abs, &e);
    return e;
}

// The workgroup's first-stage inputs in registers: x[a][r], element at(a) + r LT / R.
template <class S>
struct First {
    static constexpr int R = S::R0 == 1 ? 4 : S::R0;
    static constexpr int NINST = S::LT / R;   // of the radix-R0 stage
    static constexpr int N = S::R0 == 1 ? S::BPW : (NINST + S::T - 1) / S::T;
    static constexpr bool FULL = S::R0 == 1 || NINST % S::T == 0;
    // -1: this thread has no instance a
    static __device__ __forceinline__ int at(int a) {
        if constexpr (S::R0 == 1) return instance<S>(a) + (int)((threadIdx.x & 63) >> 4) * S::LQ;
        const int q = threadIdx.x + a * S::T;
        return FULL || q < NINST ? q : -1;
    }
};

// The workgroup's transforms from their inputs, the outputs (PRUNE: the kept ones only)
// through out.  With SPLIT each transform's inputs are scaled by the power of two that
// brings its largest |Re|, |Im| to at most 1 (and the outputs scaled back); scratch: B
// floats per wave.
template <class S, bool SPLIT, bool PRUNE, class Out>
__device__ __forceinline__ void transform_loaded(float2 *lds, const float2 *tw, const float2 *w16, float *scratch,
                                                 float2 (&x)[First<S>::N][First<S>::R], const Out &out) {
    using F = First<S>;
    const float4 *tw4 = reinterpret_cast<const float4 *>(tw);
    const int lane = threadIdx.x & 63, g = lane >> 4;
    using Engine = typename std::conditional<SPLIT, Dft16Split16, Dft16Valu>::type;
    Engine eng;
    float4 t0[S::BPW][2];
    float unscale = 1.f;
    load_twiddles<S, S::R0 == 1 ? 1 : 0>(tw4, t0);
    eng.init(w16, g, lane & 15);
    if constexpr (SPLIT) {
        float big = 0.f;
#pragma unroll
        for (int a = 0; a < F::N; ++a)
#pragma unroll
            for (int r = 0; r < F::R; ++r) big = fmaxf(big, fmaxf(fabsf(x[a][r].x), fabsf(x[a][r].y)));
        const int e = range_exponent(transform_max<S::B>(big, scratch));
        const float inv = ldexpf(1.f, -e);
        unscale = ldexpf(1.f, e);
#pragma unroll
        for (int a = 0; a < F::N; ++a)
#pragma unroll
            for (int r = 0; r < F::R; ++r) x[a][r] = make_float2(x[a][r].x * inv, x[a][r].y * inv);
    }
    if constexpr (S::R0 == 1) {
        static_assert(S::N16 >= 2, "16^a with a >= 2");
#pragma unroll
        for (int b = 0; b < S::BPW; ++b) eng.run(x[b]);
        stage_write<S, 0>(lds, x);
        __syncthreads();
        stages_from<S, 1, PRUNE>(lds, tw4, eng, t0, out, unscale);
    } else {
        // radix-R0 stage: instance q takes elements q + r LT/R0
#pragma unroll
        for (int a = 0; a < F::N; ++a) {
            const int q = threadIdx.x + a * S::T;
            dft_small(x[a]);
            const int k = q & (S::B - 1), base = (q - k) * S::R0 + k;
            if (F::FULL || q < F::NINST)
#pragma unroll
                for (int p = 0; p < S::R0; ++p) lds[lds_pos<S::PS>(base + p * S::B)] = x[a][p];
        }
        __syncthreads();
        stages_from<S, 0, PRUNE>(lds, tw4, eng, t0, out, unscale);
    }
}

struct NoPre {};

// Element at a 32-bit byte offset from a uniform base (every array here is below 4 GB):
// one vector add, where 64-bit indexing of each element costs three or four.
__device__ __forceinline__ float2 at_offset(const float2 *base, unsigned bytes) {
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(base) + bytes);
}
__device__ __forceinline__ void put_offset(float2 *base, unsigned bytes, float2 v) {
    *reinterpret_cast<float2 *>(reinterpret_cast<char *>(base) + bytes) = v;
}

}  // namespace
}  // namespace asf
