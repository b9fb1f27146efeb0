// Gate lists on the matrix cores: a pass stages tiles in LDS as the fused
// passes do, but runs its gates as blocks of four qubits.  A block is the
// product of every gate the planner could place on its four qubits, a dense
// 16 x 16 complex matrix, applied to all lines of 16 amplitudes of the tile.
//
// Why: a fused pass interprets its gates one by one on vector registers, 8
// vector instructions per amplitude for a U3 and 3 for a CNOT, and is bound by
// them.  A block costs the same whatever it holds, and a slanted stack of a
// layered circuit puts 6 to 10 gates in it.  6 layers of U3 and a CNOT ladder
// on 28 qubits (330 gates, complex64): 20.1 ms as fused passes, 12.6 ms as 50
// blocks in 6 passes; 8 layers on 14 qubits (complex128): 304 and 102 us.
//
// What bounds it: the issue of vector and matrix instructions, 61 and 12 per
// 16 lines (counters: a SIMD's matrix core is busy 35 % of the pass of 16
// blocks, 0.196 ms per block on 28 qubits); a pass's HBM traffic hides behind
// them from about four blocks on.
//
// complex64: both operands are split into three bf16 parts, x = h + m + l (each
// part is the rounded rest, 8 bits at a time; exact in the range BlkRange keeps
// a tile's larger amplitudes in and for matrix entries of 2^-110 and more), and the six
// products h h, h m, m h, m m, h l, l h are accumulated in FP32, smallest
// first, by v_mfma_f32_16x16x32_bf16: K = 32 is the 16 amplitudes' real and
// imaginary parts, so one instruction forms the real parts of 16 lines.  What
// is dropped is below 2^-26 of each product, a quarter of an FP32 rounding.
// Twelve of these instructions replace sixteen v_mfma_f32_16x16x4f32 of twice
// the time.  complex128 uses v_mfma_f64_16x16x4f64.
//
// A gate whose controls lie outside the tile makes the block's matrix depend
// on at most two index bits that are fixed in a tile: the block holds a matrix
// for each of their values.  All matrices are multiplied up on the device.
//
// Error against extended precision, relative to the fused passes' (rms of 3
// seeds on 8 to 14 qubits): complex64 0.41-0.47 on layered circuits and
// 0.67-0.77 on mixed ones, complex128 0.69-0.74 and 0.93-1.02.
//
// A tile with an infinite, NaN or huge amplitude takes a scalar path that skips
// the entries no gate of the block connects, so that such amplitudes spread no
// further than the gates carry them.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "sv_fused.h"

namespace sv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int BLK_MAX_THREADS = 512;
constexpr int BLK_EXT = 2;             // index bits outside the tile a block may depend on
constexpr int BLK_UNIT_BITS = 5;       // line bits above the 16 lines of a unit, at most

struct BPass {
    TileLayout t;
    int nblk, blk_off;
};

// The LDS byte offsets of a block's lines are XOR-linear in the line's bits, so
// the block lists them per bit.  Which tile position is which bit is free: the
// host picks the lanes' line bits (and complex64's first amplitude bit of the
// lane) so that a half-wavefront's 8-byte (quarter's 16-byte) slots fall on
// distinct banks.
struct BBlock {
    uint32_t lb[4];        // amplitude index bit i of the block
    uint32_t cb[4];        // line bits 0..3: the 16 lines of a unit
    uint32_t ub[BLK_UNIT_BITS];   // line bits 4..8: the unit
    int next;              // external index bits
    int ebit[BLK_EXT];
    int mat;               // first of its 2^next matrices
};

struct BBuild {            // one matrix: ops [op_off, op_off + nops) with the external bits at `base`
    int op_off, nops;
    uint64_t base;
};

// Matrix layout.  float: the operands of the two result tiles (tile q: real and
// imaginary rows of amplitudes 8 q .. 8 q + 7, alternating, so that a lane's
// results are whole amplitudes), three parts h, m, l each, as 64 lanes x 8
// bf16, then the matrix itself (float2, row-major), then 16 reach masks
// (column c: the rows it reaches).  Lane group g holds columns
// 2 g, 2 g + 1, 8 + 2 g, 9 + 2 g.
// double: the operands of the four k steps as 64 lanes x (Ur, Ui), then the masks.
template <typename R> struct MatBytes;
template <> struct MatBytes<float> { static constexpr uint32_t full = 6144, reach = 8192, stride = 8448; };
template <> struct MatBytes<double> { static constexpr uint32_t full = 0, reach = 4096, stride = 4352; };

__device__ __forceinline__ uint32_t bf16_round(float x) {      // finite x
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    return (u + 0x7fffu + (u >> 16 & 1u)) >> 16;
}

// sum_i c_i (vh_i + vl_i) of N terms as an unevaluated sum (hi, lo): products by
// FMA, sums with their rounding errors (Knuth's two-sum).  Nothing may be
// contracted here beyond the FMAs that are written.
template <int N>
__device__ __forceinline__ double2 dd_dot(const double (&c)[N], const double2 (&v)[N]) {
#pragma clang fp contract(off)
    double hi = 0.0, lo = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double p = c[i] * v[i].x, e = __builtin_fma(c[i], v[i].y, __builtin_fma(c[i], v[i].x, -p));
        const double t = hi + p, z = t - hi;
        lo += ((hi - (t - z)) + (p - z)) + e;
        hi = t;
    }
    const double t = hi + lo;
    return make_double2(t, lo - (t - hi));
}

// A matrix entry as the build holds it.  complex64 multiplies its matrices up in
// FP64 and rounds once; complex128 in pairs of FP64, since what a product of 5
// gates in FP64 has lost by then is as much as the gates themselves lose when
// they are applied one by one.
template <typename R> struct Entry;
template <> struct Entry<float> {
    double2 v;
    __device__ __forceinline__ Entry(double x) : v(make_double2(x, 0.0)) {}
    __device__ __forceinline__ Entry partner(int sh) const {
        Entry e(0.0);
        e.v = make_double2(__shfl_xor(v.x, sh, 64), __shfl_xor(v.y, sh, 64));
        return e;
    }
    // d * this + o * w
    __device__ __forceinline__ void mix(double2 d, double2 o, const Entry &w) { v = cmac2<double>(d, v, o, w.v); }
    __device__ __forceinline__ void scale(double2 d) { v = cmul<double>(v, d); }
    __device__ __forceinline__ double2 value() const { return v; }
};
template <> struct Entry<double> {
    double2 re, im;        // (hi, lo)
    __device__ __forceinline__ Entry(double x) : re(make_double2(x, 0.0)), im(make_double2(0.0, 0.0)) {}
    __device__ __forceinline__ Entry partner(int sh) const {
        Entry e(0.0);
        e.re = make_double2(__shfl_xor(re.x, sh, 64), __shfl_xor(re.y, sh, 64));
        e.im = make_double2(__shfl_xor(im.x, sh, 64), __shfl_xor(im.y, sh, 64));
        return e;
    }
    __device__ __forceinline__ void mix(double2 d, double2 o, const Entry &w) {
        const double2 r = dd_dot<4>({d.x, -d.y, o.x, -o.y}, {re, im, w.re, w.im});
        im = dd_dot<4>({d.y, d.x, o.y, o.x}, {re, im, w.re, w.im});
        re = r;
    }
    __device__ __forceinline__ void scale(double2 d) {
        const double2 r = dd_dot<2>({d.x, -d.y}, {re, im});
        im = dd_dot<2>({d.y, d.x}, {re, im});
        re = r;
    }
    __device__ __forceinline__ double2 value() const { return make_double2(re.x, im.x); }
};

// One workgroup per matrix, an entry per thread: wave w holds columns 4 w ..
// 4 w + 3, lane = row + 16 (column % 4), so an op's other row is the lane that
// differs in the target's bit.  The operations come through LDS in chunks (one
// memory latency each would be most of the kernel).  14-qubit circuits,
// complex128 (8 layers and 80 mixed gates, mean): 9.2 us in FP64 pairs; with the
// matrix in LDS, a wave per matrix and a barrier per op 12.0 us in FP64.
template <typename R>
__global__ __launch_bounds__(256) void k_block_build(const BBuild *__restrict__ todo, const ROp *__restrict__ ops,
                                                     unsigned char *__restrict__ mats) {
    constexpr int CH = 32;
    static_assert(sizeof(ROp) % 8 == 0, "operations are copied as 8-byte words");
    __shared__ uint64_t chunk[CH * sizeof(ROp) / 8];
    const BBuild B = todo[blockIdx.x];
    const int lane = threadIdx.x & 63, r = lane & 15, c = threadIdx.x >> 4;
    Entry<R> v(r == c ? 1.0 : 0.0);
    bool reach = r == c;                      // column c reaches row r
    for (int o = 0; o < B.nops; ++o) {
        if (o % CH == 0) {
            __syncthreads();
            const int n = (int)(sizeof(ROp) / 8) * (B.nops - o < CH ? B.nops - o : CH);
            const uint64_t *src = (const uint64_t *)(ops + B.op_off + o);
            for (int i = threadIdx.x; i < n; i += 256) chunk[i] = src[i];
            __syncthreads();
        }
        const ROp &f = ((const ROp *)chunk)[o % CH];
        if ((B.base & f.gmask) != f.gval) continue;
        const bool on = f.onm >> r & 1u;
        if (f.type == OP_PHASE) {
            if (on) v.scale(make_double2(f.u[0], f.u[1]));
            continue;
        }
        const int sh = 1 << f.j0;
        const Entry<R> w = v.partner(sh);
        const bool wreach = __shfl_xor((int)reach, sh, 64) != 0;
        if (!on) continue;
        if (f.type == OP_X) {
            v = w;
            reach = wreach;
        } else {
            const int q = r & sh ? 6 : 0;
            v.mix(make_double2(f.u[q], f.u[q + 1]), make_double2(f.u[q ? 4 : 2], f.u[q ? 5 : 3]), w);
            reach |= wreach;
        }
    }
    unsigned char *M = mats + (size_t)blockIdx.x * MatBytes<R>::stride;
    const double2 z = v.value();
    if (sizeof(R) == 4) {
        uint32_t *part = (uint32_t *)M;
        float x = (float)z.x, y = (float)z.y;
        ((float2 *)(M + MatBytes<R>::full))[r * 16 + c] = make_float2(x, y);
        // row r of U: rows 2 (r % 8) and 2 (r % 8) + 1 of tile r / 8; column c: K
        // slots 2 ks, 2 ks + 1 of lane group gc
        const int tile = r >> 3, row = 2 * (r & 7), gc = (c >> 1) & 3, ks = (c & 1) | (c >> 3 << 1);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t hx = bf16_round(x), hy = bf16_round(y);
            x -= __builtin_bit_cast(float, hx << 16);
            y -= __builtin_bit_cast(float, hy << 16);
            uint32_t *at = part + (tile * 3 + p) * 256 + (gc * 16 + row) * 4 + ks;
            at[0] = hx | (hy ^ 0x8000u) << 16;        // real row: Ur, -Ui
            at[4] = hy | hx << 16;                    // imaginary row: Ui, Ur
        }
    } else {
        ((double2 *)M)[(c >> 2) * 64 + (c & 3) * 16 + r] = z;
    }
    const uint64_t all = __ballot(reach);             // rows of the wave's four columns
    if (r == 0) ((uint32_t *)(M + MatBytes<R>::reach))[c] = (uint32_t)(all >> (lane & 48)) & 0xffffu;
}

// the matrix operands of a wavefront's lane
template <typename R> struct Operand;
template <> struct Operand<float> {
    bf16x8 a[2][3];        // result tile, parts h, m, l
    __device__ __forceinline__ void load(const unsigned char *M, int lane) {
#pragma unroll
        for (int i = 0; i < 6; ++i) a[i / 3][i % 3] = *(const bf16x8 *)(M + i * 1024 + lane * 16);
    }
};
template <> struct Operand<double> {
    double2 a[4];          // k step s: (Ur, Ui)
    __device__ __forceinline__ void load(const unsigned char *M, int lane) {
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = *(const double2 *)(M + s * 1024 + lane * 16);
    }
};

// Units of 16 lines: the lane holds four amplitudes (complex64: register
// indices 2 (lane / 16) + {0, 1, 8, 9}; complex128: lane / 16 + {0, 4, 8, 12})
// of line lane % 16, and gets the same four of the product back: the matrices
// are laid out so that the MFMA result has its rows where the operand had them.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// a unit's amplitudes as MFMA operands: v = h + m + l in bf16 parts (complex64)
template <typename R> struct Unit;
template <> struct Unit<float> {
    bf16x8 p[3];
    __device__ __forceinline__ void split(const float2 (&v)[4]) {
        uintx4 q[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            floatx2 x = {v[i].x, v[i].y};
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                q[t][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
                if (t == 2) break;
                x[0] -= __builtin_bit_cast(float, q[t][i] << 16);
                x[1] -= __builtin_bit_cast(float, q[t][i] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) p[t] = __builtin_bit_cast(bf16x8, q[t]);
    }
};
template <> struct Unit<double> {
    double2 v[4];
    __device__ __forceinline__ void split(const double2 (&x)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = x[i];
    }
};

template <int NU>
__device__ __forceinline__ void block_lines(const Operand<float> &A, const Unit<float> (&x)[NU], float2 (&v)[NU][4]) {
    floatx4 acc[NU][2];
#pragma unroll
    for (int n = 0; n < NU; ++n) acc[n][0] = acc[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    constexpr int ap[6] = {2, 0, 1, 1, 0, 0}, bp[6] = {0, 2, 1, 0, 1, 0};      // smallest products first
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int n = 0; n < NU; ++n)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                acc[n][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.a[q][ap[t]], x[n].p[bp[t]], acc[n][q], 0, 0, 0);
#pragma unroll
    for (int n = 0; n < NU; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[n][i] = make_float2(acc[n][i >> 1][2 * (i & 1)], acc[n][i >> 1][2 * (i & 1) + 1]);
}
// Each result is the sum of four products' worth of columns per k step, the steps
// added at the end in pairs: one chain over all 32 products loses up to 1.35
// times what the gates lose one by one (4 to 5 gates per block), four chains
// with the matrices above 0.7 to 0.9 times.
template <int NU>
__device__ __forceinline__ void block_lines(const Operand<double> &A, const Unit<double> (&x)[NU], double2 (&v)[NU][4]) {
#pragma unroll
    for (int n = 0; n < NU; ++n) {
        doublex4 re[4], im[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const doublex4 zero = {0, 0, 0, 0};
            re[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(A.a[s].x, x[n].v[s].x, zero, 0, 0, 0);
            im[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(A.a[s].x, x[n].v[s].y, zero, 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            re[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(-A.a[s].y, x[n].v[s].y, re[s], 0, 0, 0);
            im[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(A.a[s].y, x[n].v[s].x, im[s], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[n][i] = make_double2((re[0][i] + re[1][i]) + (re[2][i] + re[3][i]), (im[0][i] + im[1][i]) + (im[2][i] + im[3][i]));
    }
}

// The range of the fast path, by a tile's largest component.  From 2^95 on
// (complex128: 2^983; infinities and NaN among it), where a tile's norm could
// leave the range of the operands: the careful path.  Below 2^-60 (2^-900): the
// tile is scaled by 2^64 (2^512) in LDS and back on the way out, for the matrix
// cores flush the bf16 parts below 2^-126 to zero, so that a state of amplitudes
// near 2^-115 came out with a relative error of 3e-6, one near 2^-120 with 1e-4
// (and products of denormal doubles lose their last bits).  What is flushed
// beside larger amplitudes is below 2^-62 of the tile's largest.  `look` gathers
// the largest component, NaN included: one instruction per amplitude, three for
// complex128 (on the high words).
template <typename R> struct BlkRange;
template <> struct BlkRange<float> {
    using key = float;
    static constexpr float high = 0x1p95f, low = 0x1p-60f, up = 0x1p64f, down = 0x1p-64f;
    static __device__ __forceinline__ float look(float m, float2 z) {
        return __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, __builtin_fabsf(z.x)), __builtin_fabsf(z.y));
    }
    static __device__ __forceinline__ bool below(float m, float limit) { return m < limit; }
    static __device__ __forceinline__ bool zero(float m) { return m == 0.f; }       // nothing to scale
};
template <> struct BlkRange<double> {
    using key = uint32_t;
    static constexpr double high = 0x1p983, low = 0x1p-900, up = 0x1p512, down = 0x1p-512;
    static __device__ __forceinline__ uint32_t word(double x) { return (uint32_t)__double2hiint(x) & 0x7fffffffu; }
    static __device__ __forceinline__ uint32_t look(uint32_t m, double2 z) { return max(max(m, word(z.x)), word(z.y)); }
    static __device__ __forceinline__ bool below(uint32_t m, double limit) { return m < word(limit); }
    static __device__ __forceinline__ bool zero(uint32_t) { return false; }         // (0: denormals too)
};

// A tile outside that range: 16 lanes per line, one result row
// each, entry by entry over the entries the block's gates connect (an entry 1
// copies).  A line's reads all come before its writes in the same wavefront.
// Written for few registers: it shares the kernel with the fast path.
template <typename R>
__device__ __forceinline__ void block_careful(const BBlock &b, const unsigned char *M, uint32_t lines) {
    const uint32_t *reach = (const uint32_t *)(M + MatBytes<R>::reach);
    const int r = threadIdx.x & 15;
    auto slot = [&](uint32_t s0, int a) {
        return s0 ^ (a & 1 ? b.lb[0] : 0u) ^ (a & 2 ? b.lb[1] : 0u) ^ (a & 4 ? b.lb[2] : 0u) ^ (a & 8 ? b.lb[3] : 0u);
    };
    for (uint32_t line = threadIdx.x >> 4; line < lines; line += blockDim.x >> 4) {
        uint32_t s0 = 0;
        for (int i = 0; i < 9; ++i) s0 ^= line >> i & 1u ? (i < 4 ? b.cb[i] : b.ub[i - 4]) : 0u;
        // added four columns at a time and in pairs, as on the fast path
        auto add = [](cvec<R> &a, bool &any, cvec<R> b) {
            a = any ? cmake<R>(a.x + b.x, a.y + b.y) : b;
            any = true;
        };
        cvec<R> acc = cmake<R>(0, 0), half = acc, part = acc;
        bool any = false, hany = false, pany = false;
#pragma unroll 1
        for (int c = 0; c < 16; ++c) {
            const cvec<R> z = lds_ld<R>(slot(s0, c));
            const cvec<R> u = sizeof(R) == 4 ? ((const cvec<R> *)(M + MatBytes<R>::full))[r * 16 + c]
                                             : ((const cvec<R> *)M)[(c >> 2) * 64 + (c & 3) * 16 + r];
            if (reach[c] >> r & 1u) add(part, pany, u.x == (R)1 && u.y == (R)0 ? z : cmul<R>(u, z));
            if ((c & 3) == 3) {
                if (pany) add(half, hany, part);
                pany = false;
            }
            if ((c & 7) == 7) {
                if (hany) add(acc, any, half);
                hany = false;
            }
        }
        lds_st<R>(slot(s0, r), acc);
    }
}

// One pass.  Workgroups walk the tiles in strides of the grid.  A wavefront
// takes units of 16 lines; the next block's matrix is loaded while this one's
// units run.  Dynamic LDS: the tile, then three flags (no static LDS, so the tile
// starts at address 0).
// (The next tile read into registers under the last block gained nothing:
// 13.9 against 13.0 ms on the 28-qubit circuit.)
template <typename R>
__global__ __launch_bounds__(BLK_MAX_THREADS, 2) void k_blocks(cvec<R> *__restrict__ psi, const BPass *__restrict__ passes,
                                                            int pi, const BBlock *__restrict__ blocks,
                                                            const unsigned char *__restrict__ mats, uint64_t ntiles) {
    const BPass &P = passes[pi];
    const int c = P.t.c, r = P.t.r;
    const int *hpos = P.t.hpos;
    const uint32_t T = 1u << P.t.k, nt = blockDim.x;
    const uint32_t flag = T * (uint32_t)sizeof(cvec<R>);
    const int lane = threadIdx.x & 63, nw = (int)(nt >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // units per wavefront (the launch makes it a power of two, at most 8), log2 of the wavefronts
    const uint32_t upw = (T >> 8) / (uint32_t)nw;
    const int lw = __builtin_ctz((unsigned)nw);
    lptr<uint32_t> fl = (lptr<uint32_t>)(uintptr_t)flag;
    if (threadIdx.x == 0) fl[0] = fl[1] = fl[2] = 0;
    __syncthreads();

    constexpr int U = sizeof(R) == 4 ? 8 : 4;
    constexpr int LU = sizeof(R) == 4 ? 3 : 2;
    const uint64_t gthr = scatter_t(threadIdx.x, c, r, hpos);
    const uint32_t sthr = swz<R>(threadIdx.x);
    uint64_t hb[LU];
    uint32_t hs[LU];
#pragma unroll
    for (int i = 0; i < LU; ++i) {
        hb[i] = scatter_t(nt << i, c, r, hpos);
        hs[i] = swz<R>(nt << i) * (uint32_t)sizeof(cvec<R>);
    }
    auto uoff = [&](int u) {
        uint64_t o = 0;
#pragma unroll
        for (int i = 0; i < LU; ++i)
            if (u >> i & 1) o |= hb[i];
        return o;
    };
    auto uswz = [&](int u) {
        uint32_t w = 0;
#pragma unroll
        for (int i = 0; i < LU; ++i)
            if (u >> i & 1) w ^= hs[i];
        return w;
    };
    const bool big = T >= nt * U;
    const int g = lane >> 4;
    auto matrix = [&](const BBlock &b, uint64_t base) {
        int v = 0;
        for (int i = 0; i < b.next; ++i) v |= (int)(base >> b.ebit[i] & 1ull) << i;
        return mats + (size_t)(b.mat + v) * MatBytes<R>::stride;
    };

    for (uint64_t tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
        const uint64_t base = pdep64(tl, P.t.nl_mask);
        Operand<R> A, An;
        An.load(matrix(blocks[P.blk_off], base), lane);
        typename BlkRange<R>::key most = 0;
        if (big) {
            for (uint32_t t0 = 0; t0 < T; t0 += nt * U) {
                const uint64_t g0 = base | gthr | scatter_t(t0, c, r, hpos);
                const uint32_t s0 = (sthr ^ swz<R>(t0)) * (uint32_t)sizeof(cvec<R>);
                cvec<R> buf[U];
#pragma unroll
                for (int u = 0; u < U; ++u) buf[u] = psi[g0 | uoff(u)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    most = BlkRange<R>::look(most, buf[u]);
                    lds_st<R>(s0 ^ uswz(u), buf[u]);
                }
            }
        } else {
            for (uint32_t t = threadIdx.x; t < T; t += nt) {
                const cvec<R> z = psi[base | scatter_t(t, c, r, hpos)];
                most = BlkRange<R>::look(most, z);
                lds_st<R>(swz<R>(t) * (uint32_t)sizeof(cvec<R>), z);
            }
        }
        // (a NaN is not below the limit)
        const bool ok = BlkRange<R>::below(most, BlkRange<R>::high), small = BlkRange<R>::below(most, BlkRange<R>::low);
        const uint64_t huge = __ballot(!ok), plain = __ballot(!small), some = __ballot(small && !BlkRange<R>::zero(most));
        if (lane == 0) {
            if (huge) fl[0] = 1;
            if (plain) fl[1] = 1;
            if (some) fl[2] = 1;
        }
        __syncthreads();
        const bool careful = __builtin_amdgcn_readfirstlane((int)fl[0]) != 0;
        const bool scaled = !__builtin_amdgcn_readfirstlane((int)fl[1]) && __builtin_amdgcn_readfirstlane((int)fl[2]);
        if (scaled) {
            for (uint32_t t = threadIdx.x; t < T; t += nt) {
                const cvec<R> z = lds_ld<R>(t * (uint32_t)sizeof(cvec<R>));
                lds_st<R>(t * (uint32_t)sizeof(cvec<R>), cmake<R>(z.x * BlkRange<R>::up, z.y * BlkRange<R>::up));
            }
            __syncthreads();
        }

        for (int bi = 0; bi < P.nblk; ++bi) {
            const BBlock &b = blocks[P.blk_off + bi];
            A = An;
            if (bi + 1 < P.nblk) An.load(matrix(blocks[P.blk_off + bi + 1], base), lane);
            if (careful) {
                block_careful<R>(b, matrix(b, base), T >> 4);
            } else {
                // the lane's four slots in unit 0; in unit u each is XOR-ed with
                // the slots of u's bits (uniform; the units of a wavefront are
                // wave + nw j, both powers of two)
                uint32_t sl = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) sl ^= lane >> i & 1 ? b.cb[i] : 0u;
                constexpr int gb = sizeof(R) == 4 ? 1 : 0;
                sl ^= (g & 1 ? b.lb[gb] : 0u) ^ (g & 2 ? b.lb[gb + 1] : 0u);
                const uint32_t o1 = b.lb[sizeof(R) == 4 ? 0 : 2], o2 = b.lb[3];
                for (int i = 0; i < 5; ++i)
                    if (wave >> i & 1) sl ^= b.ub[i];
                const uint32_t sa[4] = {sl, sl ^ o1, sl ^ o2, sl ^ o1 ^ o2};
                auto get = [&](uint32_t x, cvec<R>(&v)[4]) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = lds_ld<R>(sa[i] ^ x);
                };
                auto put = [&](uint32_t x, const cvec<R>(&v)[4]) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) lds_st<R>(sa[i] ^ x, v[i]);
                };
                if (upw == 1) {
                    Unit<R> x[1];
                    cvec<R> v[1][4];
                    get(0, v[0]);
                    x[0].split(v[0]);
                    block_lines(A, x, v);
                    put(0, v[0]);
                } else {
                    // pairs of units, pipelined: while a pair's products run, the next
                    // pair is split and the one after it is read
                    const uint32_t j0 = b.ub[lw], j1 = b.ub[lw + 1 < 5 ? lw + 1 : 4], j2 = b.ub[lw + 2 < 5 ? lw + 2 : 4];
                    const int pairs = (int)(upw >> 1);
                    auto at = [&](int p) { return (p & 1 ? j1 : 0u) ^ (p & 2 ? j2 : 0u); };
                    Unit<R> x[2], y[2];
                    cvec<R> raw[2][4];
                    auto read = [&](int p) {
                        get(at(p), raw[0]);
                        get(at(p) ^ j0, raw[1]);
                    };
                    auto step = [&](int p, const Unit<R>(&cur)[2], Unit<R>(&nxt)[2]) {
                        cvec<R> out[2][4];
                        block_lines(A, cur, out);
                        nxt[0].split(raw[0]);
                        nxt[1].split(raw[1]);
                        if (sizeof(R) == 4) {
                            // in turn: one product, four vector instructions
#pragma unroll
                            for (int i = 0; i < 24; ++i) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                            }
                        }
                        read(p + 2 < pairs ? p + 2 : p + 1);      // the last step's read is not used
                        put(at(p), out[0]);
                        put(at(p) ^ j0, out[1]);
                    };
                    auto last = [&](int p, const Unit<R>(&cur)[2]) {
                        cvec<R> out[2][4];
                        block_lines(A, cur, out);
                        put(at(p), out[0]);
                        put(at(p) ^ j0, out[1]);
                    };
                    read(0);
                    x[0].split(raw[0]);
                    x[1].split(raw[1]);
                    if (pairs == 1) {
                        last(0, x);
                    } else {
                        read(1);
                        if (pairs == 4) {
                            step(0, x, y);
                            step(1, y, x);
                        }
                        step(pairs - 2, x, y);
                        last(pairs - 1, y);
                    }
                }
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) fl[0] = fl[1] = fl[2] = 0;
        if (scaled) {
            for (uint32_t t = threadIdx.x; t < T; t += nt) {
                const cvec<R> z = lds_ld<R>(swz<R>(t) * (uint32_t)sizeof(cvec<R>));
                psi[base | scatter_t(t, c, r, hpos)] = cmake<R>(z.x * BlkRange<R>::down, z.y * BlkRange<R>::down);
            }
        } else if (big) {
            for (uint32_t t0 = 0; t0 < T; t0 += nt * U) {
                const uint64_t g0 = base | gthr | scatter_t(t0, c, r, hpos);
                const uint32_t s0 = (sthr ^ swz<R>(t0)) * (uint32_t)sizeof(cvec<R>);
                cvec<R> buf[U];
#pragma unroll
                for (int u = 0; u < U; ++u) buf[u] = lds_ld<R>(s0 ^ uswz(u));
#pragma unroll
                for (int u = 0; u < U; ++u) psi[g0 | uoff(u)] = buf[u];
            }
        } else {
            for (uint32_t t = threadIdx.x; t < T; t += nt)
                psi[base | scatter_t(t, c, r, hpos)] = lds_ld<R>(swz<R>(t) * (uint32_t)sizeof(cvec<R>));
        }
        if (tl + gridDim.x < ntiles) __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

// both singular values 1, as far as the entries of a complex64 gate hold it
static bool unitary_gate(const double (&u)[8]) {
    const double a = u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3], b = u[4] * u[4] + u[5] * u[5] + u[6] * u[6] + u[7] * u[7];
    const double re = u[0] * u[4] + u[1] * u[5] + u[2] * u[6] + u[3] * u[7], im = u[1] * u[4] - u[0] * u[5] + u[3] * u[6] - u[2] * u[7];
    return fabs(a - 1.0) < 1e-5 && fabs(b - 1.0) < 1e-5 && fabs(re) < 1e-5 && fabs(im) < 1e-5;
}

// (Gates that are not unitary take the vector passes: the range of the blocks'
// operands rests on rows of norm 1.)
bool blocks_eligible(sv_state s, const std::vector<PGate> &gates) {
    if (s->n < 8) return false;
    bool mixes = false;
    for (const PGate &g : gates) {
        if (popcount64(g.qubits) > 4 || (g.kind == 0 && !unitary_gate(g.u))) return false;
        mixes |= g.kind == 0;
    }
    return mixes;
}

// the op with register bit i moved to perm[i]
static void permute_rop(ROp &f, const int (&perm)[4]) {
    auto bits = [&](uint32_t x) {
        uint32_t y = 0;
        for (int i = 0; i < 4; ++i)
            if (x >> i & 1) y |= 1u << perm[i];
        return y;
    };
    uint32_t on = 0;
    for (uint32_t m = 0; m < 16; ++m)
        if (f.onm >> m & 1) on |= 1u << bits(m);
    f.j0 = perm[f.j0];
    f.j1 = perm[f.j1];
    f.rmask = bits(f.rmask);
    f.rval = bits(f.rval);
    f.onm = on;
}

// passes: targets inside the window, at most BLK_EXT controls outside
static void block_passes(const std::vector<PGate> &gates, int k, int c, std::vector<PlanWindow> &wins) {
    std::vector<PlanItem> items;
    items.reserve(gates.size());
    for (const PGate &g : gates) items.push_back({g.qubits, g.need, 0, 1});
    plan_windows(items, k, (1ull << c) - 1ull, BLK_EXT, -1, 1 << 20, wins);
}

// the blocks of a pass with the local bits L: every local qubit of a gate among
// the block's four
static void blocks_of(const std::vector<PGate> &gates, const PlanWindow &w, uint64_t L, std::vector<PlanWindow> &bw) {
    std::vector<PlanItem> items;
    items.reserve(w.take.size());
    for (int i : w.take) items.push_back({gates[i].qubits & L, gates[i].qubits & L, gates[i].qubits & ~L, 1});
    plan_windows(items, 4, 0, BLK_EXT, BLK_EXT, 1 << 20, bw);
}

void plan_blocks(int n, const std::vector<PGate> &gates, int k, int c, BlockPlan &plan) {
    plan.k = k;
    plan.c = c;
    plan.nblocks = 0;
    block_passes(gates, k, c, plan.wins);
    plan.blocks.resize(plan.wins.size());
    for (size_t i = 0; i < plan.wins.size(); ++i) {
        TileLayout t;
        tile_layout(n, k, plan.wins[i].set, t);
        blocks_of(gates, plan.wins[i], ~t.nl_mask & ((1ull << n) - 1ull), plan.blocks[i]);
        plan.nblocks += (int)plan.blocks[i].size();
    }
}

template <typename R>
static sv_status run_blocks_impl(sv_state s, const std::vector<PGate> &gates, const BlockPlan &plan) {
    std::vector<BPass> passes;
    std::vector<BBlock> blocks;
    std::vector<BBuild> todo;
    std::vector<ROp> rops;
    std::vector<FOp> fops;
    const uint64_t all = (1ull << s->n) - 1ull;
    const int e = sizeof(R) == 4 ? 5 : 4;
    for (size_t wi = 0; wi < plan.wins.size(); ++wi) {
        const PlanWindow &w = plan.wins[wi];
        BPass P;
        memset(&P, 0, sizeof P);
        tile_layout(s->n, plan.k, w.set, P.t);
        P.blk_off = (int)blocks.size();
        const uint64_t L = ~P.t.nl_mask & all;
        for (const PlanWindow &q : plan.blocks[wi]) {
            BBlock b;
            memset(&b, 0, sizeof b);
            uint32_t S = 0;
            for (int i = 0; i < s->n; ++i)
                if (q.set >> i & 1) S |= 1u << popcount64(L & ((1ull << i) - 1ull));
            // a smaller block: the highest free positions as passengers
            for (int p = P.t.k - 1; p >= 0 && popcount64(S) < 4; --p) S |= 1u << p;
            const int mod = sizeof(R) == 4 ? 5 : 4;          // a tile position's bank bit: its residue
            int amp[4], na = 0, col[4], nc = 0;
            for (int p = 0; p < P.t.k; ++p)
                if (S >> p & 1) amp[na++] = p;
            if (mod == 5) {
                // amplitude bit 1 is the fifth of a half-wavefront's lane bits: the
                // block position whose bank bit the other positions can spare
                int best = 0, most = -1;
                for (int i = 0; i < 4; ++i) {
                    uint32_t banks = 0;
                    for (int p = 0; p < P.t.k; ++p)
                        if (!(S >> p & 1) && p % 5 != amp[i] % 5) banks |= 1u << p % 5;
                    if (popcount64(banks) > most) {
                        most = popcount64(banks);
                        best = i;
                    }
                }
                std::swap(amp[1], amp[best]);
            }
            uint32_t banks = mod == 5 ? 1u << amp[1] % 5 : 0u, lines = ((1u << P.t.k) - 1u) & ~S;
            for (int round = 0; round < 2; ++round)          // distinct bank bits first, then any
                for (int p = 0; p < P.t.k && nc < 4; ++p)
                    if ((lines >> p & 1) && (round || !(banks >> p % mod & 1u))) {
                        col[nc++] = p;
                        banks |= 1u << p % mod;
                        lines &= ~(1u << p);
                    }
            auto slot = [&](int p) { return swz_e(1u << p, e) * (uint32_t)sizeof(cvec<R>); };
            for (int i = 0; i < 4; ++i) b.lb[i] = slot(amp[i]);
            for (int i = 0; i < 4; ++i) b.cb[i] = slot(col[i]);
            for (int p = 0, i = 0; p < P.t.k; ++p)
                if (lines >> p & 1) b.ub[i++] = slot(p);
            // to_rops numbers the block's positions in ascending order
            int perm[4];
            for (int i = 0; i < 4; ++i) perm[popcount64(S & ((1u << amp[i]) - 1u))] = i;
            const int off = (int)rops.size();
            uint64_t ext = 0;
            for (int i : q.take) {
                const PGate &g = gates[w.take[i]];
                ext |= g.qubits & ~L;
                fops.clear();
                emit_ops(g, L, fops);
                const size_t r0 = rops.size();
                for (const FOp &f : fops) to_rops(f, S, 4, rops);
                for (size_t j = r0; j < rops.size(); ++j) permute_rop(rops[j], perm);
            }
            for (int i = 0; i < s->n; ++i)
                if (ext >> i & 1) {
                    if (b.next == BLK_EXT) return fail(SV_EDEVICE, "block with more than %d outside controls", BLK_EXT);
                    b.ebit[b.next++] = i;
                }
            b.mat = (int)todo.size();
            for (int v = 0; v < 1 << b.next; ++v) {
                BBuild t{off, (int)rops.size() - off, 0};
                for (int i = 0; i < b.next; ++i)
                    if (v >> i & 1) t.base |= 1ull << b.ebit[i];
                todo.push_back(t);
            }
            blocks.push_back(b);
        }
        P.nblk = (int)blocks.size() - P.blk_off;
        if (P.nblk) passes.push_back(P);
    }
    if (passes.empty()) return SV_OK;
    // one device blob: passes, blocks, build list, ops, matrices
    auto pad = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t bp = pad(passes.size() * sizeof(BPass)), bb = pad(blocks.size() * sizeof(BBlock)),
                 bt = pad(todo.size() * sizeof(BBuild)), bo = pad(std::max<size_t>(rops.size(), 1) * sizeof(ROp));
    std::vector<unsigned char> blob(bp + bb + bt + bo, 0);
    memcpy(blob.data(), passes.data(), passes.size() * sizeof(BPass));
    memcpy(blob.data() + bp, blocks.data(), blocks.size() * sizeof(BBlock));
    memcpy(blob.data() + bp + bb, todo.data(), todo.size() * sizeof(BBuild));
    memcpy(blob.data() + bp + bb + bt, rops.data(), rops.size() * sizeof(ROp));
    unsigned char *dev = nullptr;
    SV_HIP(hipMallocAsync((void **)&dev, blob.size() + todo.size() * MatBytes<R>::stride, s->stream));
    sv_status st = upload_plan(s, dev, blob.data(), blob.size());
    if (st != SV_OK) {
        (void)hipFreeAsync(dev, s->stream);
        return st;
    }
    unsigned char *mats = dev + blob.size();
    {
        TraceScope _ts(s->stream, "block_build", (double)(bo + todo.size() * MatBytes<R>::stride), 0.0);
        hipLaunchKernelGGL(k_block_build<R>, dim3((unsigned)todo.size()), dim3(256), 0, s->stream,
                           (const BBuild *)(dev + bp + bb), (const ROp *)(dev + bp + bb + bt), mats);
    }
    int cus = 0;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, s->device);
    for (size_t i = 0; i < passes.size(); ++i) {
        const int kk = passes[i].t.k;
        const uint64_t tiles = dim_of(s->n - kk);
        const uint32_t units = 1u << (kk - 8);
        const uint32_t waves = std::min<uint32_t>(units, tiles >= 512 ? 4 : BLK_MAX_THREADS / 64);   // units / waves <= 8
        const size_t lds = ((size_t)sizeof(cvec<R>) << kk) + 16;
        const uint64_t per = std::max<size_t>(1, 163840 / lds);
        const uint64_t slots = (uint64_t)(cus > 0 ? cus : 1) * std::min<uint64_t>(per, 32 / waves);
        TraceScope _ts(s->stream, "fused_pass", 2.0 * (double)dim_of(s->n) * sizeof(cvec<R>), 0.0);
        const dim3 grid((unsigned)std::min<uint64_t>(tiles, slots));
        hipLaunchKernelGGL(k_blocks<R>, grid, dim3(waves * 64), lds, s->stream, (cvec<R> *)s->data, (const BPass *)dev,
                           (int)i, (const BBlock *)(dev + bp), (const unsigned char *)mats, tiles);
    }
    const hipError_t err = hipGetLastError();
    (void)hipFreeAsync(dev, s->stream);
    if (err != hipSuccess) return hip_fail(err, "k_blocks launch");
    return SV_OK;
}

sv_status run_blocks(sv_state s, const std::vector<PGate> &gates, int k, int c) {
    // A pinned configuration comes here unchecked.  A block has 4 amplitude, 4
    // lane and at most 5 unit bits (BBlock::ub), so 13 in all, for both types.
    k = std::min(k, s->n);
    if (k < 8 || k > 8 + BLK_UNIT_BITS) return fail(SV_EINVAL, "block tile of %d qubits", k);
    if (!blocks_eligible(s, gates)) return fail(SV_EINVAL, "a circuit that does not run as blocks of four qubits");
    BlockPlan plan;
    plan_blocks(s->n, gates, k, std::max(0, std::min(c, k - 4)), plan);
    return run_blocks(s, gates, plan);
}

sv_status run_blocks(sv_state s, const std::vector<PGate> &gates, const BlockPlan &plan) {
    static bool lds_at_0 = [] {
        bool ok = true;
        for (const void *f : {(const void *)k_blocks<float>, (const void *)k_blocks<double>}) {
            hipFuncAttributes fa;
            ok &= hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 147456) == hipSuccess &&
                  hipFuncGetAttributes(&fa, f) == hipSuccess && fa.sharedSizeBytes == 0;
        }
        (void)hipGetLastError();
        return ok;
    }();
    if (!lds_at_0) return fail(SV_EDEVICE, "the block-pass kernels need their tile at LDS address 0");
    return s->dt == SV_C64 ? run_blocks_impl<float>(s, gates, plan) : run_blocks_impl<double>(s, gates, plan);
}

}  // namespace sv
