// Eigen-frame HHL as two fused column-tile kernels.
//
// The clock register [n_s, n_s + n_c) is split into a low group G1 =
// register bits [0, g1) and a high group G2 = [g1, n_c) (g1, g2 <= 10).  A
// tile holds C consecutive system columns j (contiguous in memory) times the
// 2^g clock values of one group, for one setting of the other group's bits
// (and the ancilla).
//
//   k_pipe_a: generate the state after phase estimation (product state over
//             the clock bits, relabelled so the cascades need no swaps), then
//             the inverse-QFT cascade on G1, in closed form.  The G1 stages act on G1
//             qubits only, so the result is still a product between the
//             groups: psi(j, y1, y2) = beta_j T_j(y1) B_j(y2), with T_j the G1
//             transform of the column's G1 factor and B_j(y2) the product of
//             the phases of the set G2 bits.  k_pipe_a therefore runs for
//             y2 = 0 only and leaves T in the clock rows y1 < 2^g1 of the
//             ancilla = 0 half, and stages every column's G2 phases.
//   k_pipe_b: the inverse-QFT cascade on G2 of T_j(y1) B_j(y2): each stage
//             maps a product state over the G2 bits to another, so the
//             cascade's output P is T_j(y1) times a product of one factor per
//             G2 bit, formed directly; then eigenvalue inversion
//             a1 = (1/y) a0 (FP64 sums of P(a=1) and the norm)
//                                                     -> ancilla = 1 half
//             and, while a line is in registers, the uncompute projected on
//             clock 0 (the QFT on the whole clock, the conjugate phases, the
//             Hadamard layer onto |0>).  That is the inner product with the
//             column phase estimation leaves, conj(P) up to the group
//             normalisations, so z_j = beta_j sum_y s_y |P_j(y)|^2
//                                                     -> FP64 partial sums
//
// Inverse cascade stage on register qubit j (relative to the clock register):
//   a1 *= conj(phase), then (a0 + a1, a0 - a1)/sqrt 2
// with phase = exp(2 pi i (v mod 2^j) / 2^(j+1)), v the register value: the
// controlled phases of the textbook QFT circuit that target qubit j.  On a
// product state no stage has to be run: each contributes one factor per line
// (product_line), with the stage's roots from a table per group and the bits
// below the group, fixed for a tile, folded into it.
#include <math.h>

#include <algorithm>
#include <string>
#include <vector>

#include "sv_device.h"
#include "sv_hhl_internal.h"
#include "sv_internal.h"

namespace sv {

struct PipeArgs {
    uint64_t N;          // 2^n_s columns
    int n_s, n_c;
    int g1, g2;          // clock groups
    int cl;              // log2 of the columns per tile
    uint64_t abit;       // ancilla bit
    double scale;        // 2^(-n_c/2)
    int sgn;             // signed (two's-complement) clock for the inversion
    uint64_t gcut;       // 0: inversion sin = 1/y; >= 1: gapped-phase-estimation flag, sin = [|y| >= gcut]
    int iters;           // work-queue items: consecutive column blocks per item
};

// HBM pointers of a solve, in the global address space: the pointers come
// from a descriptor, so without the cast every access would be a flat
// instruction, which also counts against the LDS wait counter.
template <typename T> using gptr = __attribute__((address_space(1))) T *;

// complex loads and stores through a global pointer (a native two-element
// vector, so no class member is needed on an address-space-qualified object)
template <typename R> using v2_t = R __attribute__((ext_vector_type(2)));
template <typename R>
__device__ __forceinline__ cvec<R> gld(const cvec<R> *p, uint64_t i) {
    const v2_t<R> x = ((gptr<const v2_t<R>>)p)[i];
    return cmake<R>(x.x, x.y);
}
template <typename R>
__device__ __forceinline__ void gst(cvec<R> *p, uint64_t i, cvec<R> v) {
    v2_t<R> x;
    x.x = v.x;
    x.y = v.y;
    ((gptr<v2_t<R>>)p)[i] = x;
}

// non-temporal store for the ancilla = 1 half, which k_pipe_b writes once: far
// more than the L2 and MALL hold, so it is streamed (the nt bit) instead of cached
template <typename R>
__device__ __forceinline__ void gst_nt(cvec<R> *p, uint64_t i, cvec<R> v) {
    v2_t<R> x;
    x.x = v.x;
    x.y = v.y;
    __builtin_nontemporal_store(x, &((gptr<v2_t<R>>)p)[i]);
}
template <typename R>
__device__ __forceinline__ cvec<R> cconjmul(cvec<R> a, cvec<R> b) {   // a * conj(b)
    return cmake<R>(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

__device__ __forceinline__ float ffma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double ffma(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ __forceinline__ int tw_off(int jb) { return (1 << jb) - 1; }

// The inverse cascade of a product state over G = RA + RB clock bits, along one
// line: the low RA bits are llo, the 2^RB values of the high ones fill v.  Every
// stage maps a product state to another, so the output at l is
//   p prod_b (1 + (-1)^(l_b) w_b conj(tw_b(l mod 2^b))),
// w_b = om[b C] the phase of bit b, tw_b the stage's twiddle (TW).  The factors
// of the low bits are the line's, those of the high bits branch: a node splits
// into a + a q and 2 a - (a + a q), six operations, and the upper half of a
// level's nodes has the lower half's q, turned by a quarter.
template <typename D, int RA, int RB>
__device__ __forceinline__ void product_line(cvec<D> (&v)[1 << RB], cvec<D> p, const cvec<D> *__restrict__ om, int C,
                                             const cvec<D> *__restrict__ TW, int llo) {
#pragma unroll
    for (int b = 0; b < RA; ++b) {
        const cvec<D> q = cconjmul<D>(om[b * C], TW[tw_off(b) + (llo & ((1 << b) - 1))]);
        const cvec<D> f = (llo >> b & 1) ? cmake<D>((D)1 - q.x, -q.y) : cmake<D>((D)1 + q.x, q.y);
        p = cmul<D>(p, f);
    }
    v[0] = p;
#pragma unroll
    for (int bb = 0; bb < RB; ++bb) {
        const cvec<D> w = om[(RA + bb) * C];
        const int h = 1 << bb;
        auto node = [&](int m, cvec<D> q) {
            const cvec<D> a = v[m];
            const D px = ffma(a.x, q.x, ffma(-a.y, q.y, a.x)), py = ffma(a.x, q.y, ffma(a.y, q.x, a.y));
            v[m] = cmake<D>(px, py);
            v[m + h] = cmake<D>(ffma((D)2, a.x, -px), ffma((D)2, a.y, -py));
        };
#pragma unroll
        for (int m = 0; m < (h + 1) / 2; ++m) {
            const cvec<D> q = cconjmul<D>(w, TW[tw_off(RA + bb) + llo + (m << RA)]);
            node(m, q);
            if (bb > 0) node(m + h / 2, cmake<D>(q.y, -q.x));
        }
    }
}

// Twiddle tables of one group, stage jb at offset 2^jb - 1 (2^jb entries):
// entry m = exp(2 pi i (vlow + m 2^gbase) / 2^(gbase + jb + 1)), where vlow
// (< 2^gbase) are the register bits below the group, fixed for the tile.
template <typename R>
__device__ __forceinline__ void fill_twiddles(cvec<R> *TW, int g, int gbase, uint64_t vlow) {
    for (int i = threadIdx.x; i < (1 << g) - 1; i += blockDim.x) {
        int jb = 0;
        while ((2 << jb) - 1 <= i) ++jb;
        const uint64_t m = (uint64_t)(i - ((1 << jb) - 1));
        const int j = gbase + jb;
        TW[i] = turn_phase<R>((vlow + (m << gbase)) << (63 - j));
    }
}

// tile decomposition: column block and the setting of the other group's bits
__device__ __forceinline__ void tile_coords(const PipeArgs &A, uint64_t &j0, uint64_t &o) {
    const uint64_t nb = A.N >> A.cl;
    const uint64_t tid = (uint64_t)blockIdx.x + (uint64_t)blockIdx.y * gridDim.x;
    j0 = (tid % nb) << A.cl;
    o = tid / nb;
}

// ---------------------------------------------------------------------------
// k_pipe_a: phase-estimation state + inverse cascade on G1
// ---------------------------------------------------------------------------
// In FP64 for both types, rounded once on the store: the table is small (2^g1 of
// the 2^n_c clock rows), and its errors enter |P|^2 of k_pipe_b twice, alike
// (complex64 solves of 10 + 10 qubits: rms error of p_post 4.9e-8, 2.0e-7 with a
// complex64 table).  The stages act on a product state, so the table is a
// product tree per line, like k_pipe_b's, with no tile: 35 us of a 32-qubit
// solve (75 us with the stages' butterflies through an LDS tile).
template <typename R, int RA, int RB, int NT>
__device__ __forceinline__ void pipe_a_body(const PipeArgs &A, const PipeSolve &S, uint64_t j0) {
    constexpr int G = RA + RB;
    cvec<R> *__restrict__ psi = (cvec<R> *)S.psi;
    const gptr<const double> __restrict__ lam = (gptr<const double>)S.lam;
    extern __shared__ unsigned char smem_raw[];
    const int C = 1 << A.cl;
    using D = double;
    cvec<D> *TW = reinterpret_cast<cvec<D> *>(smem_raw);            // [2^G - 1] (+1 pad)
    cvec<D> *om = TW + (1 << G);                                     // [G][C] exp(2 pi i F) of the G1 bits
    const int n_c = A.n_c;
    fill_twiddles<D>(TW, G, 0, 0);
    // the phases of every clock bit and column; bit b carries frac(phi_j 2^(n_c-1-b)).
    // Those of the G2 bits are staged for k_pipe_b in clock rows 2^g1 + r (r < g2)
    // of the ancilla = 0 half, which the solve leaves unused otherwise (only the
    // rows below 2^g1 hold the G1 table)
    for (int e = threadIdx.x; e < n_c * C; e += NT) {
        const int b = e / C, c = e - b * C;
        const uint64_t f = turn_fraction(lam[j0 + c], S.T0, n_c - 1 - b);
        if (b < G) om[e] = turn_phase<D>(f);
        else gst<R>(psi, ((((uint64_t)1 << G) + (uint64_t)(b - G)) << A.n_s) + j0 + c, turn_phase<R>(f));
    }
    __syncthreads();
    // the G Hadamards below omit their 1/sqrt(2): 2^(-G/2) joins the amplitude scale
    const cvec<D> root = cmake<D>(A.scale * exp2(-0.5 * G), 0.0);
    // clock index (k << RA) + llo (G2 value 0): a base for the line and a stride for k
    const int nl = C << RA;
    const uint64_t ks = 1ull << (RA + A.n_s);
    for (int line = threadIdx.x; line < nl; line += NT) {
        const int c = line & (C - 1), llo = line >> A.cl;
        cvec<D> v[1 << RB];
        product_line<D, RA, RB>(v, root, om + c, C, TW, llo);
        cvec<R> *p = psi + ((uint64_t)llo << A.n_s) + j0 + c;
#pragma unroll
        for (int k = 0; k < (1 << RB); ++k) gst<R>(p, k * ks, cmake<R>((R)v[k].x, (R)v[k].y));
    }
}

// beta = V^H b for 64 columns of a dense V: a lane per column, the waves share
// the rows.  b (host memory that the device can read, at most 1024 entries) is
// staged in LDS.
template <int NT>
__device__ __forceinline__ void head_cols(const PipeHead &H, unsigned blk) {
    extern __shared__ unsigned char smem_raw[];
    double2 *bs = reinterpret_cast<double2 *>(smem_raw);
    double2 *part = bs + H.N;
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (uint64_t i = threadIdx.x; i < H.N; i += NT) bs[i] = H.b[i];
    __syncthreads();
    const uint64_t j = (uint64_t)blk * 64 + lane;
    double2 acc = make_double2(0.0, 0.0);
    if (j < H.N)
#pragma unroll 8
        for (uint64_t i = w; i < H.N; i += NW) {
            const double2 v = H.V[i * H.N + j], x = bs[i];
            acc.x = fma(v.x, x.x, fma(v.y, x.y, acc.x));       // conj(v) x
            acc.y = fma(v.x, x.y, fma(-v.y, x.x, acc.y));
        }
    part[w * 64 + lane] = acc;
    __syncthreads();
    if (w || j >= H.N) return;
    for (int k = 1; k < NW; ++k) {
        acc.x += part[k * 64 + lane].x;
        acc.y += part[k * 64 + lane].y;
    }
    H.beta[j] = acc;
}

template <typename R, int RA, int RB, int NT>
__global__ __launch_bounds__(NT) void k_pipe_a(PipeArgs A, PipeSolve one, PipeHead H) {
    if (blockIdx.x >= gridDim.x - H.cols) {
        head_cols<NT>(H, blockIdx.x - (gridDim.x - H.cols));
        return;
    }
    uint64_t j0, o;
    tile_coords(A, j0, o);
    pipe_a_body<R, RA, RB, NT>(A, one, j0);
}

// ---------------------------------------------------------------------------
// k_pipe_b: inverse cascade on G2 and the inversion rotation
// ---------------------------------------------------------------------------
// Writes the state after the rotation (the ancilla = 1 half; not for a
// batch's work-queue items, PERS: no call shows a batch's states), as
// 2^-G2 s_y a(y).  In the half the qubits are
// relabelled in memory, from the bottom: the tile's columns, G2, the other
// column bits, G1, so that a tile is one block of 2^(g2 + cl) amplitudes and
// streams out whole.  (As 2^g2 rows of 512 B per tile, the stores of a 32-qubit
// solve took 3.02-3.07 ms.)
//
// The projection.  Only the clock sum of each transformed column is needed,
//   z = sum_y ph(y) (F v)(y),
// F the forward cascade on the whole clock (the QFT of the uncompute, from
// the top bit down) and ph(y) = prod_b om_b^(y_b) the conjugate phases of
// the controlled powers, a product over the clock bits.  Moved onto the
// input, z = sum_y v(y) K(y) with K the transposed cascade applied to ph,
//   K(y) = prod_b (1 + (-1)^(y_b) t_b(y mod 2^b) om_b),
// t_b the stage's twiddle: factor by factor the conjugate of the amplitudes
// formed here, K = conj(P) 2^((n_c + g1)/2).  With v = 2^-G2 s beta P and the
// 2^(-(n_c + g1)/2) of the Hadamards left out, z_j = beta_j sum_y 2^-G2 s_y |P|^2:
// a real sum per column, taken while the line is in registers.  A third kernel
// that read the half back and contracted it with K took 2.5 of the 5.8 ms of a
// 32-qubit complex64 solve, and 90 of the 247 us of a 26-qubit complex128 one.
// Bound by the stores: 17.2 GB in 2.70 ms, 6.4 TB/s (a plain fill: 6.9).
//
// Tile: columns [j0, j0 + C)
// at G1 value o; a work-queue item (PERS) runs A.iters column blocks j0 + it 2^cl.
// The FP64 partial pair goes to slot `slot`.
template <typename R, int RA, int RB, int NT, bool PERS>
__device__ __forceinline__ void pipe_b_body(const PipeArgs &A, const PipeSolve &S, uint64_t j0, uint64_t o,
                                            uint64_t slot) {
    constexpr int G = RA + RB;
    cvec<R> *__restrict__ psi = (cvec<R> *)S.psi;
    const double2 *__restrict__ beta = S.beta;
    const gptr<double> __restrict__ part = (gptr<double>)S.part;
    const gptr<double> __restrict__ zpart = (gptr<double>)S.zpart;
    extern __shared__ unsigned char smem_raw[];
    const int C = 1 << A.cl;
    cvec<R> *TW = reinterpret_cast<cvec<R> *>(smem_raw);            // [2^G] twiddles of G2 at G1 value o
    R *s2t = reinterpret_cast<R *>(TW + (1 << G));                  // [2^G] s_y^2 2^-G
    R *srt = s2t + (1 << G);                                         // [2^G] s_y 2^-G
    // two sets (alternate tiles) of the column data: om[G][C] the phases of
    // the G2 bits (staged by k_pipe_a in clock rows 2^g1 + b), tT[C] the
    // G1 table entries T_j(o), be[C] the columns' beta; then two sets of the
    // lines' sums of s_y |P|^2
    const int ncd = (G + 2) * C;
    cvec<R> *cd = reinterpret_cast<cvec<R> *>(srt + (1 << G));
    R *zl = reinterpret_cast<R *>(cd + 2 * ncd);
    __shared__ double red[2][NT / 64];
    const int iters = PERS ? A.iters : 1;
    const uint64_t jstep = PERS ? 1ull << A.cl : 0;
    const int g1 = A.g1, n_c = A.n_c;
    auto col_data = [&](int e, uint64_t j) -> cvec<R> {
        const int b = e / C, cq = e - b * C;
        if (b > G) {
            const double2 bj = gld<double>(beta, j + cq);
            return cmake<R>((R)bj.x, (R)bj.y);
        }
        return b < G ? gld<R>(psi, ((((uint64_t)1 << g1) + (uint64_t)b) << A.n_s) + j + cq)
                     : gld<R>(psi, (o << A.n_s) | (j + cq));
    };
    // read before the twiddles are built, so that their latency overlaps that work
    for (int e = threadIdx.x; e < ncd; e += NT) cd[e] = col_data(e, j0);
    fill_twiddles<R>(TW, G, g1, o);
    // rotation of clock value y = o + l 2^g1 (natural order after the inverse
    // transform): sin = 1/y (y >= 1).  The G Hadamards of the inverse cascade
    // and the G of the forward one omit their 1/sqrt(2) each, so 2^-G is
    // folded into the rotation (and into the FP64 weights of the sums, taken
    // where the amplitudes are 2^(G/2) too large).
    const double fold = exp2(-(double)G);
    for (int l = threadIdx.x; l < (1 << G); l += NT) {
        const uint64_t y = o | ((uint64_t)l << g1);
        const double ys = (A.sgn && (y >> (n_c - 1))) ? (double)y - exp2((double)n_c) : (double)y;
        const double sd = !y ? 0.0 : A.gcut ? (fabs(ys) >= (double)A.gcut ? 1.0 : 0.0) : 1.0 / ys;
        s2t[l] = (R)(sd * sd * fold);
        srt[l] = (R)(sd * fold);
    }
    __syncthreads();
    const int nl = C << RA;
    // clock value o + (l << g1), l = llo + (k << RA), of column j0 + c is entry
    // (l << cl) + c of the tile's block: a base for the line and a stride for k
    const uint64_t ks = 1ull << (RA + A.cl);
    double pa = 0.0, nt = 0.0;
    for (int it = 0; it < iters; ++it) {
        const bool more = PERS && it + 1 < iters;
        const cvec<R> *om = cd + (it & 1) * ncd, *tT = om + G * C, *be = tT + C;
        R *zt = zl + (it & 1) * nl;
        // the inverse-QFT output on the G2 register of column j at y = o + l 2^g1,
        // l = llo + (k << RA): the input of the G2 stages is T_j(o) times a product
        // state over the G2 bits
        for (int line = threadIdx.x; line < nl; line += NT) {
            const int c = line & (C - 1), llo = line >> A.cl;
            cvec<R> v[1 << RB];
            product_line<R, RA, RB>(v, tT[c], om + c, C, TW, llo);
            // |P|^2 summed over the line in the amplitude precision, weighted by
            // s_y^2 for P(a = 1), by s_y for z and by one for the norm (the
            // rotation keeps each pair's norm); |beta|^2 and the sums over lines
            // and tiles in FP64
            R lpa = 0, lnt = 0, lz = 0;
            const R *s2l = s2t + llo, *srl = srt + llo;
            const cvec<R> bc = be[c];
            cvec<R> *ps = psi + (A.abit + (o << (G + A.n_s)) + (j0 << G) + ((uint64_t)llo << A.cl) + c);
#pragma unroll
            for (int k = 0; k < (1 << RB); ++k) {
                const R a2 = v[k].x * v[k].x + v[k].y * v[k].y;
                const R sr = srl[k << RA];
                lpa += s2l[k << RA] * a2;
                lz += sr * a2;
                lnt += a2;
                if (!PERS) gst_nt<R>(ps, k * ks, cmul<R>(cmake<R>(v[k].x * sr, v[k].y * sr), bc));
            }
            const double b2 = (double)bc.x * (double)bc.x + (double)bc.y * (double)bc.y;
            pa += b2 * (double)lpa;
            nt += b2 * ((double)lnt * fold);
            zt[(llo << A.cl) + c] = lz;
        }
        // an item's run: the next tile's column data go to the other set, last
        // read in the previous tile (before the last barrier).  (Reading them
        // into registers during the tile cost the work-queue kernel more in
        // spills than it hid.)
        if (more) {
            cvec<R> *nxt = cd + ((it + 1) & 1) * ncd;
            for (int e = threadIdx.x; e < ncd; e += NT) nxt[e] = col_data(e, j0 + jstep);
        }
        __syncthreads();
        for (int cq = threadIdx.x; cq < C; cq += NT) {
            double z = 0.0;
#pragma unroll
            for (int l = 0; l < (1 << RA); ++l) z += (double)zt[(l << A.cl) + cq];
            zpart[o * A.N + j0 + cq] = z;
        }
        j0 += jstep;
    }
    pa = wave_sum_f64(pa);
    nt = wave_sum_f64(nt);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = pa;
        red[1][threadIdx.x >> 6] = nt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sp = 0.0, sn = 0.0;
        for (int w = 0; w < NT / 64; ++w) {
            sp += red[0][w];
            sn += red[1][w];
        }
        part[2 * slot] = sp;
        part[2 * slot + 1] = sn;
    }
}

template <typename R, int RA, int RB, int NT>
__global__ __launch_bounds__(NT) void k_pipe_b(PipeArgs A, PipeSolve one) {
    uint64_t j0, o;
    tile_coords(A, j0, o);               // o = value of the G1 bits
    pipe_b_body<R, RA, RB, NT, false>(A, one, j0, o,
                                      (uint64_t)blockIdx.x + (uint64_t)blockIdx.y * gridDim.x);
}


// ---------------------------------------------------------------------------
// a batch as one persistent kernel over device work queues
// ---------------------------------------------------------------------------
struct QClass {
    PipeArgs A[2];            // launch parameters of the two kernels' items
    int g[2];                 // the group each transforms: g1, g2
    uint32_t per_o[2];        // items per value of the other clock group
};
struct QSolve {
    PipeSolve S;
    uint32_t cls;
    uint32_t items[2];        // items of the two kernels (the finish waits for the last)
};
constexpr int kMaxQueues = 8;
struct QueueArgs {
    const QClass *cls;
    const QSolve *solves;
    const uint64_t *items;    // the queues' item codes, queue after queue
    const FinishJob *fin;
    unsigned *cnt;            // [2 nsolves] done counters, [kMaxQueues] heads, finished solves
    unsigned *flag;
    uint64_t wait_ticks;      // bound of one dependency wait, in wall-clock ticks
    uint32_t nsolves;
    int local;                // 1: one queue per XCC, served by that XCC's blocks; 0: one queue for all
                              // blocks, with device-scope synchronisation
    uint32_t qstart[kMaxQueues + 1];
    int qof[16];              // local: the queue of every XCC id (-1: none)
};

// the accelerator complex die (its own L2) the wave runs on
__device__ __forceinline__ int xcc_id() { return (int)(__builtin_amdgcn_s_getreg((20) | (0 << 6) | ((4 - 1) << 11)) & 15u); }

// Wait for *c >= target, bounded by `ticks` of the constant-rate wall clock
// (a quarter second): on expiry the flag is set and the item runs anyway,
// and once the flag is set no wait blocks any more, so every block drains.
// Then the acquire: a queue served by one XCC shares that XCC's L2 with its
// producers, so only the CU's vector L1 is invalidated (a line there may
// hold data another phase has since rewritten); otherwise the device-scope
// acquire (L1 and the XCC's L2).  The block barrier follows.
__device__ __forceinline__ void queue_wait(unsigned *c, unsigned target, unsigned *flag, uint64_t ticks, bool local) {
    if (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
        const uint64_t t0 = wall_clock64();
        while (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
            if (wall_clock64() - t0 > ticks) {
                __hip_atomic_fetch_or(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
    }
    if (local) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        asm volatile("buffer_inv sc0" ::: "memory");
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
}

template <typename R, int G>
__device__ __forceinline__ void queue_item(int ph, const PipeArgs &A, const PipeSolve &S, uint64_t j0, uint64_t o,
                                           uint64_t slot) {
    constexpr int RA = (G + 1) / 2, RB = G / 2;     // the register split of dispatch_g
    if (ph == 0)
        pipe_a_body<R, RA, RB, 256>(A, S, j0);
    else
        pipe_b_body<R, RA, RB, 256, true>(A, S, j0, o, slot);
}

// Every block serves one queue and takes its items from the queue's head
// until it is empty; the next item's code and the position of the one after
// it are fetched while the current one runs.  An item code holds the phase (bits 62-63: 0 and 1 the two
// kernels, 2 the finish), the solve (bits 42-61), the number of items of the
// previous phase of the solve that it waits for (bits 21-41) and the item's
// index within its phase of the solve (bits 0-20).  With one queue per XCC, a block reads the XCC it runs on and
// serves that XCC's queue: every producer and consumer of a solve then
// share one L2, and no L2 write-back or invalidation is needed (the XCCs
// present are probed when the queues are built; dispatch spreads the
// blocks of a launch over all of them, from a starting XCC that varies
// between launches).  GMAX bounds the clock groups of the batch: the registers of
// a kernel are those of its widest group, so batches of groups <= 6 bits
// get a form without the 7- and 8-bit bodies, held to four waves per SIMD
// for complex64 (128 VGPRs, a few spilled) and two for complex128 (256).
template <typename R, int GMAX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(GMAX == 6 ? (sizeof(R) == 4 ? 4 : 2) : 1))) void
k_pipe_queue(QueueArgs Q) {
    __shared__ uint64_t sh_code;
    const bool local = Q.local != 0;
    const int q = local ? Q.qof[xcc_id()] : 0;
    if (q < 0) return;
    unsigned *const head = Q.cnt + 2 * (size_t)Q.nsolves + q;
    unsigned *const finished = Q.cnt + 2 * (size_t)Q.nsolves + kMaxQueues;
    const uint32_t base = Q.qstart[q], nitems = Q.qstart[q + 1] - base;
    // thread 0: the code of the block's next item (~0: none left) and the
    // queue position of the one after, both in flight during an item
    uint64_t next_code = ~0ull;
    uint32_t pend = 0;
    if (threadIdx.x == 0) {
        const uint32_t i = __hip_atomic_fetch_add(head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (i < nitems) next_code = Q.items[base + i];
        pend = i < nitems ? __hip_atomic_fetch_add(head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : nitems;
    }
    for (;;) {
        if (threadIdx.x == 0) {
            const uint64_t code = next_code;
            if (code != ~0ull) {
                next_code = pend < nitems ? Q.items[base + pend] : ~0ull;
                if (pend < nitems) pend = __hip_atomic_fetch_add(head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const unsigned ph = (unsigned)(code >> 62), sv = (unsigned)(code >> 42) & 0xFFFFFu;
                if (ph > 0)
                    queue_wait(Q.cnt + 2 * (size_t)sv + ph - 1, (unsigned)(code >> 21) & 0x1FFFFFu, Q.flag,
                               Q.wait_ticks, local);
            }
            sh_code = code;
        }
        // also the barrier between the last item's LDS reads and this one's writes
        __syncthreads();
        const uint64_t code = sh_code;
        if (code == ~0ull) break;
        const int ph = (int)(code >> 62);
        const uint32_t sv = (uint32_t)(code >> 42) & 0xFFFFFu;
        const uint64_t t = code & 0x1FFFFFu;
        if (ph == 2) {
            batch_finish_body(Q.fin[sv]);
            if (threadIdx.x == 0) __hip_atomic_fetch_add(finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        const QSolve &qs = Q.solves[sv];
        const QClass &c = Q.cls[qs.cls];
        const PipeArgs A = c.A[ph];
        const PipeSolve S = qs.S;
        const uint64_t per = c.per_o[ph];
        const uint64_t o = t / per;
        const uint64_t j0 = ((t - o * per) * (uint64_t)A.iters) << A.cl;
        switch (c.g[ph]) {
        case 1: queue_item<R, 1>(ph, A, S, j0, o, t); break;
        case 2: queue_item<R, 2>(ph, A, S, j0, o, t); break;
        case 3: queue_item<R, 3>(ph, A, S, j0, o, t); break;
        case 4: queue_item<R, 4>(ph, A, S, j0, o, t); break;
        case 5: queue_item<R, 5>(ph, A, S, j0, o, t); break;
        case 6: queue_item<R, 6>(ph, A, S, j0, o, t); break;
        case 7:
            if (GMAX >= 7) queue_item<R, 7>(ph, A, S, j0, o, t);
            break;
        default:
            if (GMAX >= 8) queue_item<R, 8>(ph, A, S, j0, o, t);
            break;
        }
        // publish the item: every wave's stores complete (the block barrier
        // alone waits for LDS traffic only): in the XCC's L2 for a local
        // queue, else released at device scope; then one thread counts it
        if (local) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        }
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(Q.cnt + 2 * (size_t)sv + ph, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// the XCC of every block of a grid (one wave per block)
__global__ void k_xcc_probe(int *__restrict__ out) {
    if (threadIdx.x == 0) out[blockIdx.x] = xcc_id();
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------

template <typename R, int RA, int RB, int NT>
static sv_status launch_pipe(int which, hipStream_t st, const PipeSolve &one,
                             const PipeHead &head, const PipeArgs &A, dim3 grid, size_t lds) {
    // tiles above 64 KiB need a larger dynamic LDS limit; the request plus the
    // kernels' static LDS must stay within the 160 KiB of a workgroup
    constexpr int kLim = 144 * 1024;
    static bool attr_done = false;
    if (!attr_done) {
        hipError_t e0 = hipFuncSetAttribute((const void *)k_pipe_a<R, RA, RB, NT>,
                                            hipFuncAttributeMaxDynamicSharedMemorySize, kLim);
        hipError_t e1 = hipFuncSetAttribute((const void *)k_pipe_b<R, RA, RB, NT>,
                                            hipFuncAttributeMaxDynamicSharedMemorySize, kLim);
        (void)hipGetLastError();
        if (e0 != hipSuccess || e1 != hipSuccess)
            return fail(SV_EDEVICE, "cannot raise the LDS limit of the pipeline kernels");
        attr_done = true;
    }
    if (lds > (size_t)kLim) return fail(SV_EUNSUPPORTED, "pipeline tile needs %zu bytes of LDS", lds);
    // algorithmic bytes: the ancilla half is 2^(n_s + n_c) amplitudes; the G1
    // table 2^(n_s + g1)
    const double half = (double)A.N * (double)(1ull << A.n_c) * sizeof(cvec<R>);
    const double table = (double)A.N * (double)(1ull << A.g1) * sizeof(cvec<R>);
    if (which == 0) {
        TraceScope ts(st, "pipe_a_init_iqft", table, 0.0);
        dim3 g = grid;
        g.x += head.cols;
        const size_t need = head.cols ? (head.N + NT) * sizeof(double2) : 0;
        hipLaunchKernelGGL((k_pipe_a<R, RA, RB, NT>), g, dim3(NT), std::max(lds, need), st, A, one, head);
    } else {
        TraceScope ts(st, "pipe_b_iqft_ry", half + table, 0.0);
        hipLaunchKernelGGL((k_pipe_b<R, RA, RB, NT>), grid, dim3(NT), lds, st, A, one);
    }
    SV_HIP(hipGetLastError());
    return SV_OK;
}

template <typename R, int RA, int RB>
static sv_status launch_nt(int which, hipStream_t st, const PipeSolve &one,
                           const PipeHead &head, const PipeArgs &A, int nt, dim3 grid, size_t lds) {
    if (nt == 512) return launch_pipe<R, RA, RB, 512>(which, st, one, head, A, grid, lds);
    return launch_pipe<R, RA, RB, 256>(which, st, one, head, A, grid, lds);
}

template <typename R>
static sv_status dispatch_g(int which, hipStream_t st, const PipeSolve &one,
                            const PipeHead &head, const PipeArgs &A, int g, int nt, dim3 grid, size_t lds) {
    switch (g) {
    case 1: return launch_nt<R, 1, 0>(which, st, one, head, A, nt, grid, lds);
    case 2: return launch_nt<R, 1, 1>(which, st, one, head, A, nt, grid, lds);
    case 3: return launch_nt<R, 2, 1>(which, st, one, head, A, nt, grid, lds);
    case 4: return launch_nt<R, 2, 2>(which, st, one, head, A, nt, grid, lds);
    case 5: return launch_nt<R, 3, 2>(which, st, one, head, A, nt, grid, lds);
    case 6: return launch_nt<R, 3, 3>(which, st, one, head, A, nt, grid, lds);
    case 7: return launch_nt<R, 4, 3>(which, st, one, head, A, nt, grid, lds);
    case 8: return launch_nt<R, 4, 4>(which, st, one, head, A, nt, grid, lds);
    case 9: return launch_nt<R, 5, 4>(which, st, one, head, A, nt, grid, lds);
    case 10: return launch_nt<R, 5, 5>(which, st, one, head, A, nt, grid, lds);
    }
    return fail(SV_EUNSUPPORTED, "clock group of %d bits", g);
}

int pipe_supported(int n_s, int n_c) { return n_c >= 2 && n_c <= 20 && n_s >= 0; }

static const int PIPE_LDS_LIMIT = 144 * 1024;

// columns per tile for a group of g bits by default (tile of at most 2^13
// c64 / 2^12 c128 amplitudes)
static int default_cl(int n_s, int g, size_t elem) {
    const int tile_log = elem == 8 ? 13 : 12;
    int cl = tile_log - g;
    if (cl > 6) cl = 6;
    if (cl > n_s) cl = n_s;
    if (cl < 0) cl = 0;
    return cl;
}

static size_t pipe_lds(int which, int cl, int g, size_t e) {
    const size_t C = (size_t)1 << cl;
    if (which == 0)        // the twiddles and the column phases (FP64)
        return (((size_t)1 << g) + (size_t)g * C) * sizeof(double2);
    // the twiddles, two rotation tables, two sets of column data and of line sums
    return ((size_t)1 << g) * e + 2 * ((size_t)1 << g) * (e / 2) + 2 * (size_t)(g + 2) * C * e +
           2 * (C << ((g + 1) / 2)) * (e / 2);
}

struct PipePlan {
    PipeArgs A[2];
    int nt[2];
    dim3 grid[2];
    size_t lds[2];
};

static void make_plan(PipePlan &P, int n_s, int n_c, size_t e, const int cl[2], const int nt[2]) {
    PipeArgs A;
    A.N = dim_of(n_s);
    A.n_s = n_s;
    A.n_c = n_c;
    A.g1 = (n_c + 1) / 2;
    A.g2 = n_c - A.g1;
    A.abit = 1ull << (n_s + n_c);
    A.scale = 1.0 / sqrt((double)(1ull << n_c));
    A.sgn = 0;
    A.gcut = 0;
    A.iters = 1;
    for (int w = 0; w < 2; ++w) {
        const int g = w == 1 ? A.g2 : A.g1;
        P.A[w] = A;
        const int c = cl[w];
        P.A[w].cl = c;
        P.nt[w] = nt[w];
        // k_pipe_a writes the G1 table only (G2 value 0)
        const uint64_t tiles = w == 0 ? (A.N >> c) : (A.N >> c) << (n_c - g);
        P.grid[w] = tiles <= 0x7fffffffull ? dim3((unsigned)tiles)
                                           : dim3(1u << 30, (unsigned)(tiles >> 30));
        P.lds[w] = pipe_lds(w, c, g, e);
    }
}

template <typename R>
static sv_status run_one(hipStream_t st, const PipePlan &P, int w, const PipeSolve &one, const PipeHead &head = {}) {
    const int g = w == 1 ? P.A[w].g2 : P.A[w].g1;
    return dispatch_g<R>(w, st, one, head, P.A[w], g, P.nt[w], P.grid[w], P.lds[w]);
}

// The autotuner: per (dtype, n_s, n_c) time every feasible (columns per
// tile, threads per workgroup) for each of the two kernels on the real
// operands of one solve (each kernel is idempotent given its input half)
// and keep the fastest; results live in the process-wide tuning cache.
template <typename R>
static sv_status tune_pipe(hipStream_t st, int n_s, int n_c, const PipeSolve &one, int cl_out[2],
                           int nt_out[2]) {
    const size_t e = sizeof(cvec<R>);
    const int g1 = (n_c + 1) / 2, g2 = n_c - g1;
    for (int w = 0; w < 2; ++w) {
        cl_out[w] = default_cl(n_s, w == 1 ? g2 : g1, e);
        nt_out[w] = 256;
    }
    for (int w = 0; w < 2; ++w) {
        const int g = w == 1 ? g2 : g1;
        // Every candidate is timed in two alternating rounds and keeps its
        // faster one: single timings of a few-millisecond kernel differ by
        // more than the candidates do.
        std::vector<std::pair<int, int>> cand;
        for (int cl = 3; cl <= 7; ++cl) {
            if (cl > n_s) break;
            for (int nt : {256, 512})
                if (pipe_lds(w, cl, g, e) <= (size_t)PIPE_LDS_LIMIT) cand.push_back({cl, nt});
        }
        std::vector<float> tbest(cand.size(), 1e30f);
        for (int round = 0; round < 2; ++round)
            for (size_t i = 0; i < cand.size(); ++i) {
                int cls[2] = {cl_out[0], cl_out[1]}, nts[2] = {nt_out[0], nt_out[1]};
                cls[w] = cand[i].first;
                nts[w] = cand[i].second;
                PipePlan P;
                make_plan(P, n_s, n_c, e, cls, nts);
                float ms = 0.f;
                SV_TRY(time_stream(st, 2, &ms, [&]() { return run_one<R>(st, P, w, one); }));
                if (ms < tbest[i]) tbest[i] = ms;
            }
        int bcl = cl_out[w], bnt = nt_out[w];
        float best = 1e30f;
        for (size_t i = 0; i < cand.size(); ++i)
            if (tbest[i] < best) {
                best = tbest[i];
                bcl = cand[i].first;
                bnt = cand[i].second;
            }
        cl_out[w] = bcl;
        nt_out[w] = bnt;
        // the next kernel reads what this one writes: leave its output in place
        PipePlan P;
        make_plan(P, n_s, n_c, e, cl_out, nt_out);
        SV_TRY(run_one<R>(st, P, w, one));
    }
    return SV_OK;
}

// a cached choice of the launch parameters (an entry's third pair belonged to a
// third kernel; it is kept as zeros so that saved entries of either kind serve)
static bool pipe_cached(const std::string &key, int cl[2], int nt[2]) {
    std::vector<int> cached;
    if (!tune_lookup(key, cached) || cached.size() != 6) return false;
    for (int w = 0; w < 2; ++w) {
        cl[w] = cached[2 * w];
        nt[w] = cached[2 * w + 1];
    }
    return true;
}

static std::string pipe_key(int n_s, int n_c, size_t e) {
    return std::string("eigpipe/") + (e == 8 ? "c64/" : "c128/") + std::to_string(n_s) + "/" + std::to_string(n_c);
}

// launch parameters for a shape: cached, tuned on `one` if allowed, else defaults
template <typename R>
static sv_status pipe_config(hipStream_t st, int n_s, int n_c, const PipeSolve &one, int cl[2], int nt[2]) {
    const size_t e = sizeof(cvec<R>);
    const int g1 = (n_c + 1) / 2, g2 = n_c - g1;
    const std::string key = pipe_key(n_s, n_c, e);
    if (pipe_cached(key, cl, nt)) return SV_OK;
    if (autotune_enabled()) {
        SV_TRY(tune_pipe<R>(st, n_s, n_c, one, cl, nt));
        tune_store(key, {cl[0], nt[0], cl[1], nt[1], 0, 0});
        return SV_OK;
    }
    for (int w = 0; w < 2; ++w) {
        cl[w] = default_cl(n_s, w == 1 ? g2 : g1, e);
        nt[w] = 256;
    }
    return SV_OK;
}

void pipe_config_batch(int n_s, int n_c, size_t elem, int cl[2]) {
    const int g1 = (n_c + 1) / 2;
    int nt[2];
    if (pipe_cached(pipe_key(n_s, n_c, elem), cl, nt)) return;
    cl[0] = default_cl(n_s, g1, elem);
    cl[1] = default_cl(n_s, n_c - g1, elem);
}

template <typename R>
sv_status pipe_run(sv_state s, int n_s, int n_c, bool sgn, uint64_t gcut, const PipeHead &head, const double2 *beta, const double *lam,
                   double T0, DevBuf &part, double *zpart, uint64_t *nparts) {
    const size_t e = sizeof(cvec<R>);
    SV_TRY(part.ensure(2 * pipe_b_blocks(n_s, n_c, e) * sizeof(double)));     // every candidate of the tuner
    PipeSolve one{s->data, beta, lam, T0, (double *)part.p, zpart};
    int cl[2], nt[2];
    SV_TRY(pipe_config<R>(s->stream, n_s, n_c, one, cl, nt));
    PipePlan P;
    make_plan(P, n_s, n_c, e, cl, nt);
    for (int w = 0; w < 2; ++w) {
        P.A[w].sgn = sgn ? 1 : 0;
        P.A[w].gcut = gcut;
    }
    *nparts = (uint64_t)P.grid[1].x * P.grid[1].y;
    // a default of few columns per tile (complex128, 2^10 clock values per group)
    // or a pinned one has more tiles than the tuner's candidates
    SV_TRY(part.ensure(2 * *nparts * sizeof(double)));
    one.part = (double *)part.p;
    for (int w = 0; w < 2; ++w) SV_TRY(run_one<R>(s->stream, P, w, one, head));
    return SV_OK;
}
template sv_status pipe_run<float>(sv_state, int, int, bool, uint64_t, const PipeHead &, const double2 *,
                                   const double *, double, DevBuf &, double *, uint64_t *);
template sv_status pipe_run<double>(sv_state, int, int, bool, uint64_t, const PipeHead &, const double2 *,
                                    const double *, double, DevBuf &, double *, uint64_t *);

// ---------------------------------------------------------------------------
// the work queues' plan: items of about 2^15 amplitudes (runs of consecutive
// column blocks for k_pipe_b); the solves spread over one
// queue per XCC, each queue numbered phase-major, its solves largest first
// ---------------------------------------------------------------------------
template <typename R>
sv_status pipe_queue_build(sv_state ctx, hipStream_t st, PipeQueue &q, DevBuf &desc,
                           const std::vector<QueueClassIn> &cls, const std::vector<int> &solve_cls,
                           const std::vector<PipeSolve> &solves, unsigned *cnt, unsigned *flag) {
    (void)st;
    const size_t e = sizeof(cvec<R>);
    const int ns = (int)solves.size();
    if (ns < 1 || ns >= (1 << 20) || solve_cls.size() != solves.size())
        return fail(SV_EINVAL, "work queue of %d solves", ns);
    constexpr int kLim = 144 * 1024;
    static bool attr_done = false;
    if (!attr_done) {
        const hipError_t h6 =
            hipFuncSetAttribute((const void *)k_pipe_queue<R, 6>, hipFuncAttributeMaxDynamicSharedMemorySize, kLim);
        const hipError_t h8 =
            hipFuncSetAttribute((const void *)k_pipe_queue<R, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, kLim);
        (void)hipGetLastError();
        if (h6 != hipSuccess || h8 != hipSuccess) return fail(SV_EDEVICE, "cannot raise the LDS limit of the queue kernel");
        attr_done = true;
    }
    std::vector<QClass> qc(cls.size());
    size_t lds = 0;
    int gmax = 1;
    for (size_t k = 0; k < cls.size(); ++k) {
        const QueueClassIn &ci = cls[k];
        const int nt[2] = {256, 256};
        PipePlan P;
        make_plan(P, ci.n_s, ci.n_c, e, ci.cl, nt);
        for (int w = 0; w < 2; ++w) {
            PipeArgs A = P.A[w];
            const int g = w == 1 ? A.g2 : A.g1;
            // tiles of at most 2^11 amplitudes: LDS for four blocks per CU
            while (A.cl > 0 && ((1ull << A.cl) << g) > (1ull << 11)) --A.cl;
            const uint64_t C = 1ull << A.cl, nb = A.N >> A.cl;
            int iters = 1;
            // a run of column blocks reads each next block's column data ahead
            if (w > 0)
                while ((uint64_t)iters < nb && (((uint64_t)iters * 2 * C) << g) <= (1ull << 15)) iters *= 2;
            A.iters = iters;
            qc[k].A[w] = A;
            qc[k].g[w] = g;
            if (g > gmax) gmax = g;
            qc[k].per_o[w] = (uint32_t)(nb / (uint64_t)iters);
            const size_t b = pipe_lds(w, A.cl, g, e);
            if (b > lds) lds = b;
        }
    }
    if (lds > (size_t)kLim) return fail(SV_EUNSUPPORTED, "queue items need %zu bytes of LDS", lds);
    std::vector<QSolve> qs(ns);
    std::vector<double> cost(ns);
    q.nparts.assign(ns, 0);
    double bytes = 0.0;
    for (int k = 0; k < ns; ++k) {
        const QClass &c = qc[solve_cls[k]];
        qs[k].S = solves[k];
        qs[k].cls = (uint32_t)solve_cls[k];
        const int g1 = c.A[0].g1;
        qs[k].items[0] = c.per_o[0];
        qs[k].items[1] = c.per_o[1] << g1;
        q.nparts[k] = qs[k].items[1];
        if (q.nparts[k] > pipe_b_blocks(c.A[0].n_s, c.A[0].n_c, e))
            return fail(SV_EDEVICE, "queue partials exceed their buffer");
        const double half = (double)c.A[0].N * (double)(1ull << c.A[0].n_c) * e;
        const double table = (double)c.A[0].N * (double)(1ull << g1) * e;
        cost[k] = half + 2.0 * table;      // as if stored: the balance of the queues
        bytes += 2.0 * table;
    }
    // resident blocks, and the XCC each of them lands on
    // the queue kernel carries bodies for clock groups of up to 8 bits; a
    // batch with wider groups runs its classes' own kernels instead
    if (gmax > 8) return fail(SV_EUNSUPPORTED, "work queue for clock groups of %d bits", gmax);
    q.gmax = gmax <= 6 ? 6 : 8;
    const void *kfn = q.gmax == 6 ? (const void *)k_pipe_queue<R, 6> : (const void *)k_pipe_queue<R, 8>;
    int per_cu = 0, dev = 0, ncu = 0, khz = 0;
    SV_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, 256, lds));
    SV_HIP(hipGetDevice(&dev));
    SV_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    SV_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (per_cu < 1) return fail(SV_EUNSUPPORTED, "the queue kernel does not fit a CU with %zu bytes of LDS", lds);
    q.wait_ticks = (uint64_t)(khz > 0 ? khz : 100000) * 250;     // 0.25 s
    q.blocks = per_cu * ncu;
    std::vector<int> ids(q.blocks);
    {
        DevBuf probe;
        SV_TRY(probe.alloc(ids.size() * sizeof(int)));
        hipLaunchKernelGGL(k_xcc_probe, dim3((unsigned)q.blocks), dim3(256), 0, ctx->stream, (int *)probe.p);
        SV_HIP(hipGetLastError());
        SV_TRY(download(ctx, ids.data(), probe.p, ids.size() * sizeof(int)));
    }
    // queues: one per XCC that the probe's blocks landed on (each held an
    // even share of them), else one queue with device-scope synchronisation
    std::vector<int> distinct, count;
    for (int b = 0; b < q.blocks; ++b) {
        const auto it = std::find(distinct.begin(), distinct.end(), ids[b]);
        if (it == distinct.end()) {
            distinct.push_back(ids[b]);
            count.push_back(1);
        } else {
            ++count[it - distinct.begin()];
        }
    }
    const int D = (int)distinct.size();
    // SV_QUEUE_LOCAL=0 forces the single queue with device-scope
    // synchronisation (the fallback), so that it can be tested on any box
    const char *lenv = getenv("SV_QUEUE_LOCAL");
    bool even = D >= 1 && D <= kMaxQueues && !(lenv && atoi(lenv) == 0);
    for (int i = 0; i < D && even; ++i) even = distinct[i] >= 0 && distinct[i] < 16 && count[i] * D >= q.blocks / 2;
    if (even) {
        std::sort(distinct.begin(), distinct.end());
        q.nq = D;
        for (int i = 0; i < D; ++i) q.xcc[i] = distinct[i];
    } else {
        q.nq = 1;
        q.xcc[0] = -1;
    }
    // solves to queues, longest first to the least loaded queue
    std::vector<int> order(ns);
    for (int k = 0; k < ns; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost[x] > cost[y]; });
    std::vector<std::vector<int>> members(q.nq);
    std::vector<double> load(q.nq, 0.0);
    for (int k : order) {
        int best = 0;
        for (int i = 1; i < q.nq; ++i)
            if (load[i] < load[best]) best = i;
        members[best].push_back(k);
        load[best] += cost[k];
    }
    // each queue phase-major, its solves largest first; a code carries the
    // item count its wait targets (that of the solve's previous phase)
    for (int k = 0; k < ns; ++k)
        for (int ph = 0; ph < 2; ++ph)
            if (qs[k].items[ph] >= (1u << 21))
                return fail(SV_EUNSUPPORTED, "%u items in one phase of a solve", qs[k].items[ph]);
    std::vector<uint64_t> items;
    for (int i = 0; i < q.nq; ++i) {
        q.qstart[i] = (uint32_t)items.size();
        for (int ph = 0; ph < 2; ++ph)
            for (int k : members[i]) {
                q.items_per_phase[ph] += qs[k].items[ph];
                const uint64_t wait = ph > 0 ? qs[k].items[ph - 1] : 0;
                for (uint64_t t = 0; t < qs[k].items[ph]; ++t)
                    items.push_back(((uint64_t)ph << 62) | ((uint64_t)k << 42) | (wait << 21) | t);
            }
        for (int k : members[i]) items.push_back((2ull << 62) | ((uint64_t)k << 42) | ((uint64_t)qs[k].items[1] << 21));
        if (items.size() >= 0xffffffffull) return fail(SV_EUNSUPPORTED, "work queue of %zu items", items.size());
    }
    q.qstart[q.nq] = (uint32_t)items.size();
    q.items_per_phase[2] = (uint64_t)ns;
    // descriptors: classes, solves, item codes
    const size_t o_cls = 0, o_sol = (qc.size() * sizeof(QClass) + 255) & ~(size_t)255;
    const size_t o_items = o_sol + ((qs.size() * sizeof(QSolve) + 255) & ~(size_t)255);
    SV_TRY(desc.alloc(o_items + items.size() * sizeof(uint64_t)));
    char *d = (char *)desc.p;
    SV_TRY(upload(ctx, d + o_cls, qc.data(), qc.size() * sizeof(QClass)));
    SV_TRY(upload(ctx, d + o_sol, qs.data(), qs.size() * sizeof(QSolve)));
    SV_TRY(upload(ctx, d + o_items, items.data(), items.size() * sizeof(uint64_t)));
    q.d_cls = d + o_cls;
    q.d_solves = d + o_sol;
    q.d_items = (const uint64_t *)(d + o_items);
    q.nitems = (uint32_t)items.size();
    q.nsolves = (uint32_t)ns;
    q.cnt = cnt;
    q.flag = flag;
    q.lds = lds;
    q.bytes = bytes;
    return SV_OK;
}

template <typename R>
sv_status pipe_queue_launch(hipStream_t st, const PipeQueue &q, const FinishJob *d_fin) {
    QueueArgs Q;
    Q.cls = (const QClass *)q.d_cls;
    Q.solves = (const QSolve *)q.d_solves;
    Q.items = q.d_items;
    Q.fin = d_fin;
    Q.cnt = q.cnt;
    Q.flag = q.flag;
    Q.wait_ticks = q.wait_ticks;
    Q.nsolves = q.nsolves;
    Q.local = q.xcc[0] >= 0 ? 1 : 0;
    for (int i = 0; i <= kMaxQueues; ++i) Q.qstart[i] = i <= q.nq ? q.qstart[i] : q.qstart[q.nq];
    for (int i = 0; i < 16; ++i) Q.qof[i] = -1;
    if (Q.local)
        for (int i = 0; i < q.nq; ++i) Q.qof[q.xcc[i]] = i;
    TraceScope ts(st, "pipe_queue", q.bytes, 0.0);
    if (q.gmax == 6)
        hipLaunchKernelGGL((k_pipe_queue<R, 6>), dim3((unsigned)q.blocks), dim3(256), q.lds, st, Q);
    else
        hipLaunchKernelGGL((k_pipe_queue<R, 8>), dim3((unsigned)q.blocks), dim3(256), q.lds, st, Q);
    SV_HIP(hipGetLastError());
    return SV_OK;
}
template sv_status pipe_queue_build<float>(sv_state, hipStream_t, PipeQueue &, DevBuf &,
                                           const std::vector<QueueClassIn> &, const std::vector<int> &,
                                           const std::vector<PipeSolve> &, unsigned *, unsigned *);
template sv_status pipe_queue_build<double>(sv_state, hipStream_t, PipeQueue &, DevBuf &,
                                            const std::vector<QueueClassIn> &, const std::vector<int> &,
                                            const std::vector<PipeSolve> &, unsigned *, unsigned *);
template sv_status pipe_queue_launch<float>(hipStream_t, const PipeQueue &, const FinishJob *);
template sv_status pipe_queue_launch<double>(hipStream_t, const PipeQueue &, const FinishJob *);

uint64_t pipe_b_blocks_for(int n_s, int n_c, int cl) {
    const int g1 = (n_c + 1) / 2;
    return (dim_of(n_s) >> cl) << g1;
}

// upper bounds of the k_pipe_b block count (one FP64 partial pair each) and
// the rows of column sums, over every configuration the tuner may pick
uint64_t pipe_b_blocks(int n_s, int n_c, size_t elem) {
    (void)elem;
    return pipe_b_blocks_for(n_s, n_c, n_s < 3 ? n_s : 3);
}
int pipe_rows(int n_c) { return 1 << ((n_c + 1) / 2); }
int pipe_table_rows(int n_c) { return pipe_rows(n_c) + n_c - (n_c + 1) / 2; }

}  // namespace sv
