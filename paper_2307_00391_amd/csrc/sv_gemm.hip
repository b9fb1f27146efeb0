// Controlled dense unitary on a register of m qubits [lo, lo + m) as a
// complex GEMM on the matrix cores (MFMA): every amplitude row whose control
// bits match is a length-2^m vector v, replaced by U v.  Rows are gathered
// straight from the state (row r starts at pdep(r, row_mask) | row_fix, its
// element k at stride 2^lo), multiplied out of place into a compact buffer
// and scattered back.  complex64 uses v_mfma_f32_16x16x4f32 (FP32 in, FP32 accumulate);
// complex128 uses v_mfma_f64_16x16x4f64.  A complex product is four real
// MFMAs: re += ar br - ai bi, im += ar bi + ai br.
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "sv_device.h"
#include "sv_internal.h"

namespace sv {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename R> struct MfmaT;
// Operands of both: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16].
// Results: the FP32 form keeps four consecutive rows per lane group
// (row 4 (l / 16) + v), the FP64 form interleaves them (row l / 16 + 4 v);
// the column is l % 16 in both.
template <> struct MfmaT<float> {
    using acc = floatx4;
    static __device__ __forceinline__ acc mfma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) * 4 + v; }
};
template <> struct MfmaT<double> {
    using acc = doublex4;
    static __device__ __forceinline__ acc mfma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};

constexpr int GBM = 64, GBN = 64, GBK = 16;

template <typename R>
struct GemmArgs {
    const cvec<R> *in;   // rows of length K
    cvec<R> *out;        // M x N, row-major, compact
    const cvec<R> *U;    // B(kk, n) = trans ? U[kk * N + n] : U[n * K + kk]  (conj if conjb)
    uint64_t M;
    int N, K;
    uint64_t row_mask, row_fix;   // row r starts at pdep(r, row_mask) | row_fix
    int ksh;                      // element k of a row at offset k << ksh
    int trans, conjb;
};

// 256 threads: 4 waves as 2 x 2, each wave a 32 x 32 output block made of
// 2 x 2 MFMA 16 x 16 tiles.  Operands are staged in LDS as separate real and
// imaginary planes, k-major, so the 16 lanes that share a k read 16
// consecutive words; the next k step's operands are in flight (in
// registers) while a step's MFMAs run.
template <typename R>
__global__ __launch_bounds__(256) void k_cgemm(GemmArgs<R> A) {
    using M_ = MfmaT<R>;
    using acc_t = typename M_::acc;
    __shared__ R As_re[GBK][GBM], As_im[GBK][GBM], Bs_re[GBK][GBN], Bs_im[GBK][GBN];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const uint64_t row0 = (uint64_t)blockIdx.x * GBM;
    const int n0 = blockIdx.y * GBN;

    // this thread's A-load row and its base offset in the state: four
    // threads along k per row when the row is contiguous (ksh = 0), else one
    // row per lane, so that a wavefront reads 64 neighbouring rows
    const int a_row = A.ksh ? (tid & 63) : tid >> 2, a_k = A.ksh ? (tid >> 6) * 4 : (tid & 3) * 4;
    const uint64_t ar = row0 + a_row;
    const bool a_ok = ar < A.M;
    const uint64_t a_base = a_ok ? (pdep64(ar, A.row_mask) | A.row_fix) : 0;

    acc_t acc_re[2][2], acc_im[2][2];
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j)
            for (int v = 0; v < 4; ++v) acc_re[i][j][v] = acc_im[i][j][v] = (R)0;

    const R csgn = A.conjb ? (R)-1 : (R)1;
    // The next k step's operands are loaded into registers while this step's
    // MFMAs run, and written to the LDS after the step's closing barrier.
    // Thread roles: A rows as above; B as (n, four k) or (k, four n).
    const int b_n = A.trans ? (tid & 15) * 4 : tid >> 2, b_k = A.trans ? tid >> 4 : (tid & 3) * 4;
    cvec<R> pa[4], pb[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kk = k0 + a_k + i;
            pa[i] = cmake<R>((R)0, (R)0);
            if (a_ok && kk < A.K) pa[i] = A.in[a_base + ((uint64_t)kk << A.ksh)];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pb[i] = cmake<R>((R)0, (R)0);
            if (!A.trans) {
                const int kk = k0 + b_k + i, nn = n0 + b_n;
                if (kk < A.K && nn < A.N) pb[i] = A.U[(uint64_t)nn * A.K + kk];
            } else {
                const int kk = k0 + b_k, nn = n0 + b_n + i;
                if (kk < A.K && nn < A.N) pb[i] = A.U[(uint64_t)kk * A.N + nn];
            }
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < A.K; k0 += GBK) {
        // A tile: 64 rows x 16 k; B tile: 16 k x 64 n
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            As_re[a_k + i][a_row] = pa[i].x;
            As_im[a_k + i][a_row] = pa[i].y;
            const int bk = A.trans ? b_k : b_k + i, bn = A.trans ? b_n + i : b_n;
            Bs_re[bk][bn] = pb[i].x;
            Bs_im[bk][bn] = csgn * pb[i].y;
        }
        __syncthreads();
        if (k0 + GBK < A.K) fetch(k0 + GBK);
#pragma unroll
        for (int kc = 0; kc < GBK / 4; ++kc) {
            const int kr = kc * 4 + (lane >> 4), li = lane & 15;
            R ar_[2], ai_[2], br_[2], bi_[2];
            for (int i = 0; i < 2; ++i) {
                ar_[i] = As_re[kr][wm * 32 + i * 16 + li];
                ai_[i] = As_im[kr][wm * 32 + i * 16 + li];
                br_[i] = Bs_re[kr][wn * 32 + i * 16 + li];
                bi_[i] = Bs_im[kr][wn * 32 + i * 16 + li];
            }
            for (int i = 0; i < 2; ++i)
                for (int j = 0; j < 2; ++j) {
                    acc_re[i][j] = M_::mfma(ar_[i], br_[j], acc_re[i][j]);
                    acc_re[i][j] = M_::mfma(-ai_[i], bi_[j], acc_re[i][j]);
                    acc_im[i][j] = M_::mfma(ar_[i], bi_[j], acc_im[i][j]);
                    acc_im[i][j] = M_::mfma(ai_[i], br_[j], acc_im[i][j]);
                }
        }
        __syncthreads();
    }
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j)
            for (int v = 0; v < 4; ++v) {
                const uint64_t r = row0 + wm * 32 + i * 16 + M_::row(lane, v);
                const int c = n0 + wn * 32 + j * 16 + (lane & 15);
                if (r < A.M && c < A.N) A.out[r * A.N + c] = cmake<R>(acc_re[i][j][v], acc_im[i][j][v]);
            }
}

// The same product with one wavefront per 16 x 16 output tile and no LDS:
// each lane loads its MFMA operands straight from memory (A[row][k] for row
// l % 16, k = l / 16 of each 4-wide k step, and B[k][col] alike).  For small
// products (the basis changes of a Kronecker plan: 256 x 256 x 256) the
// 64 x 64 block tiles leave most of the chip idle; here every tile is a
// wavefront.  The k steps and the four real MFMAs of a complex product run in
// the same order as in k_cgemm, so both give the same bits.
template <typename R>
__global__ __launch_bounds__(256) void k_cgemm_w(GemmArgs<R> A) {
    using M_ = MfmaT<R>;
    using acc_t = typename M_::acc;
    const int lane = threadIdx.x & 63;
    const uint64_t tiles_n = (uint64_t)((A.N + 15) / 16);
    const uint64_t tile = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint64_t tm = tile / tiles_n, tn = tile % tiles_n;
    if (tm * 16 >= A.M) return;                       // the whole wavefront (no barriers below)
    const uint64_t r = tm * 16 + (lane & 15);
    const int c = (int)(tn * 16) + (lane & 15);
    const int kq = lane >> 4;
    const bool r_ok = r < A.M, c_ok = c < A.N;
    const uint64_t a_base = r_ok ? (pdep64(r, A.row_mask) | A.row_fix) : 0;
    const R csgn = A.conjb ? (R)-1 : (R)1;
    acc_t acc_re, acc_im;
    for (int v = 0; v < 4; ++v) acc_re[v] = acc_im[v] = (R)0;
#pragma unroll 4
    for (int k0 = 0; k0 < A.K; k0 += 4) {
        const int kk = k0 + kq;
        cvec<R> a = cmake<R>((R)0, (R)0), b = cmake<R>((R)0, (R)0);
        if (r_ok && kk < A.K) a = A.in[a_base + ((uint64_t)kk << A.ksh)];
        if (c_ok && kk < A.K) b = A.trans ? A.U[(uint64_t)kk * A.N + c] : A.U[(uint64_t)c * A.K + kk];
        acc_re = M_::mfma(a.x, b.x, acc_re);
        acc_re = M_::mfma(-a.y, csgn * b.y, acc_re);
        acc_im = M_::mfma(a.x, csgn * b.y, acc_im);
        acc_im = M_::mfma(a.y, b.x, acc_im);
    }
    for (int v = 0; v < 4; ++v) {
        const uint64_t rr = tm * 16 + M_::row(lane, v);
        if (rr < A.M && c_ok) A.out[rr * A.N + c] = cmake<R>(acc_re[v], acc_im[v]);
    }
}

// Small products: a workgroup computes (16 TA) x (16 TB) outputs with KS groups
// of TA TB wavefronts, each group one KS-th of the k range, so that products of
// a few hundred rows and columns still give every SIMD a wavefront or more:
//   16 x 16, k in four parts:   256 x 256 outputs are 256 workgroups;
//   32 x 32, k in two parts:    1024 x 256 outputs are 256 workgroups of 8 waves.
// Operands go through LDS (16 k at a time, whole amplitudes, one pad column so
// that the k-major rows fall on different banks), two stages; the next two are
// in registers while one is multiplied.  The parts are added in order.  A
// wavefront per tile straight from memory (k_cgemm_w) leaves three SIMDs of
// four idle at 256 x 256 and waits for its 64-byte pieces of 16 rows.  Bound:
// the latency of the operand loads (a third of the FP64 matrix rate at 1024 x
// 256 x 256).  Controlled unitary on the given rows, copy back included, N = K
// = 256, complex128: 256 rows 36.4 -> 13.5 us, 512 rows 37.7 -> 17.3, 1024 rows
// 40.0 -> 23.4; complex64: 23.9 -> 11.3, 24.5 -> 13.4, 25.8 -> 16.3.  At 2048 x
// 1024 the 64 x 64 tiles are as fast.
template <typename R, int TA, int TB, int KS>
__global__ __launch_bounds__(64 * TA * TB * KS) void k_cgemm_k(GemmArgs<R> A) {
    using M_ = MfmaT<R>;
    using acc_t = typename M_::acc;
    constexpr int PT = 64 * TA * TB, TM = 16 * TA, TN = 16 * TB, KC = 16;
    constexpr int NA = TM * KC / PT, NB = TN * KC / PT;
    struct Stage {
        cvec<R> a[KC][TM + 1], b[KC][TN + 1];
    };
    constexpr int NW = TA * TB;
    union Lds {
        Stage st[2][KS];
        R red[KS > 1 ? KS - 1 : 1][NW][8][64];
    };
    __shared__ Lds lds;
    const int part = threadIdx.x / PT, pt = threadIdx.x % PT, lane = pt & 63, wave = pt >> 6;
    const int wm = wave / TB, wn = wave % TB;
    const uint64_t row0 = (uint64_t)blockIdx.x * TM;
    const int n0 = blockIdx.y * TN;
    const int chunks = (A.K + KC * KS - 1) / (KC * KS);
    const int kbeg = part * chunks * KC, kend = kbeg + chunks * KC < A.K ? kbeg + chunks * KC : A.K;

    // this thread's elements: lanes along k where k is contiguous in memory
    // (16 of them: 128 or 256 bytes), along rows or columns otherwise
    int a_row[NA], a_k[NA], b_n[NB], b_k[NB];
    uint64_t a_base[NA];
    bool a_ok[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int e = pt + i * PT;
        a_row[i] = A.ksh ? e % TM : e / KC;
        a_k[i] = A.ksh ? e / TM : e % KC;
        const uint64_t r = row0 + (uint64_t)a_row[i];
        a_ok[i] = r < A.M;
        a_base[i] = a_ok[i] ? (pdep64(r, A.row_mask) | A.row_fix) : 0;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int e = pt + i * PT;
        b_n[i] = A.trans ? e % TN : e / KC;
        b_k[i] = A.trans ? e / TN : e % KC;
    }
    const R csgn = A.conjb ? (R)-1 : (R)1;
    struct Regs {
        cvec<R> a[NA], b[NB];
    };
    auto fetch = [&](int ch, Regs &p) {
        const int k0 = kbeg + ch * KC;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int kk = k0 + a_k[i];
            p.a[i] = cmake<R>((R)0, (R)0);
            if (a_ok[i] && kk < kend) p.a[i] = A.in[a_base[i] + ((uint64_t)kk << A.ksh)];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int kk = k0 + b_k[i], nn = n0 + b_n[i];
            p.b[i] = cmake<R>((R)0, (R)0);
            if (kk < kend && nn < A.N) p.b[i] = A.trans ? A.U[(uint64_t)kk * A.N + nn] : A.U[(uint64_t)nn * A.K + kk];
        }
    };
    auto stage = [&](Stage &S, const Regs &p) {
#pragma unroll
        for (int i = 0; i < NA; ++i) S.a[a_k[i]][a_row[i]] = p.a[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) S.b[b_k[i]][b_n[i]] = cmake<R>(p.b[i].x, csgn * p.b[i].y);
    };
    acc_t acc_re, acc_im;
    for (int v = 0; v < 4; ++v) acc_re[v] = acc_im[v] = (R)0;
    auto multiply = [&](const Stage &S) {
#pragma unroll
        for (int kc = 0; kc < KC / 4; ++kc) {
            const int kr = kc * 4 + (lane >> 4), li = lane & 15;
            const cvec<R> a = S.a[kr][wm * 16 + li], b = S.b[kr][wn * 16 + li];
            acc_re = M_::mfma(a.x, b.x, acc_re);
            acc_im = M_::mfma(a.x, b.y, acc_im);
            acc_re = M_::mfma(-a.y, b.y, acc_re);
            acc_im = M_::mfma(a.y, b.x, acc_im);
        }
    };
    // two chunks ahead in registers, one in LDS (fetches past the end read nothing)
    Regs p0, p1;
    fetch(0, p0);
    fetch(1, p1);
    stage(lds.st[0][part], p0);
    __syncthreads();
    for (int ch = 0; ch < chunks; ch += 2) {
        fetch(ch + 2, p0);
        multiply(lds.st[0][part]);
        stage(lds.st[1][part], p1);
        __syncthreads();
        if (ch + 1 >= chunks) break;
        fetch(ch + 3, p1);
        multiply(lds.st[1][part]);
        stage(lds.st[0][part], p0);
        __syncthreads();
    }
    if (KS > 1) {
        if (part > 0)
            for (int v = 0; v < 4; ++v) {
                lds.red[part - 1][wave][v][lane] = acc_re[v];
                lds.red[part - 1][wave][4 + v][lane] = acc_im[v];
            }
        __syncthreads();
        if (part > 0) return;
        for (int p = 0; p < KS - 1; ++p)
            for (int v = 0; v < 4; ++v) {
                acc_re[v] += lds.red[p][wave][v][lane];
                acc_im[v] += lds.red[p][wave][4 + v][lane];
            }
    }
    for (int v = 0; v < 4; ++v) {
        const uint64_t r = row0 + wm * 16 + M_::row(lane, v);
        const int c = n0 + wn * 16 + (lane & 15);
        if (r < A.M && c < A.N) A.out[r * A.N + c] = cmake<R>(acc_re[v], acc_im[v]);
    }
}

// Rows of 256 elements and more, contiguous in the state: a workgroup copies
// 256 elements of four rows, whose numbers (and so their bit deposits, a loop
// over the row bits) are uniform.  With the deposit per element the copy of
// 1024 rows of 256 took 6.5 us.
template <typename R>
__global__ __launch_bounds__(256) void k_scatter_long(cvec<R> *__restrict__ psi, const cvec<R> *__restrict__ src,
                                                      int mbits, uint64_t row_mask, uint64_t row_fix) {
    const int per = mbits - 8;                                     // log2 of a row's 256-element pieces
    const uint64_t piece0 = (uint64_t)blockIdx.x * 4;              // (M is a power of two: four whole pieces)
    cvec<R> v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = src[((piece0 + q) << 8) + threadIdx.x];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t p = piece0 + q;
        psi[(pdep64(p >> per, row_mask) | row_fix) + ((p & ((1ull << per) - 1ull)) << 8) + threadIdx.x] = v[q];
    }
}

template <typename R>
__global__ void k_scatter_rows(cvec<R> *__restrict__ psi, const cvec<R> *__restrict__ src, uint64_t M, int mbits,
                               uint64_t row_mask, uint64_t row_fix, int ksh) {
    const uint64_t total = M << mbits;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t cm = (1ull << mbits) - 1ull;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint64_t r = i >> mbits;
        psi[(pdep64(r, row_mask) | row_fix) + ((i & cm) << ksh)] = src[i];
    }
}

// host: Out(M x N) = rows(In) * B, with B as described in GemmArgs
template <typename R>
static sv_status cgemm_ks(hipStream_t st, const cvec<R> *in, cvec<R> *out, const cvec<R> *U, uint64_t M, int N,
                          int K, uint64_t row_mask, uint64_t row_fix, int ksh, int trans, int conjb) {
    GemmArgs<R> a;
    a.in = in;
    a.out = out;
    a.U = U;
    a.M = M;
    a.N = N;
    a.K = K;
    a.row_mask = row_mask;
    a.row_fix = row_fix;
    a.ksh = ksh;
    a.trans = trans;
    a.conjb = conjb;
    const uint64_t gm = (M + GBM - 1) / GBM;
    const unsigned gn = (unsigned)((N + GBN - 1) / GBN);
    if (gm > 0x7fffffffull) return fail(SV_EUNSUPPORTED, "GEMM with too many rows");
    const uint64_t wtiles = ((M + 15) / 16) * (uint64_t)((N + 15) / 16);
    const uint64_t wblocks = (wtiles + 3) / 4;
    // the tile shape: 64 x 64 per workgroup (0), 16 x 16 per wavefront (1), or
    // k in parts: 16 x 16 in four (2), 32 x 32 in two (3).  Tuned per shape by
    // timing them on this call's operands (the product is out of place, so it
    // can be run again), cached; without tuning, parts wherever the 64 x 64
    // tiles would not fill the chip, the smaller ones up to two per compute unit.
    const std::string key = std::string("cgemm/") + (sizeof(R) == 4 ? "c64/" : "c128/") + std::to_string(M) + "/" +
                            std::to_string(N) + "/" + std::to_string(K) + "/" + std::to_string(trans) +
                            (ksh ? "/s" + std::to_string(ksh) : std::string());
    auto launch = [&](int shape) -> sv_status {
        TraceScope _ts(st, "cgemm", ((double)M * (N + K) + (double)N * K) * sizeof(cvec<R>), 8.0 * (double)M * N * K);
        if (shape == 1) {
            if (wblocks > 0x7fffffffull) return fail(SV_EUNSUPPORTED, "GEMM with too many tiles");
            hipLaunchKernelGGL(k_cgemm_w<R>, dim3((unsigned)wblocks), dim3(256), 0, st, a);
        } else if (shape == 2) {
            hipLaunchKernelGGL((k_cgemm_k<R, 1, 1, 4>), dim3((unsigned)((M + 15) / 16), (unsigned)((N + 15) / 16)), dim3(256),
                               0, st, a);
        } else if (shape == 3) {
            hipLaunchKernelGGL((k_cgemm_k<R, 2, 2, 2>), dim3((unsigned)((M + 31) / 32), (unsigned)((N + 31) / 32)), dim3(512),
                               0, st, a);
        } else {
            hipLaunchKernelGGL(k_cgemm<R>, dim3((unsigned)gm, gn), dim3(256), 0, st, a);
        }
        SV_HIP(hipGetLastError());
        return SV_OK;
    };
    std::vector<int> cached;
    // (grids of at most 2^22 workgroups in x: threads per launch stay below 2^32)
    const bool parts_ok = (M + 15) / 16 <= (1ull << 22) && N <= (1 << 19);
    int shape = gm * gn < 256 && parts_ok ? (wtiles <= 512 ? 2 : 3) : 0;
    if (tune_lookup(key, cached) && cached.size() == 1 && (cached[0] == 0 || cached[0] == 1 ||
                                                           (parts_ok && (cached[0] == 2 || cached[0] == 3)))) {
        shape = cached[0];
    } else if (autotune_enabled() && wblocks <= 0x7fffffffull) {
        // The parts only up to four 64 x 64 tiles per compute unit: beyond, the
        // large shape is the faster one (shapes 0 and 3, complex64 and complex128:
        // 128 tiles 65 34 99 51 us, 512: 181 185 308 322, 1024: 320 358 721 636,
        // 2048: 625 706 1164 1279).  One timing each as a first pass; products of a few microseconds
        // vary by more than the shapes differ and a wrong pick is up to twice as
        // slow (11 and 20 us), so those within half of the best are timed twice
        // more, which stays below a millisecond.
        const int ncand = gm * gn <= 1024 && parts_ok ? 4 : 2;
        float t[4] = {1e30f, 1e30f, 1e30f, 1e30f}, best = 1e30f;
        auto time = [&](int c, int reps) -> sv_status {
            float ms = 0.f;
            SV_TRY(time_stream(st, reps, &ms, [&]() { return launch(c); }));
            t[c] = std::min(t[c], ms);
            return SV_OK;
        };
        for (int c = 0; c < ncand; ++c) SV_TRY(time(c, 2));
        const float first = *std::min_element(t, t + 4);
        for (int round = 0; round < 2 && first < 0.05f; ++round)
            for (int c = 0; c < ncand; ++c)
                if (t[c] < 1.5f * first) SV_TRY(time(c, 4));
        for (int c = 0; c < ncand; ++c)
            if (t[c] < best) {
                best = t[c];
                shape = c;
            }
        tune_store(key, {shape});
    }
    return launch(shape);
}

template <typename R>
sv_status cgemm(hipStream_t st, const cvec<R> *in, cvec<R> *out, const cvec<R> *U, uint64_t M, int N, int K,
                uint64_t row_mask, uint64_t row_fix, int trans, int conjb) {
    return cgemm_ks<R>(st, in, out, U, M, N, K, row_mask, row_fix, 0, trans, conjb);
}
template sv_status cgemm<float>(hipStream_t, const float2 *, float2 *, const float2 *, uint64_t, int, int, uint64_t,
                                uint64_t, int, int);
template sv_status cgemm<double>(hipStream_t, const double2 *, double2 *, const double2 *, uint64_t, int, int,
                                 uint64_t, uint64_t, int, int);

// the register [lo, lo + m), controls cmask fixed to cval
template <typename R>
static sv_status ctrl_mask_unitary_at(sv_state s, const cvec<R> *U, int lo, int m, uint64_t cmask, uint64_t cval,
                                      int adjoint) {
    const uint64_t all = (s->n >= 64) ? ~0ull : ((1ull << s->n) - 1ull);
    // rows: every value of the bits outside the register and the controls,
    // with the controls fixed to cval
    const uint64_t row_mask = all & ~(((1ull << m) - 1ull) << lo) & ~cmask;
    const uint64_t row_fix = cval & cmask;
    const uint64_t M = dim_of(popcount64(row_mask));
    const int N = 1 << m;
    SV_TRY(ensure_scratch(s, (size_t)M * N * sizeof(cvec<R>)));
    cvec<R> *out = (cvec<R> *)s->scratch;
    SV_TRY(cgemm_ks<R>(s->stream, (const cvec<R> *)s->data, out, U, M, N, N, row_mask, row_fix, lo, adjoint, adjoint));
    const uint64_t total = M * (uint64_t)N;
    uint64_t g = (total + 1023) / 1024;
    if (g > (1u << 20)) g = 1u << 20;
    {
        TraceScope _ts(s->stream, "scatter_rows", 2.0 * (double)total * sizeof(cvec<R>), 0.0);
        const uint64_t gl = total / 1024;
        // whole rows while a launch is short; the grid-stride copy of k_scatter_rows
        // streams better when it is long.  Copies of 2^18 .. 2^22 elements, rows of
        // 256 (whole rows and, behind, elements): complex64 6.5 7.0, 7.5 8.2, 10.9
        // 10.9, 13.9 12.7, 23.5 19.7 us, complex128 7.2 8.3, 9.5 9.9, 10.6 10.1,
        // 15.1 14.8, 24.4 24.1; rows of 1024: 6.3 7.7, 6.7 6.7, 10.4 8.2, 12.5 11.1,
        // 21.1 17.8 and 6.6 9.4, 7.1 9.5, 9.8 9.0, 14.1 14.0, 24.5 23.4.
        if (lo == 0 && m >= 8 && gl >= 1 && gl <= 512)
            hipLaunchKernelGGL(k_scatter_long<R>, dim3((unsigned)gl), dim3(256), 0, s->stream, (cvec<R> *)s->data,
                               (const cvec<R> *)out, m, row_mask, row_fix);
        else
            hipLaunchKernelGGL(k_scatter_rows<R>, dim3((unsigned)g), dim3(256), 0, s->stream, (cvec<R> *)s->data,
                               (const cvec<R> *)out, M, m, row_mask, row_fix, lo);
    }
    SV_HIP(hipGetLastError());
    return SV_OK;
}

template <typename R>
sv_status ctrl_mask_unitary_impl(sv_state s, const cvec<R> *U, int m, uint64_t cmask, uint64_t cval, int adjoint) {
    return ctrl_mask_unitary_at<R>(s, U, 0, m, cmask, cval, adjoint);
}
template sv_status ctrl_mask_unitary_impl<float>(sv_state, const float2 *, int, uint64_t, uint64_t, int);
template sv_status ctrl_mask_unitary_impl<double>(sv_state, const double2 *, int, uint64_t, uint64_t, int);

template <typename R>
sv_status ctrl_unitary_impl(sv_state s, const cvec<R> *U, int m, int ctrl, int ctrl_val, int adjoint) {
    const uint64_t cm = ctrl >= 0 ? 1ull << ctrl : 0ull;
    return ctrl_mask_unitary_impl<R>(s, U, m, cm, ctrl_val ? cm : 0ull, adjoint);
}
template sv_status ctrl_unitary_impl<float>(sv_state, const float2 *, int, int, int, int);
template sv_status ctrl_unitary_impl<double>(sv_state, const double2 *, int, int, int, int);

}  // namespace sv

using namespace sv;

extern "C" sv_status sv_apply_ctrl_unitary(sv_state s, const void *U, int sys_lo, int m, int ctrl, int ctrl_val,
                                           int adjoint) {
    clear_error();
    SV_TRY(check_state(s));
    if (!U) return fail(SV_EINVAL, "U is NULL");
    if (m < 1 || sys_lo < 0 || sys_lo + m > s->n) return fail(SV_EINVAL, "register [%d,%d) outside the state", sys_lo, sys_lo + m);
    if (ctrl >= s->n || (ctrl >= sys_lo && ctrl < sys_lo + m)) return fail(SV_EINVAL, "control %d invalid", ctrl);
    if (m > 16) return fail(SV_EUNSUPPORTED, "dense register of %d qubits", m);
    const uint64_t cm = ctrl >= 0 ? 1ull << ctrl : 0ull, cv = ctrl_val ? cm : 0ull;
    if (s->dt == SV_C64)
        return ctrl_mask_unitary_at<float>(s, (const float2 *)U, sys_lo, m, cm, cv, adjoint ? 1 : 0);
    return ctrl_mask_unitary_at<double>(s, (const double2 *)U, sys_lo, m, cm, cv, adjoint ? 1 : 0);
}
