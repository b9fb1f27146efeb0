// QSP-1: binary-tree state preparation (appendix "Quantum State
// Preparation"; the Grover-Rudolph tree in Prakash's form).
//
// Tree over the register value r of [q_lo, q_lo + m): leaves carry |b_r|^2,
// inner nodes the sum of their children.  Level l decides qubit
// q_lo + m - 1 - l (most significant first); node p of level l is the value of
// the l qubits above it.  Each node with weight w > 0 is an Ry(t) with
// cos^2(t/2) = zero-child / w, controlled on those qubits taking the value p;
// a final diagonal restores arg(b_r).
//
//   mode 0: the circuit on the state: |0...0>, one Ry on the top qubit, then
//           per level one uniformly controlled Ry pass (every node of the
//           level is one control value), then the phase diagonal pass;
//   mode 1: the same circuit applied to |0...0> in one write pass: each
//           amplitude is the product of the rotation entries on its tree
//           path times its phase (a thread expands the subtree below one
//           node of level m - 5 in registers); zero outside the register.
#include <math.h>
#include <string.h>

#include "sv_device.h"
#include "sv_internal.h"

namespace sv {

// heap-ordered (cos, sin) of every node, node k = 2^l + p at 2k, 2k + 1.
// A thread owns the 2^C leaves below one node of level m - C: it walks the
// m - C levels above that node once, then expands its subtree in registers.
// The leaves of a block's QSP_NT subtrees (QSP_NT 2^C consecutive register
// values) go through LDS (one pad element per thread, so the row writes are
// conflict-free) and leave in register order, so that each store and each
// phase-table read of a wavefront covers consecutive addresses.
constexpr int QSP_NT = 128;

template <typename R, int C>
__global__ __launch_bounds__(QSP_NT) void k_qsp_tree(cvec<R> *__restrict__ psi, int q_lo, int m,
                                                     const R *__restrict__ cs, const cvec<R> *__restrict__ ph) {
    constexpr int L = 1 << C, LP = L + 1;
    __shared__ R leaves[QSP_NT * LP];
    const uint64_t nsub = 1ull << (m - C);          // subtrees
    const uint64_t R_ = 1ull << m;
    for (uint64_t t0 = (uint64_t)blockIdx.x * QSP_NT; t0 < nsub; t0 += (uint64_t)gridDim.x * QSP_NT) {
        const uint64_t t = t0 + threadIdx.x;
        if (t < nsub) {
            R a = 1;
            uint64_t node = 1;
            for (int l = 0; l < m - C; ++l) {
                const uint64_t bit = (t >> (m - C - 1 - l)) & 1ull;
                a *= cs[2 * node + bit];
                node = 2 * node + bit;
            }
            R v[L];
            v[0] = a;
#pragma unroll
            for (int l = 0; l < C; ++l) {
                // the 2^l values of this level, at nodes (node << l) + q, split into their children
#pragma unroll
                for (int q = (1 << l) - 1; q >= 0; --q) {
                    const uint64_t nd = (node << l) + (uint64_t)q;
                    const R x = v[q];
                    v[2 * q] = x * cs[2 * nd];
                    v[2 * q + 1] = x * cs[2 * nd + 1];
                }
            }
#pragma unroll
            for (int j = 0; j < L; ++j) leaves[threadIdx.x * LP + j] = v[j];
        }
        __syncthreads();
        // leaf e of the block is register value (t0 << C) + e
        const uint64_t rbase = t0 << C;
        for (int e = threadIdx.x; e < QSP_NT * L; e += QSP_NT) {
            const uint64_t r = rbase + (uint64_t)e;
            if (r >= R_) break;
            const R x = leaves[(e >> C) * LP + (e & (L - 1))];
            const cvec<R> p = ph[r];
            psi[r << q_lo] = cmake<R>(x * p.x, x * p.y);
        }
        __syncthreads();
    }
}

template <typename R>
__global__ __launch_bounds__(256) void k_zero(cvec<R> *__restrict__ psi, uint64_t dim) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim; i += stride) psi[i] = cmake<R>(0, 0);
}

// psi[i] *= ph[register value of i] (a diagonal gate on the register)
template <typename R>
__global__ __launch_bounds__(256) void k_reg_phase(cvec<R> *__restrict__ psi, uint64_t dim, int q_lo, int m,
                                                   const cvec<R> *__restrict__ ph) {
    const uint64_t rmask = (1ull << m) - 1ull;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim; i += stride)
        psi[i] = cmul<R>(psi[i], ph[(i >> q_lo) & rmask]);
}

static unsigned grid_of(uint64_t items) {
    uint64_t g = (items + 1023) / 1024;
    if (g < 1) g = 1;
    if (g > (1u << 20)) g = 1u << 20;
    return (unsigned)g;
}

// ---------------------------------------------------------------------------
// The tree's tables, built on the device: leaf weights |b_r|^2 and inner sums
// in FP64, pairwise in heap order; (cos, sin) of every node from the FP64
// weights, rounded once; the phase of every leaf.  On the host the same took
// all but 0.1 of the 40 ms of a 2^20-point preparation (square roots, atan2,
// cos and sin one at a time); here the call takes 0.80 ms, bound by the host's
// copy of b into pinned memory (16 MiB, 0.42 ms) and its transfer (0.30 ms).
// ---------------------------------------------------------------------------

// A block reduces 2^QSP_BL consecutive nodes by up to QSP_BL levels in LDS.
// (Blocks of 512 leaves: a 2^16-leaf chunk of the upload still fills 128
// compute units.)
constexpr int QSP_BL = 9, QSP_BT = 256;

// (cos, sin) of the node with children weights (wl, wr); node weight 0: no gate
template <typename R>
__device__ __forceinline__ double qsp_node(double wl, double wr, R *__restrict__ cs) {
    const double w = wl + wr;
    const bool on = w > 0.0;
    cs[0] = (R)(on ? sqrt(wl / w) : 1.0);
    cs[1] = (R)(on ? sqrt(wr / w) : 0.0);
    return w;
}

// levels `lev` - 1 ... lev - nl above the nodes w[0][0..2^nl) of level `lev` that
// start at index `first` of their level; returns the top weight (thread 0)
template <typename R>
__device__ __forceinline__ double qsp_reduce(double (&w)[2][1 << QSP_BL], int lev, int nl, uint64_t first,
                                             R *__restrict__ cs) {
    for (int s = 1; s <= nl; ++s) {
        const int cnt = 1 << (nl - s);
        const double *src = w[(s - 1) & 1];
        double *dst = w[s & 1];
        const uint64_t node0 = (1ull << (lev - s)) + (first >> s);
        for (int i = threadIdx.x; i < cnt; i += blockDim.x)
            dst[i] = qsp_node<R>(src[2 * i], src[2 * i + 1], cs + 2 * (node0 + (uint64_t)i));
        __syncthreads();
    }
    return w[nl & 1][0];
}

// leaves [r0, r0 + gridDim.x 2^nl): weights, phases, the lowest nl levels; the
// block's top weight goes to top[its index].  A non-finite entry sets *bad.
template <typename R>
__global__ __launch_bounds__(QSP_BT) void k_qsp_leaves(const double2 *__restrict__ b, uint64_t r0, int m, int nl,
                                                       R *__restrict__ cs, cvec<R> *__restrict__ ph,
                                                       double *__restrict__ top, int *__restrict__ bad) {
    __shared__ double w[2][1 << QSP_BL];
    const uint64_t o = (uint64_t)blockIdx.x << nl;
    for (int i = threadIdx.x; i < (1 << nl); i += blockDim.x) {
        const double2 z = b[o + i];
        if (!isfinite(z.x) || !isfinite(z.y)) *bad = 1;
        const double wt = z.x * z.x + z.y * z.y;
        w[0][i] = wt;
        const double h = hypot(z.x, z.y);
        ph[r0 + o + i] = wt > 0.0 ? cmake<R>((R)(z.x / h), (R)(z.y / h)) : cmake<R>((R)1, (R)0);
    }
    __syncthreads();
    const double t = qsp_reduce<R>(w, m, nl, r0 + o, cs);
    if (threadIdx.x == 0) top[((r0 + o) >> nl)] = t;
}

// nl levels above level `lev`, whose weights are wt[0..2^lev)
template <typename R>
__global__ __launch_bounds__(QSP_BT) void k_qsp_levels(const double *__restrict__ wt, int lev, int nl, R *__restrict__ cs,
                                                       double *__restrict__ top) {
    __shared__ double w[2][1 << QSP_BL];
    const uint64_t o = (uint64_t)blockIdx.x << nl;
    for (int i = threadIdx.x; i < (1 << nl); i += blockDim.x) w[0][i] = wt[o + i];
    __syncthreads();
    const double t = qsp_reduce<R>(w, lev, nl, o, cs);
    if (threadIdx.x == 0) top[blockIdx.x] = t;
}

// Builds the tables in the state's scratch arena: dcs (2 R entries, node k at
// 2k, 2k + 1) and dph (R phases).  b crosses in chunks of 2^QSP_CHUNK entries
// through two pinned and two device slots, so that the host's copy of one
// chunk, the transfer of the last and the reduction of the one before
// overlap.  Reports the root weight (0: b = 0) and non-finite entries before
// anything of the state is written.  Synchronises the stream.
constexpr int QSP_CHUNK = 16;

template <typename R>
static sv_status build_tables(sv_state s, const double *b, int m, R **dcs, cvec<R> **dph) {
    const uint64_t N = 1ull << m;
    const int ck = m < QSP_CHUNK ? m : QSP_CHUNK, bl = m < QSP_BL ? m : QSP_BL;
    const size_t cbytes = sizeof(double2) << ck;
    auto pad = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t bcs = pad(2 * N * sizeof(R)), bph = pad(N * sizeof(cvec<R>)), bst = pad(cbytes);
    const size_t btop = pad((N >> bl) * sizeof(double));
    SV_TRY(ensure_scratch(s, bcs + bph + 2 * bst + 2 * btop + 256));
    char *p = (char *)s->scratch;
    *dcs = (R *)p;
    *dph = (cvec<R> *)(p + bcs);
    double2 *stage[2] = {(double2 *)(p + bcs + bph), (double2 *)(p + bcs + bph + bst)};
    double *top[2] = {(double *)(p + bcs + bph + 2 * bst), (double *)(p + bcs + bph + 2 * bst + btop)};
    // root weight and flag, copied back together
    double *res = (double *)(p + bcs + bph + 2 * bst + 2 * btop);
    SV_TRY(ensure_pinned(s, 2 * bst + 256));
    SV_HIP(hipStreamSynchronize(s->stream));   // the pinned slots may still be in use
    hipLaunchKernelGGL(k_zero<double>, dim3(1), dim3(64), 0, s->stream, (double2 *)res, (uint64_t)1);
    hipEvent_t ev[2] = {nullptr, nullptr};
    sv_status st = SV_OK;
    auto run = [&]() -> sv_status {
        const uint64_t nch = N >> ck;
        if (nch > 2)
            for (int i = 0; i < 2; ++i) SV_HIP(hipEventCreateWithFlags(&ev[i], hipEventDisableTiming));
        for (uint64_t c = 0; c < nch; ++c) {
            const int q = (int)(c & 1);
            char *pin = (char *)s->pinned + (size_t)q * bst;
            if (c >= 2) SV_HIP(hipEventSynchronize(ev[q]));
            memcpy(pin, b + 2 * (c << ck), cbytes);
            SV_HIP(hipMemcpyAsync(stage[q], pin, cbytes, hipMemcpyHostToDevice, s->stream));
            if (ev[q]) SV_HIP(hipEventRecord(ev[q], s->stream));
            hipLaunchKernelGGL(k_qsp_leaves<R>, dim3(1u << (ck - bl)), dim3(QSP_BT), 0, s->stream,
                               (const double2 *)stage[q], c << ck, m, bl, *dcs, *dph, m == bl ? res : top[0],
                               (int *)(res + 1));
        }
        int cur = 0;
        for (int lev = m - bl; lev > 0;) {
            const int nl = lev < QSP_BL ? lev : QSP_BL;
            hipLaunchKernelGGL(k_qsp_levels<R>, dim3(1u << (lev - nl)), dim3(QSP_BT), 0, s->stream,
                               (const double *)top[cur], lev, nl, *dcs, lev == nl ? res : top[cur ^ 1]);
            lev -= nl;
            cur ^= 1;
        }
        SV_HIP(hipGetLastError());
        double out[2];
        SV_TRY(download(s, out, res, sizeof out));
        int bad;
        memcpy(&bad, &out[1], sizeof bad);
        if (bad) return fail(SV_EINVAL, "b has a non-finite entry");
        if (!(out[0] > 0.0)) return fail(SV_EZERONORM, "|b| = 0");
        return SV_OK;
    };
    st = run();
    if (st != SV_OK) (void)hipStreamSynchronize(s->stream);   // no transfer may outlive the call
    for (int i = 0; i < 2; ++i)
        if (ev[i]) (void)hipEventDestroy(ev[i]);
    return st;
}

template <typename R>
static sv_status qsp_impl(sv_state s, const double *b, int q_lo, int m, int mode) {
    const uint64_t N = 1ull << m, dim = dim_of(s->n);
    R *dcs = nullptr;
    cvec<R> *dph = nullptr;
    SV_TRY(build_tables<R>(s, b, m, &dcs, &dph));
    cvec<R> *psi = (cvec<R> *)s->data;
    if (mode == 1) {
        if (N != dim) {   // qubits outside the register: |0>
            TraceScope tz(s->stream, "qsp_zero", (double)dim * sizeof(cvec<R>), 0.0);
            hipLaunchKernelGGL(k_zero<R>, dim3(grid_of(dim)), dim3(256), 0, s->stream, psi, dim);
        }
        // algorithmic bytes: the register written once, its (cos, sin) tree and phase table read once
        TraceScope ts(s->stream, "qsp_tree", (double)N * 3.0 * sizeof(cvec<R>), 0.0);
        const uint64_t nsub = N >> (m < 5 ? m : 5);
        const uint64_t nblk = (nsub + QSP_NT - 1) / QSP_NT;
        const dim3 g((unsigned)(nblk < (1u << 20) ? nblk : (1u << 20)));
        auto launch = [&](auto kern) {
            hipLaunchKernelGGL(kern, g, dim3(QSP_NT), 0, s->stream, psi, q_lo, m, (const R *)dcs, (const cvec<R> *)dph);
        };
        switch (m < 5 ? m : 5) {
        case 1: launch(k_qsp_tree<R, 1>); break;
        case 2: launch(k_qsp_tree<R, 2>); break;
        case 3: launch(k_qsp_tree<R, 3>); break;
        case 4: launch(k_qsp_tree<R, 4>); break;
        default: launch(k_qsp_tree<R, 5>); break;
        }
    } else {
        // mode 0: the circuit, level by level.  Level l is one uniformly
        // controlled Ry on the qubits above its target; its table is the
        // level's stretch of dcs.
        SV_TRY(sv_init_basis(s, 0));
        const int top = q_lo + m - 1;
        for (int l = 0; l < m; ++l)
            SV_TRY(uniform_ry_table(s, top - l, top - l + 1, l, dcs + (2ull << l), 1ull << (top - l), 0));
        TraceScope ts(s->stream, "reg_phase", 2.0 * (double)dim * sizeof(cvec<R>), 0.0);
        hipLaunchKernelGGL(k_reg_phase<R>, dim3(grid_of(dim)), dim3(256), 0, s->stream, psi, dim, q_lo, m,
                           (const cvec<R> *)dph);
    }
    SV_HIP(hipGetLastError());
    SV_HIP(hipStreamSynchronize(s->stream));   // the tables live in the scratch arena
    return SV_OK;
}

}  // namespace sv

using namespace sv;

extern "C" {

sv_status sv_qsp_prepare(sv_state s, const double *b, int q_lo, int m, int mode) {
    clear_error();
    SV_TRY(check_state(s));
    if (!b) return fail(SV_EINVAL, "b is NULL");
    if (m < 1 || m > 26 || q_lo < 0 || q_lo + m > s->n)
        return fail(SV_EINVAL, "register [%d, %d) outside the state (or wider than 26 qubits)", q_lo, q_lo + m);
    if (mode != 0 && mode != 1) return fail(SV_EINVAL, "mode must be 0 or 1");
    return s->dt == SV_C64 ? qsp_impl<float>(s, b, q_lo, m, mode) : qsp_impl<double>(s, b, q_lo, m, mode);
}

}  // extern "C"
