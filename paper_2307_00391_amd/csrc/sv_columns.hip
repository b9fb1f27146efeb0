// Batched eigen-frame HHL, a column per lane.
//
// In the eigen frame a solve is independent columns: for eigenvalue j the
// clock amplitudes after phase estimation are, with w_b the phase of clock bit
// b and t_b(x) = exp(2 pi i x / 2^(b+1)),
//   P(y) = 2^-n_c prod_b (1 + (-1)^(y_b) w_b conj(t_b(y mod 2^b)))
// (each stage of the inverse QFT maps a product state to a product state), the
// rotation multiplies them by s_y = 1 / y, and the uncompute projected on clock
// 0 is the inner product with conj(P):
//   z_j = beta_j sum_y s_y |P|^2, P(a = 1) = sum_j |beta_j|^2 sum_y s_y^2 |P|^2.
// A batch shows no state, so every amplitude is formed, rotated and summed in
// registers.
//
// k_batch_cols: 64 columns of one clock width (of any solves) per workgroup,
// one per lane; its four waves, and 2^sp workgroups, share the clock values.
// All lanes of a wave are at the same y, so the twiddles and rotations are
// scalars (s_load from small tables per clock width, FMAs take them as
// operands) and nothing else is read: the kernel is bound by vector issue.
// A line is the 2^RB values of the top RB bits over one value lo of the L bits
// below: the root prod_(b < L) (low bits once per o, the next three per line),
// then the top bits as a product tree, a node splitting into a + a q and
// 2 a - (a + a q) (six operations), with the 32nd roots of the line bits as
// constants.  All but the leaves and their sums in FP64 for both types, since
// the errors enter |P|^2 twice, alike.  (With two of a line's five levels in FP64:
// 115 instead of 134 us for the sweep below, and up to three times the errors;
// all of it in FP64: 160-178 us.)
// A sweep of 1024 complex64 solves (n_s 4..10, n_c 8..12): 134 us, about 18
// vector instructions per amplitude; the column tiles of k_pipe_a and k_pipe_b
// took 850 us at 37 operations, with tables, partial column sums and twiddles
// through memory.
#include <math.h>

#include <algorithm>
#include <map>
#include <vector>

#include "sv_device.h"
#include "sv_hhl_internal.h"
#include "sv_internal.h"

namespace sv {

// read-only tables behind scalar loads
template <typename T> using cptr = const __attribute__((address_space(4))) T *;

constexpr int COL_RB = 5;      // clock bits of a line (fewer for n_c < 5)
constexpr int COL_MID = 3;     // bits of the root formed per line

struct ColClass {
    const double *W;           // exp(2 pi i k / 2^L), k < 2^(L-1)
    const double *E;           // [2^L][8] exp(2 pi i lo / 2^(L + kb + 1)), kb < RB
    const void *S;             // [2^L][2^RB] (s_y, s_y^2), y = lo + (k << L)
    const uint2 *map;          // (solve, column) of every lane, solve ~0 for none
    int n_c, sp;
    uint32_t block0, nblocks;
};

// cos(2 pi k / 32) and sin(2 pi k / 32)
__device__ constexpr double cos32(int k) {
    constexpr double c[9] = {1.0,
                             0.98078528040323044913,
                             0.92387953251128675613,
                             0.83146961230254523708,
                             0.70710678118654752440,
                             0.55557023301960222474,
                             0.38268343236508977173,
                             0.19509032201612826785,
                             0.0};
    k &= 31;
    return k <= 8 ? c[k] : k <= 16 ? -c[16 - k] : k <= 24 ? -c[k - 16] : c[32 - k];
}
__device__ constexpr double sin32(int k) { return cos32(k - 8); }

__device__ __forceinline__ float cfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double cfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// (a + a q, a - a q)
template <typename R>
__device__ __forceinline__ void split(cvec<R> a, cvec<R> q, cvec<R> &p, cvec<R> &m) {
    const R px = cfma(a.x, q.x, cfma(-a.y, q.y, a.x)), py = cfma(a.x, q.y, cfma(a.y, q.x, a.y));
    p = cmake<R>(px, py);
    m = cmake<R>(cfma((R)2, a.x, -px), cfma((R)2, a.y, -py));
}

// every node m < 2^kb of a level of the line's tree with its q: Q turned by
// -m / 2^(kb+1), the upper half of the nodes another quarter
template <typename R, typename F>
__device__ __forceinline__ void tree_level(int kb, cvec<R> Q, F node) {
    if (kb == 0) {
        node(0, Q);
        return;
    }
    const int h = 1 << (kb - 1);
#pragma unroll
    for (int m = 0; m < h; ++m) {
        const R c = (R)cos32(m << (4 - kb)), sn = (R)sin32(m << (4 - kb));
        const cvec<R> q = m == 0 ? Q : cmake<R>(cfma(Q.x, c, Q.y * sn), cfma(Q.y, c, -(Q.x * sn)));
        node(m, q);
        node(m + h, cmake<R>(q.y, -q.x));
    }
}

// r times the factor of clock bit b at the values x = lo mod 2^b, bit set or not
__device__ __forceinline__ double2 bit_factor(double2 r, double2 w, cptr<double> W, uint32_t k, bool set) {
    const double tx = W[2 * k], ty = set ? -W[2 * k + 1] : W[2 * k + 1];
    const double sx = set ? -tx : tx;
    // +-q = w conj(t) (+-1)
    const double qx = cfma(w.x, sx, w.y * ty), qy = cfma(w.y, sx, -(w.x * ty));
    return make_double2(cfma(r.x, qx, cfma(-r.y, qy, r.x)), cfma(r.x, qy, cfma(r.y, qx, r.y)));
}

template <typename R, int RB>
__global__ __launch_bounds__(256) void k_batch_cols(const ColClass *__restrict__ cls, int ncls,
                                                    const ColSolve *__restrict__ solves) {
    __shared__ double2 w[20][64];
    __shared__ double red[3][3][64];
    int ci = 0;
    while (ci + 1 < ncls && blockIdx.x >= cls[ci + 1].block0) ++ci;
    const ColClass T = cls[ci];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t blk = blockIdx.x - T.block0, splt = blk & ((1u << T.sp) - 1);
    const uint2 *mp = T.map + (size_t)(blk >> T.sp) * 64;
    uint2 cm = mp[lane];
    const bool live = cm.x != ~0u;
    if (!live) cm = mp[0];
    const ColSolve S = solves[cm.x];
    const int n_c = T.n_c, L = n_c - RB;
    // the column's phases; the waves share the bits
    for (int b = wv; b < n_c; b += 4) w[b][lane] = turn_phase<double>(turn_fraction(S.lam[cm.y], S.T0, n_c - 1 - b));
    __syncthreads();
    double2 wt[RB];
#pragma unroll
    for (int kb = 0; kb < RB; ++kb) wt[kb] = w[L + kb][lane];
    const cptr<double> W = (cptr<double>)T.W, E = (cptr<double>)T.E;
    const cptr<R> Sy = (cptr<R>)T.S;
    // workers: the waves of the 2^sp workgroups of these columns; they part the
    // values of the lowest bits o first, then the line's root bits
    const int mid = L < COL_MID ? L : COL_MID, La = L - mid;
    const int lu = T.sp + 2, so = lu < La ? lu : La;
    const uint32_t u = splt * 4 + wv;
    double z = 0.0, pa = 0.0, nt = 0.0;
    for (uint32_t o = u & ((1u << so) - 1); o < (1u << La); o += 1u << so) {
        double2 t = make_double2(ldexp(1.0, -n_c), 0.0);
        for (int b = 0; b < La; ++b)
            t = bit_factor(t, w[b][lane], W, (o & ((1u << b) - 1)) << (L - 1 - b), o >> b & 1);
        for (uint32_t node = u >> so; node < (1u << mid); node += 1u << (lu - so)) {
            const uint32_t lo = o + (node << La);
            double2 r = t;
            for (int b = La; b < L; ++b)
                r = bit_factor(r, w[b][lane], W, (lo & ((1u << b) - 1)) << (L - 1 - b), lo >> b & 1);
            const cptr<double> El = E + 16 * lo;
            const cptr<R> Sl = Sy + ((size_t)lo << (RB + 1));
            // Q_b = w_b conj(exp(2 pi i lo / 2^(b+1)))
            auto Q = [&](int kb) {
                const double ex = El[2 * kb], ey = El[2 * kb + 1];
                return make_double2(cfma(wt[kb].x, ex, wt[kb].y * ey), cfma(wt[kb].y, ex, -(wt[kb].x * ey)));
            };
            double2 v[1 << (RB - 1)];
            v[0] = r;
#pragma unroll
            for (int kb = 0; kb < RB - 1; ++kb)
                tree_level<double>(kb, Q(kb), [&](int m, double2 q) { split<double>(v[m], q, v[m], v[m + (1 << kb)]); });
            // the leaves k = m and m + 2^(RB-1): the sums, in FP32 in four chains (one
            // chain of a line's 32 terms rounds the peak's share up to 31 times: rms
            // error of p_post over 1152 solves of 9 clock bits 2.75e-7, four chains
            // 1.35e-7, the column tiles before 2.19e-7; the launch takes as long)
            constexpr int NCH = sizeof(R) == 4 ? 4 : 1;
            R lz[4] = {0, 0, 0, 0}, lpa[4] = {0, 0, 0, 0}, lnt[4] = {0, 0, 0, 0};
            const double2 qd = Q(RB - 1);
            tree_level<R>(RB - 1, cmake<R>((R)qd.x, (R)qd.y), [&](int m, cvec<R> q) {
                constexpr int h = 1 << (RB - 1);
                cvec<R> p, n;
                split<R>(cmake<R>((R)v[m].x, (R)v[m].y), q, p, n);
                const R p2 = cfma(p.x, p.x, p.y * p.y), n2 = cfma(n.x, n.x, n.y * n.y);
                const int q4 = m & (NCH - 1);
                lnt[q4] += p2 + n2;
                lz[q4] = cfma(Sl[2 * m], p2, cfma(Sl[2 * (m + h)], n2, lz[q4]));
                lpa[q4] = cfma(Sl[2 * m + 1], p2, cfma(Sl[2 * (m + h) + 1], n2, lpa[q4]));
            });
            auto total = [](const R (&x)[4]) { return (double)(NCH == 1 ? x[0] : (x[0] + x[1]) + (x[2] + x[3])); };
            z += total(lz);
            pa += total(lpa);
            nt += total(lnt);
        }
    }
    if (wv) {
        red[wv - 1][0][lane] = z;
        red[wv - 1][1][lane] = pa;
        red[wv - 1][2][lane] = nt;
    }
    __syncthreads();
    if (wv || !live) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        z += red[k][0][lane];
        pa += red[k][1][lane];
        nt += red[k][2][lane];
    }
    const double2 be = S.beta[cm.y];
    const double b2 = be.x * be.x + be.y * be.y;
    const uint64_t i = (uint64_t)splt * S.N + cm.y;
    S.zpart[i] = z;
    S.part[2 * i] = b2 * pa;
    S.part[2 * i + 1] = b2 * nt;
}

// the tables of one clock width
template <typename R>
__global__ void k_col_tables(double2 *__restrict__ W, double2 *__restrict__ E, cvec<R> *__restrict__ S, int n_c,
                             int rb) {
    const int L = n_c - rb;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x, i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (L > 0)
        for (uint64_t k = i0; k < (1ull << (L - 1)); k += step) W[k] = turn_phase<double>(k << (64 - L));
    for (uint64_t i = i0; i < (8ull << L); i += step) {
        const int kb = (int)(i & 7);
        E[i] = kb < rb ? turn_phase<double>((i >> 3) << (63 - (L + kb))) : make_double2(0.0, 0.0);
    }
    for (uint64_t i = i0; i < (1ull << n_c); i += step) {
        const uint64_t y = (i >> rb) + ((i & ((1ull << rb) - 1)) << L);
        const double sd = y ? 1.0 / (double)y : 0.0;
        S[i] = cmake<R>((R)sd, (R)(sd * sd));
    }
}

// log2 of the workgroups sharing 64 columns, per clock width: none more than
// 2^10 amplitudes per wave and lane (a longer wave delays the end of a launch:
// 2^10 is about 25 us of a SIMD to itself), and more while the batch has fewer
// than 1024 workgroups and a wave more than two lines
std::map<int, int> cols_splits(const std::map<int, uint64_t> &ncols) {
    std::map<int, int> sp;
    for (const auto &kv : ncols) sp[kv.first] = std::max(0, kv.first - 12);
    for (;;) {
        uint64_t blocks = 0;
        bool grown = false;
        for (const auto &kv : ncols) blocks += ((kv.second + 63) / 64) << sp[kv.first];
        if (blocks >= 1024) break;
        for (auto &kv : sp)
            if (kv.first - COL_RB - 2 - kv.second > 1) {
                ++kv.second;
                grown = true;
            }
        if (!grown) break;
    }
    return sp;
}

static int col_rb(int n_c) { return std::min(n_c, COL_RB); }

template <typename R>
sv_status cols_build(sv_state ctx, ColPlan &p, DevBuf &buf, const std::vector<int> &ns, const std::vector<int> &nc,
                     const std::map<int, int> &sp, const std::vector<ColSolve> &solves) {
    // the columns per clock width, solves in order of size so that a workgroup
    // of narrow solves holds whole ones
    std::map<int, std::vector<int>> by;
    for (size_t k = 0; k < solves.size(); ++k) by[nc[k]].push_back((int)k);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = (off + 255) & ~(size_t)255;
        const size_t o = off;
        off += bytes;
        return o;
    };
    const size_t o_sol = take(solves.size() * sizeof(ColSolve)), o_cls = take(by.size() * sizeof(ColClass));
    struct Lay {
        size_t W, E, S, map;
        uint64_t groups;
    };
    std::map<int, Lay> lay;
    for (auto &kv : by) {
        uint64_t cols = 0;
        for (int k : kv.second) cols += dim_of(ns[k]);
        Lay l;
        l.groups = (cols + 63) / 64;
        const uint64_t lines = 1ull << (kv.first - col_rb(kv.first));
        l.W = take(lines * sizeof(double2));
        l.E = take(8 * lines * sizeof(double2));
        l.S = take((1ull << kv.first) * sizeof(cvec<R>));
        l.map = take(l.groups * 64 * sizeof(uint2));
        lay[kv.first] = l;
    }
    SV_TRY(buf.alloc(off));
    char *d = (char *)buf.p;
    SV_TRY(upload(ctx, d + o_sol, solves.data(), solves.size() * sizeof(ColSolve)));
    // widest first: their workgroups run longest
    std::vector<ColClass> cls;
    for (int rb = COL_RB; rb >= 2; --rb) {
        ColLaunch L{(int)cls.size(), 0, 0, rb};
        uint64_t blocks = 0;
        for (auto it = by.rbegin(); it != by.rend(); ++it) {
            const int n_c = it->first;
            if (col_rb(n_c) != rb) continue;
            const Lay &l = lay[n_c];
            std::vector<int> &mem = it->second;
            std::stable_sort(mem.begin(), mem.end(), [&](int x, int y) { return ns[x] > ns[y]; });
            std::vector<uint2> map;
            map.reserve(l.groups * 64);
            for (int k : mem)
                for (uint64_t j = 0; j < dim_of(ns[k]); ++j) map.push_back(make_uint2((unsigned)k, (unsigned)j));
            map.resize(l.groups * 64, make_uint2(~0u, 0u));
            SV_TRY(upload(ctx, d + l.map, map.data(), map.size() * sizeof(uint2)));
            const uint64_t nb = l.groups << sp.at(n_c);
            // (a grid holds less than 2^32 threads)
            if (blocks + nb >= 1ull << 24) return fail(SV_EUNSUPPORTED, "batch of too many columns");
            cls.push_back(ColClass{(const double *)(d + l.W), (const double *)(d + l.E), d + l.S, (const uint2 *)(d + l.map), n_c,
                                   sp.at(n_c), (uint32_t)blocks, (uint32_t)nb});
            blocks += nb;
            ++L.ncls;
            hipLaunchKernelGGL(k_col_tables<R>, dim3(64), dim3(256), 0, ctx->stream, (double2 *)(d + l.W),
                               (double2 *)(d + l.E), (cvec<R> *)(d + l.S), n_c, rb);
            SV_HIP(hipGetLastError());
        }
        L.blocks = (uint32_t)blocks;
        if (L.ncls) p.launches.push_back(L);
    }
    SV_TRY(upload(ctx, d + o_cls, cls.data(), cls.size() * sizeof(ColClass)));
    p.d_cls = d + o_cls;
    p.d_solves = (const ColSolve *)(d + o_sol);
    p.bytes = 0.0;
    p.flops = 0.0;
    for (auto &kv : by)
        for (int k : kv.second) {
            p.bytes += 24.0 * (double)dim_of(ns[k]) * (double)(1 << sp.at(kv.first));
            p.flops += 24.0 * (double)dim_of(ns[k] + kv.first);
        }
    return SV_OK;
}

template <typename R>
sv_status cols_launch(hipStream_t st, const ColPlan &p) {
    TraceScope ts(st, "batch_cols", p.bytes, p.flops);
    for (const ColLaunch &l : p.launches) {
        const ColClass *c = (const ColClass *)p.d_cls + l.cls0;
        const dim3 g(l.blocks), b(256);
        switch (l.rb) {
        case 2: hipLaunchKernelGGL((k_batch_cols<R, 2>), g, b, 0, st, c, l.ncls, p.d_solves); break;
        case 3: hipLaunchKernelGGL((k_batch_cols<R, 3>), g, b, 0, st, c, l.ncls, p.d_solves); break;
        case 4: hipLaunchKernelGGL((k_batch_cols<R, 4>), g, b, 0, st, c, l.ncls, p.d_solves); break;
        default: hipLaunchKernelGGL((k_batch_cols<R, 5>), g, b, 0, st, c, l.ncls, p.d_solves); break;
        }
        SV_HIP(hipGetLastError());
    }
    return SV_OK;
}

template sv_status cols_build<float>(sv_state, ColPlan &, DevBuf &, const std::vector<int> &, const std::vector<int> &,
                                     const std::map<int, int> &, const std::vector<ColSolve> &);
template sv_status cols_build<double>(sv_state, ColPlan &, DevBuf &, const std::vector<int> &,
                                      const std::vector<int> &, const std::map<int, int> &,
                                      const std::vector<ColSolve> &);
template sv_status cols_launch<float>(hipStream_t, const ColPlan &);
template sv_status cols_launch<double>(hipStream_t, const ColPlan &);

}  // namespace sv
