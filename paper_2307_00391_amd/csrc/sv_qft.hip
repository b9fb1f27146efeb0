// Quantum Fourier transform of a register in as few passes over the state as
// its tiles allow.
//
// A register of m qubits is cut into groups of consecutive qubits, one pass
// per group.  A pass holds tiles of 2^k amplitudes: the lowest few index bits
// (so that HBM accesses are runs of 128 bytes or more) and the group's bits.
// Inside a tile the group runs in radix steps of up to 4 qubits: a thread
// holds the 16 amplitudes that differ in the step's bits, transforms them in
// registers (constant 16th roots of unity) and multiplies by the twiddles of
// the register bits below; the tile passes between steps through LDS.  The
// first step reads HBM straight into registers and the last one writes it
// from there wherever its register bits lie above the contiguous run.
//
// What bounds it: HBM, at the rate that tiles of 64 KiB with their load,
// transform and store phases reach.  A plain pass over 1 GiB of complex64
// takes 0.41-0.45 ms (4.8-5.2 TB/s), over 512 MiB of complex128 0.24-0.26 ms
// (4.2-4.5 TB/s; twice the vector work per amplitude), the mirrored pass 0.58.
// One butterfly stage per LDS round trip with a sincos per butterfly, and the
// reversal as a pass of single amplitudes, took 1.2 and 0.70 ms instead:
// 4.24 -> 1.86 ms for 24 qubits of 27 (complex64, exact order), and 2.93 ->
// 0.76 ms for the spectral gradient of 17 qubits of 25 (complex128).
// Tiles of 128 KiB (one workgroup per compute unit) save a pass on some
// registers and lose more to the phases: 2.09 against 1.99 ms.
//
// Two orders are built: the descending cascade (DIF: natural order in,
// bit-reversed out) and its mirror (DIT: bit-reversed in, natural out), each
// with either sign of the exponent.  A transform in exact index order runs
// the descending cascade; its last pass holds the lowest g and the highest g
// register bits of two tiles whose middle bits mirror each other, and writes
// each tile's bit-reversed image over the other: the reversal costs no pass.
// The spectral gradient needs no reversal at all: its rotation sits between
// a descending transform and an ascending one, and reads the wavenumber from
// the reversed index.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "sv_fused.h"

namespace sv {

constexpr int QFT_MAX_STEPS = 4;
constexpr int QFT_MAX_THREADS = 512;

struct QftStep {
    int R;             // qubits transformed: register bits 0..R-1 of the step's 4 (the rest are passengers)
    int j;             // register-relative position of the lowest of them
    int dep;           // a passenger is one of the register bits below j
    int ipos[4];       // tile positions of the 4 register bits, ascending
    uint32_t lb[4];    // LDS byte offset (swizzled) of register bit i
    uint64_t gb[4];    // index offset of register bit i
};

struct QftTile {
    uint64_t nl_mask, fix_val;      // tile number deposit, fixed bits
    uint64_t tile0;                 // first tile of this launch
    int k;                          // tile bits: [0, c) | r1 bits at p1 | r2 bits at p2
    int c, p1, r1, p2, r2;
    int lo, m;                      // the register
    int nsteps;
    int direct_in, direct_out;      // first / last step moves HBM <-> registers itself
    int rev_tp, rev_w;              // bit reversal of the tile field [rev_tp, rev_tp + rev_w) on the way out
    int mid_lo, mid_w;              // the mirrored middle bits, two or more (two tiles per workgroup); mid_w = 0: none
    QftStep st[QFT_MAX_STEPS];
};

__device__ __forceinline__ uint64_t tile_index(const QftTile &A, uint32_t t) {
    uint64_t g = t & ((1u << A.c) - 1u);
    const uint32_t h = t >> A.c;
    g |= (uint64_t)(h & ((1u << A.r1) - 1u)) << A.p1;
    if (A.r2) g |= (uint64_t)(h >> A.r1) << A.p2;
    return g;
}

// exp(2 pi i t / 2^64): the nearest quarter turn exactly, the rest (at most an
// eighth of a turn) by the Taylor series of sine and cosine, cut where the
// next term is below a quarter of the type's rounding.  The reduction is exact
// in the integer, which a library sincospi has to redo in floating point:
// 18 against some 35 instructions in FP32, 35 against some 80 in FP64, and a
// step needs up to 8 of them per 16 amplitudes.
template <typename R> __device__ __forceinline__ cvec<R> turn_root(uint64_t t);
template <> __device__ __forceinline__ float2 turn_root<float>(uint64_t t) {
    const uint32_t h = (uint32_t)(t >> 32), q = (h + 0x20000000u) >> 30;
    const float z = (float)(int32_t)(h - (q << 30)) * 1.4629180792671596e-9f;      // 2 pi / 2^32
    const float y = z * z;
    const float s = fmaf(z * y, fmaf(y, fmaf(y, fmaf(y, 2.7557319e-6f, -1.9841270e-4f), 8.3333333e-3f), -0.16666667f), z);
    const float c = fmaf(y, fmaf(y, fmaf(y, fmaf(y, fmaf(y, -2.7557319e-7f, 2.4801587e-5f), -1.3888889e-3f), 4.1666667e-2f), -0.5f), 1.0f);
    const float a = q & 1u ? s : c, b = q & 1u ? c : s;
    return make_float2((q + 1u) & 2u ? -a : a, q & 2u ? -b : b);
}
template <> __device__ __forceinline__ double2 turn_root<double>(uint64_t t) {
    const uint32_t q = (uint32_t)((t + 0x2000000000000000ull) >> 62);
    const int64_t r = (int64_t)(t - ((uint64_t)q << 62));
    const double x = fma((double)(int32_t)(r >> 32), 4294967296.0, (double)(uint32_t)r);
    const double z = x * 3.4061215800865545e-19;                                   // 2 pi / 2^64
    const double y = z * z;
    double s = -7.6471637318198165e-13, c = 4.7794773323873853e-14;                // -1/15!, 1/16!
    s = fma(s, y, 1.6059043836821613e-10);
    s = fma(s, y, -2.5052108385441720e-8);
    s = fma(s, y, 2.7557319223985893e-6);
    s = fma(s, y, -1.9841269841269841e-4);
    s = fma(s, y, 8.3333333333333333e-3);
    s = fma(s, y, -1.6666666666666667e-1);
    s = fma(z * y, s, z);
    c = fma(c, y, -1.1470745597729725e-11);
    c = fma(c, y, 2.0876756987868099e-9);
    c = fma(c, y, -2.7557319223985893e-7);
    c = fma(c, y, 2.4801587301587302e-5);
    c = fma(c, y, -1.3888888888888889e-3);
    c = fma(c, y, 4.1666666666666667e-2);
    c = fma(c, y, -0.5);
    c = fma(c, y, 1.0);
    const double a = q & 1u ? s : c, b = q & 1u ? c : s;
    return make_double2((q + 1u) & 2u ? -a : a, q & 2u ? -b : b);
}

// exp(sgn 2 pi i l / 2^(s+1)), l < 2^s, s <= 3
template <typename R, int SGN>
__device__ __forceinline__ cvec<R> root_mul(cvec<R> z, int l, int s) {
    const int q = l << (3 - s);                 // sixteenths of a turn, 0..7
    constexpr double C1 = 0.92387953251128675613, S1 = 0.38268343236508977173, H = 0.70710678118654752440;
    const double co[8] = {1.0, C1, H, S1, 0.0, -S1, -H, -C1};
    const double si[8] = {0.0, S1, H, C1, 1.0, C1, H, S1};
    if (q == 0) return z;
    if (q == 4) return SGN > 0 ? cmake<R>(-z.y, z.x) : cmake<R>(z.y, -z.x);
    if (q == 2) {
        const R h = (R)H;
        return SGN > 0 ? cmake<R>(h * (z.x - z.y), h * (z.x + z.y)) : cmake<R>(h * (z.x + z.y), h * (z.y - z.x));
    }
    if (q == 6) {
        const R h = (R)H;
        return SGN > 0 ? cmake<R>(-h * (z.x + z.y), h * (z.x - z.y)) : cmake<R>(h * (z.y - z.x), -h * (z.x + z.y));
    }
    const R c = (R)co[q], sn = (R)(SGN > 0 ? si[q] : -si[q]);
    return cmake<R>(z.x * c - z.y * sn, z.x * sn + z.y * c);
}

// The step on one line: transform of register bits 0..RA-1, with the twiddles
// W_i = exp(SGN 2 pi i vlow / 2^(j+1+i)) of register bit i after it (DIF) or
// before it (DIT), scaled by 2^(-RA/2).  vlow: the register bits below j;
// passengers may be among them (dep), and then it is formed per passenger value.
template <typename R, int SGN, bool DIT, int RA>
__device__ __forceinline__ void radix_line(cvec<R> (&v)[16], const QftStep &S, uint64_t gline, int lo) {
    constexpr int NA = 1 << RA, NF = 16 >> RA;
    const R sc = RA == 4 ? (R)0.25 : RA == 3 ? (R)0.35355339059327376220 : RA == 2 ? (R)0.5 : (R)0.70710678118654752440;
    auto twiddle = [&]() {
        if (S.j == 0) return;
        const uint64_t lowmask = (1ull << S.j) - 1ull;
        if (!S.dep) {
            const uint64_t vl = (gline >> lo) & lowmask;
#pragma unroll
            for (int i = 0; i < RA; ++i) {
                const uint64_t turns = vl << (63 - S.j - i);
                const cvec<R> w = turn_root<R>(SGN > 0 ? turns : 0ull - turns);
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (e >> i & 1) v[e] = cmul<R>(v[e], w);
            }
            return;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            uint64_t g = gline;
#pragma unroll
            for (int i = RA; i < 4; ++i)
                if (f >> (i - RA) & 1) g |= S.gb[i];
            const uint64_t vl = (g >> lo) & lowmask;
#pragma unroll
            for (int i = 0; i < RA; ++i) {
                const uint64_t turns = vl << (63 - S.j - i);
                const cvec<R> w = turn_root<R>(SGN > 0 ? turns : 0ull - turns);
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    if (a >> i & 1) v[f * NA + a] = cmul<R>(v[f * NA + a], w);
            }
        }
    };
    // scaled first: the step's sums then stay below 2^(RA/2) times the largest
    // amplitude, where the unscaled ones reach 2^RA times it and overflow earlier
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = cmake<R>(v[e].x * sc, v[e].y * sc);
    if (DIT) twiddle();
#pragma unroll
    for (int q = 0; q < RA; ++q) {
        const int s = DIT ? q : RA - 1 - q;
        const int half = 1 << s;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (e & half) continue;
            const int l = e & (half - 1);
            const cvec<R> x = v[e];
            if (DIT) {
                const cvec<R> y = root_mul<R, SGN>(v[e | half], l, s);
                v[e] = cmake<R>(x.x + y.x, x.y + y.y);
                v[e | half] = cmake<R>(x.x - y.x, x.y - y.y);
            } else {
                const cvec<R> y = v[e | half];
                v[e] = cmake<R>(x.x + y.x, x.y + y.y);
                v[e | half] = root_mul<R, SGN>(cmake<R>(x.x - y.x, x.y - y.y), l, s);
            }
        }
    }
    if (!DIT) twiddle();
}

// one radix step over a tile; `in` / `out`: HBM straight to / from registers
template <typename R, int SGN, bool DIT>
__device__ __forceinline__ void tile_step(cvec<R> *__restrict__ psi, const QftTile &A, const QftStep &S, uint64_t base,
                                          unsigned char *lds, uint32_t th, uint32_t nt, bool in, bool out) {
    const uint32_t lines = A.k > 4 ? 1u << (A.k - 4) : 1u;
    for (uint32_t line = th; line < lines; line += nt) {
        uint32_t bt = line;
#pragma unroll
        for (int i = 0; i < 4; ++i) bt = ((bt >> S.ipos[i]) << (S.ipos[i] + 1)) | (bt & ((1u << S.ipos[i]) - 1u));
        const uint64_t gl = base | tile_index(A, bt);
        const uint32_t sl = swz<R>(bt) * (uint32_t)sizeof(cvec<R>);
        cvec<R> v[16];
        if (in) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                uint64_t o = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e >> i & 1) o |= S.gb[i];
                v[e] = psi[gl | o];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                uint32_t o = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e >> i & 1) o ^= S.lb[i];
                v[e] = *(const cvec<R> *)(lds + (sl ^ o));
            }
        }
        switch (S.R) {
        case 1: radix_line<R, SGN, DIT, 1>(v, S, gl, A.lo); break;
        case 2: radix_line<R, SGN, DIT, 2>(v, S, gl, A.lo); break;
        case 3: radix_line<R, SGN, DIT, 3>(v, S, gl, A.lo); break;
        default: radix_line<R, SGN, DIT, 4>(v, S, gl, A.lo); break;
        }
        if (out) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                uint64_t o = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e >> i & 1) o |= S.gb[i];
                psi[gl | o] = v[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                uint32_t o = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e >> i & 1) o ^= S.lb[i];
                *(cvec<R> *)(lds + (sl ^ o)) = v[e];
            }
        }
    }
}

// Staging copies of a tile by `nt` threads (this one is `th`), eight amplitudes
// in flight per thread: with a load, a wait and a store per amplitude these
// copies were bound by latency (the mirrored last pass took 1.54 ms at 1 GiB).
template <typename R>
__device__ __forceinline__ void tile_in(const cvec<R> *__restrict__ psi, const QftTile &A, uint64_t base,
                                        unsigned char *lds, uint32_t th, uint32_t nt) {
    constexpr int U = 8;
    const uint32_t T = 1u << A.k;
    uint32_t t = th;
    for (; t + (U - 1) * nt < T; t += U * nt) {
        cvec<R> b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = psi[base | tile_index(A, t + u * nt)];
#pragma unroll
        for (int u = 0; u < U; ++u) *(cvec<R> *)(lds + swz<R>(t + u * nt) * sizeof(cvec<R>)) = b[u];
    }
    for (; t < T; t += nt) *(cvec<R> *)(lds + swz<R>(t) * sizeof(cvec<R>)) = psi[base | tile_index(A, t)];
}

// tile element t receives the element whose field is t's field reversed
template <typename R>
__device__ __forceinline__ void tile_out(cvec<R> *__restrict__ psi, const QftTile &A, uint64_t base,
                                         const unsigned char *lds, uint32_t th, uint32_t nt) {
    constexpr int U = 8;
    const uint32_t T = 1u << A.k, fm = (1u << A.rev_w) - 1u;
    auto src = [&](uint32_t t) {
        if (A.rev_w) t = (t & ~(fm << A.rev_tp)) | ((__brev((t >> A.rev_tp) & fm) >> (32 - A.rev_w)) << A.rev_tp);
        return *(const cvec<R> *)(lds + swz<R>(t) * sizeof(cvec<R>));
    };
    uint32_t t = th;
    for (; t + (U - 1) * nt < T; t += U * nt) {
        cvec<R> b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = src(t + u * nt);
#pragma unroll
        for (int u = 0; u < U; ++u) psi[base | tile_index(A, t + u * nt)] = b[u];
    }
    for (; t < T; t += nt) psi[base | tile_index(A, t)] = src(t);
}

// The tile of this workgroup.  Workgroups go round the eight XCDs in turn; each
// XCD takes a contiguous eighth of the tiles, so that the tiles that share
// memory pages and 256-byte channels run on one L2 (2.09 -> 1.99 ms for a
// 24-qubit transform on 2^27 complex64 amplitudes).
__device__ __forceinline__ uint64_t tile_number(const QftTile &A) {
    const uint64_t b = blockIdx.x;
    return A.tile0 + ((gridDim.x & 7u) ? b : (b & 7u) * (gridDim.x >> 3) + (b >> 3));
}

// one pass: the steps of one group on every tile
template <typename R, int SGN, bool DIT>
__global__ __launch_bounds__(QFT_MAX_THREADS) void k_qft_pass(cvec<R> *__restrict__ psi, QftTile A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint64_t tl = tile_number(A);
    uint64_t base = pdep64(tl, A.nl_mask) | A.fix_val;
    uint64_t base2 = base;
    if (A.mid_w) {
        // Two tiles whose middle bits mirror each other; the lower of the two
        // takes both.  The middle values are walked in blocks of 2^h lowest by
        // 2^h highest bits, so that the tiles in flight and their mirrors both
        // stay within few memory pages (walked in order, every mirror lies in
        // a page of its own: 1.61 against 1.54 ms a pass at 1 GiB, both before
        // the staging copies above kept eight amplitudes in flight: 0.68, and
        // 0.58 with the step reading HBM itself).
        const int w = A.mid_w, h = w / 2 < 5 ? w / 2 : 5;
        const uint64_t mm = (1ull << w) - 1ull, t = (base >> A.mid_lo) & mm, hm = (1ull << h) - 1ull;
        const uint64_t mv = (t & hm) | ((t >> h & hm) << (w - h)) | (t >> (2 * h) << h);
        const uint64_t rv = __brevll(mv) >> (64 - w);
        if (rv < mv) return;
        base = (base & ~(mm << A.mid_lo)) | (mv << A.mid_lo);
        base2 = (base & ~(mm << A.mid_lo)) | (rv << A.mid_lo);
    }
    // mirrored tiles: the upper half of the workgroup has the second one
    // (nothing to do where a tile is its own mirror)
    const uint32_t nt = A.mid_w ? blockDim.x / 2 : blockDim.x;
    const uint32_t q = threadIdx.x / nt, th = threadIdx.x % nt;
    const bool on = q == 0 || base2 != base;
    const uint32_t tbytes = (A.k < 4 ? 16u : 1u << A.k) * (uint32_t)sizeof(cvec<R>);
    unsigned char *lds = smem + q * tbytes;
    const uint64_t from = q ? base2 : base, to = q ? base : base2;
    if (!A.direct_in) {
        if (on) tile_in<R>(psi, A, from, lds, th, nt);
        __syncthreads();
    }
    for (int i = 0; i < A.nsteps; ++i) {
        const bool last = i == A.nsteps - 1;
        if (on)
            tile_step<R, SGN, DIT>(psi, A, A.st[i], from, lds, th, nt, i == 0 && A.direct_in, last && A.direct_out);
        if (!(last && A.direct_out)) __syncthreads();
    }
    if (!A.direct_out && on) tile_out<R>(psi, A, to, lds, th, nt);
}

// The spectral gradient's middle pass, on tiles of the register's lowest
// group and the rotated qubit: the last group of the inverse transform (DIF,
// negative sign), the rotation e^{i arg Lambda_k} Ry(t_k) of the pair (anc = 0,
// anc = 1) with k the reversed register index, and the first group of the
// transform back (DIT).  sin(t_k/2) = |k'| / (N/2 - 1), k' = k (k < N/2) or
// k - N (k > N/2); arg = +-pi/2 is an exact multiplication by +-i; k = 0 and
// k = N/2 are left alone.
template <typename R>
__global__ __launch_bounds__(QFT_MAX_THREADS) void k_spectral_mid(cvec<R> *__restrict__ psi, QftTile A, QftTile D,
                                                                  int anc_pos) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint64_t tl = tile_number(A);
    const uint64_t base = pdep64(tl, A.nl_mask);
    if (!A.direct_in) {
        tile_in<R>(psi, A, base, smem, threadIdx.x, blockDim.x);
        __syncthreads();
    }
    for (int i = 0; i < A.nsteps; ++i) {
        tile_step<R, -1, false>(psi, A, A.st[i], base, smem, threadIdx.x, blockDim.x, i == 0 && A.direct_in, false);
        __syncthreads();
    }
    const uint64_t half = 1ull << (A.m - 1);
    const double den = (double)(half - 1);
    const uint32_t T = 1u << A.k, ab = 1u << anc_pos;
    for (uint32_t p = threadIdx.x; p < T / 2; p += blockDim.x) {
        const uint32_t t = ((p >> anc_pos) << (anc_pos + 1)) | (p & (ab - 1u));
        const uint64_t rv = (base | tile_index(A, t)) >> A.lo;
        const uint64_t k = __brevll(rv) >> (64 - A.m);      // the low m bits of rv, reversed
        if (k == 0 || k == half) continue;
        const bool pos = k < half;
        const double sd = (double)(pos ? k : 2 * half - k) / den;      // exactly 1 at the largest |k'|
        const R sn = (R)sd, cs = (R)sqrt(fmax(0.0, 1.0 - sd * sd));
        cvec<R> *q0 = (cvec<R> *)(smem + swz<R>(t) * sizeof(cvec<R>));
        cvec<R> *q1 = (cvec<R> *)(smem + swz<R>(t | ab) * sizeof(cvec<R>));
        const cvec<R> a0 = *q0, a1 = *q1;
        const cvec<R> b0 = cmake<R>(cs * a0.x - sn * a1.x, cs * a0.y - sn * a1.y);
        const cvec<R> b1 = cmake<R>(sn * a0.x + cs * a1.x, sn * a0.y + cs * a1.y);
        *q0 = pos ? cmake<R>(-b0.y, b0.x) : cmake<R>(b0.y, -b0.x);
        *q1 = pos ? cmake<R>(-b1.y, b1.x) : cmake<R>(b1.y, -b1.x);
    }
    __syncthreads();
    for (int i = 0; i < D.nsteps; ++i) {
        const bool out = i == D.nsteps - 1 && D.direct_out;
        tile_step<R, 1, true>(psi, D, D.st[i], base, smem, threadIdx.x, blockDim.x, false, out);
        if (!out) __syncthreads();
    }
    if (!D.direct_out) tile_out<R>(psi, D, base, smem, threadIdx.x, blockDim.x);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

// contiguous low bits of a tile: runs of 128 bytes
static int qft_run_bits(sv_dtype dt) { return dt == SV_C128 ? 3 : 4; }

// tile bits: 64 KiB of LDS, so that two workgroups share a compute unit
static int qft_tile_bits(sv_state s, int max_local) {
    int k = s->dt == SV_C128 ? 12 : 13;
    if (max_local > 0) k = std::min(k, std::max(max_local, 8));
    return k;
}

static int tile_position(const QftTile &A, int q) {        // tile position of index bit q (-1: not in the tile)
    if (q < A.c) return q;
    if (q >= A.p1 && q < A.p1 + A.r1) return A.c + q - A.p1;
    if (q >= A.p2 && q < A.p2 + A.r2) return A.c + A.r1 + q - A.p2;
    return -1;
}

static int index_position(const QftTile &A, int t) {
    if (t < A.c) return t;
    if (t < A.c + A.r1) return A.p1 + t - A.c;
    return A.p2 + t - A.c - A.r1;
}

// steps of the register bits [j0, j0 + jn), which lie in the tile, in the
// order of the cascade; sets direct_in / direct_out (for a tile without
// reversal)
static void plan_steps(QftTile &A, sv_dtype dt, int j0, int jn, bool dit) {
    const int e = dt == SV_C128 ? 4 : 5;
    const uint32_t eb = (uint32_t)amp_bytes(dt);
    const int ns = (jn + 3) / 4;
    A.nsteps = ns;
    const int kv = std::max(A.k, 4);       // a tile below 16 amplitudes has passengers outside it (LDS padding only)
    int at = j0 + jn;
    for (int i = 0; i < ns; ++i) {
        // four qubits per step from the top: the remainder comes last, where the
        // passengers lie above it and share its twiddles
        const int R = std::min(4, at - j0);
        at -= R;
        QftStep &S = A.st[dit ? ns - 1 - i : i];
        memset(&S, 0, sizeof S);
        S.R = R;
        S.j = at;
        int pos[4];
        uint32_t used = 0;
        for (int b = 0; b < R; ++b) {
            pos[b] = tile_position(A, A.lo + at + b);
            used |= 1u << pos[b];
        }
        // passengers: the highest free positions, so that a wavefront's lanes
        // differ in the lowest tile bits
        for (int p = kv - 1, b = R; b < 4; --p)
            if (!(used >> p & 1)) {
                pos[b++] = p;
                used |= 1u << p;
            }
        for (int b = 0, p = 0; p < kv; ++p)
            if (used >> p & 1) S.ipos[b++] = p;
        for (int b = 0; b < 4; ++b) {
            S.lb[b] = swz_e(1u << pos[b], e) * eb;
            S.gb[b] = pos[b] < A.k ? 1ull << index_position(A, pos[b]) : 0ull;
            if (b >= R && (S.gb[b] >> A.lo & ((1ull << at) - 1ull))) S.dep = 1;
        }
    }
    // straight from or to HBM where runs of 64 bytes stay inside a wavefront's
    // access (the line's other half follows in another of the same 16 accesses)
    const int rb = qft_run_bits(dt), run = A.c == A.p1 ? A.c + A.r1 : A.c;
    auto direct = [&](const QftStep &S) { return A.k >= 4 && run >= rb && S.ipos[0] >= rb - 1; };
    A.direct_in = direct(A.st[0]);
    A.direct_out = direct(A.st[ns - 1]);
}

// The tile of a pass over the register bits [j0, j0 + jn): a run of low bits,
// the group, and up to `kfill` bits in all (more low bits, then the bits
// above the group), so that a workgroup has work for a wavefront or more.
static sv_status group_tile(sv_state s, int lo, int m, int j0, int jn, int kmax, uint64_t fix_mask, uint64_t fix_val,
                            QftTile &A) {
    memset(&A, 0, sizeof A);
    A.lo = lo;
    A.m = m;
    A.p1 = lo + j0;
    A.r1 = jn;
    const int kfill = std::min(kmax, 10);
    // runs of 256 bytes where the group leaves room, else of 128
    A.c = std::min(A.p1, std::min(qft_run_bits(s->dt) + 1, kmax - jn));
    if (A.c + A.r1 < kfill) A.c = std::min(A.p1, kfill - A.r1);
    while (A.c + A.r1 < kfill && A.p1 + A.r1 < s->n && !(fix_mask >> (A.p1 + A.r1) & 1)) ++A.r1;
    A.k = A.c + A.r1;
    const uint64_t all = (1ull << s->n) - 1ull;
    const uint64_t L = ((1ull << A.c) - 1ull) | (((1ull << A.r1) - 1ull) << A.p1);
    if (L & fix_mask) return fail(SV_EINVAL, "qft: a restricted bit overlaps the pass's local qubits");
    A.nl_mask = all & ~L & ~fix_mask;
    A.fix_val = fix_val;
    return SV_OK;
}

static unsigned block_of(const QftTile &A) {
    const uint32_t lines = A.k > 4 ? 1u << (A.k - 4) : 1u;
    unsigned nt = lines < 64 ? 64 : lines > (uint32_t)QFT_MAX_THREADS ? (unsigned)QFT_MAX_THREADS : lines;
    if (A.mid_w) nt = nt * 2 > (unsigned)QFT_MAX_THREADS ? (unsigned)QFT_MAX_THREADS : nt * 2;
    return nt;
}

// Launches of at most 2^22 workgroups: a grid holds less than 2^32 threads, which
// small tiles (a small max_local) on a large state would exceed.
template <typename F>
static void each_grid(QftTile &A, F launch) {
    const uint64_t tiles = 1ull << popcount64(A.nl_mask), most = 1ull << 22;
    for (A.tile0 = 0; A.tile0 < tiles; A.tile0 += most) launch(dim3((unsigned)std::min(tiles, most)));
}

static size_t tile_bytes(const QftTile &A, sv_dtype dt) {
    return ((size_t)1 << std::max(A.k, 4)) * amp_bytes(dt);
}

template <typename R, int SGN, bool DIT>
static sv_status launch_qft(sv_state s, QftTile A) {
    const uint64_t tiles = 1ull << popcount64(A.nl_mask);
    const bool in_regs = A.nsteps == 1 && A.direct_in && A.direct_out;     // never touches LDS
    const size_t lds = in_regs ? 0 : tile_bytes(A, s->dt) * (A.mid_w ? 2 : 1);
    TraceScope _ts(s->stream, "qft_pass", 2.0 * (double)(tiles << A.k) * sizeof(cvec<R>), 0.0);
    each_grid(A, [&](dim3 grid) {
        hipLaunchKernelGGL((k_qft_pass<R, SGN, DIT>), grid, dim3(block_of(A)), lds, s->stream, (cvec<R> *)s->data, A);
    });
    SV_HIP(hipGetLastError());
    return SV_OK;
}

static sv_status launch_pass(sv_state s, const QftTile &A, int sgn, bool dit) {
    if (s->dt == SV_C64)
        return sgn > 0 ? (dit ? launch_qft<float, 1, true>(s, A) : launch_qft<float, 1, false>(s, A))
                       : (dit ? launch_qft<float, -1, true>(s, A) : launch_qft<float, -1, false>(s, A));
    return sgn > 0 ? (dit ? launch_qft<double, 1, true>(s, A) : launch_qft<double, 1, false>(s, A))
                   : (dit ? launch_qft<double, -1, true>(s, A) : launch_qft<double, -1, false>(s, A));
}

// sizes of the groups of the register bits [j0, j0 + jn), lowest first:
// `low` bounds the lowest group, `up` the others; as few as possible, the upper ones even
static std::vector<int> cut_groups(int jn, int low, int up) {
    const int p = 1 + (jn > low ? (jn - low + up - 1) / up : 0);
    std::vector<int> g(p);
    int left = jn;
    for (int i = p - 1; i > 0; --i) {
        g[i] = std::min(up, (left + i) / (i + 1));
        left -= g[i];
    }
    g[0] = left;
    return g;
}

// the largest group of a pass whose lowest bit is index bit p
static int group_cap(sv_state s, int kmax, int p) { return kmax - std::min(p, qft_run_bits(s->dt)); }

// register bits [j0, j0 + jn) by plain passes (no reversal)
static sv_status run_groups(sv_state s, int lo, int m, int j0, int jn, int sgn, bool dit, uint64_t fix_mask,
                            uint64_t fix_val, int kmax) {
    if (!jn) return SV_OK;
    const std::vector<int> g = cut_groups(jn, group_cap(s, kmax, lo + j0), kmax - qft_run_bits(s->dt));
    std::vector<int> at(g.size());
    for (size_t i = 0, a = (size_t)j0; i < g.size(); a += (size_t)g[i++]) at[i] = (int)a;
    for (size_t q = 0; q < g.size(); ++q) {
        const size_t i = dit ? q : g.size() - 1 - q;
        QftTile A;
        SV_TRY(group_tile(s, lo, m, at[i], g[i], kmax, fix_mask, fix_val, A));
        plan_steps(A, s->dt, at[i], g[i], dit);
        SV_TRY(launch_pass(s, A, sgn, dit));
    }
    return SV_OK;
}

sv_status run_qft_cascade(sv_state s, const QftSpec &q, int max_local) {
    if (q.m < 1 || q.lo < 0 || q.lo + q.m > s->n) return fail(SV_EINVAL, "qft register out of range");
    if ((((1ull << q.m) - 1ull) << q.lo) & q.fix_mask)
        return fail(SV_EINVAL, "qft: a restricted bit overlaps the register");
    return run_groups(s, q.lo, q.m, 0, q.m, q.inverse ? -1 : 1, q.inverse != 0, q.fix_mask, q.fix_val,
                      qft_tile_bits(s, max_local));
}

// the transform in exact index order
static sv_status run_qft_ordered(sv_state s, int lo, int m, int sgn, int max_local) {
    const int kmax = qft_tile_bits(s, max_local), rb = qft_run_bits(s->dt);
    const int c = std::min(lo, rb);
    if (m + c <= kmax) {
        // the whole register in one tile: reversed on the way out
        QftTile A;
        SV_TRY(group_tile(s, lo, m, 0, m, kmax, 0, 0, A));
        plan_steps(A, s->dt, 0, m, false);
        A.rev_tp = A.c;
        A.rev_w = m;
        A.direct_out = 0;
        return launch_pass(s, A, sgn, false);
    }
    // the last pass: two tiles of the lowest g and the highest g register bits
    const int g = std::min((kmax - 1 - c) / 2, m / 2);
    SV_TRY(run_groups(s, lo, m, g, m - g, sgn, false, 0, 0, kmax));
    QftTile A;
    memset(&A, 0, sizeof A);
    A.lo = lo;
    A.m = m;
    A.c = c;
    A.p1 = lo;
    A.r1 = g;
    A.p2 = lo + m - g;
    A.r2 = g;
    A.k = c + 2 * g;
    A.nl_mask = ((1ull << s->n) - 1ull) & ~(((1ull << c) - 1ull) | (((1ull << g) - 1ull) << A.p1) |
                                            (((1ull << g) - 1ull) << A.p2));
    plan_steps(A, s->dt, 0, g, false);
    A.rev_tp = c;
    A.rev_w = 2 * g;
    A.direct_out = 0;
    A.mid_lo = lo + g;
    A.mid_w = m - 2 * g;      // at least 2: m > kmax - c and 2 g < kmax - c
    return launch_pass(s, A, sgn, false);
}

}  // namespace sv

using namespace sv;

extern "C" {

sv_status sv_qft(sv_state s, int q_lo, int m, int inverse, int swaps, int max_local) {
    clear_error();
    SV_TRY(check_state(s));
    if (m < 1 || q_lo < 0 || q_lo + m > s->n) return fail(SV_EINVAL, "register [%d,%d) outside the state", q_lo, q_lo + m);
    if (swaps) return run_qft_ordered(s, q_lo, m, inverse ? -1 : 1, max_local);
    return run_qft_cascade(s, QftSpec{q_lo, m, inverse ? 1 : 0, 0, 0}, max_local);
}

sv_status sv_spectral_derivative(sv_state s, int q_lo, int m, int anc, int max_local) {
    clear_error();
    SV_TRY(check_state(s));
    if (m < 2 || q_lo < 0 || q_lo + m > s->n)
        return fail(SV_EINVAL, "register [%d, %d) outside the state or narrower than 2 qubits", q_lo, q_lo + m);
    if (m > 30) return fail(SV_EINVAL, "register wider than 30 qubits");
    if (anc < 0 || anc >= s->n || (anc >= q_lo && anc < q_lo + m))
        return fail(SV_EINVAL, "qubit %d is outside the state or inside the register", anc);
    const int kmax = qft_tile_bits(s, max_local), rb = qft_run_bits(s->dt);
    // the middle pass: low run, lowest group, the rotated qubit
    const int c = std::min(q_lo, rb);
    const int g = std::min(m, kmax - c - 1);
    SV_TRY(run_groups(s, q_lo, m, g, m - g, -1, false, 0, 0, kmax));
    QftTile A;
    memset(&A, 0, sizeof A);
    A.lo = q_lo;
    A.m = m;
    A.c = c;
    A.p1 = q_lo;
    A.r1 = g;
    // A narrow register alone makes tiles of a few amplitudes, one per workgroup:
    // they are filled to 2^10 with more low bits, then with the bits above the
    // register and above the rotated qubit.  2 of 27 qubits at 8, complex128:
    // 5.09 -> 0.78 ms, and 3.75 with the transforms and the rotation in passes of
    // their own.
    const int kfill = std::min(kmax, 10);
    auto place_anc = [&] {
        A.p2 = anc >= A.c ? anc : 0;
        A.r2 = anc >= A.c ? 1 : 0;
        return A.c + A.r1 + A.r2;
    };
    while (place_anc() < kfill && A.c < q_lo) ++A.c;
    while (A.c + A.r1 + A.r2 < kfill) {
        if (q_lo + A.r1 < s->n && !(A.r2 && q_lo + A.r1 == A.p2)) ++A.r1;
        else if (A.r2 && A.p2 + A.r2 < s->n) ++A.r2;
        else break;
    }
    A.k = A.c + A.r1 + A.r2;
    A.nl_mask = ((1ull << s->n) - 1ull) & ~(((1ull << A.c) - 1ull) | (((1ull << A.r1) - 1ull) << A.p1) |
                                            (((1ull << A.r2) - 1ull) << A.p2));
    QftTile D = A;
    plan_steps(A, s->dt, 0, g, false);
    plan_steps(D, s->dt, 0, g, true);
    {
        TraceScope ts(s->stream, "spectral_mid", 2.0 * (double)dim_of(s->n) * amp_bytes(s->dt), 0.0);
        const size_t lds = tile_bytes(A, s->dt);
        const dim3 nt(block_of(A));
        const int ap = tile_position(A, anc);
        each_grid(A, [&](dim3 grid) {
            if (s->dt == SV_C64)
                hipLaunchKernelGGL(k_spectral_mid<float>, grid, nt, lds, s->stream, (float2 *)s->data, A, D, ap);
            else
                hipLaunchKernelGGL(k_spectral_mid<double>, grid, nt, lds, s->stream, (double2 *)s->data, A, D, ap);
        });
        SV_HIP(hipGetLastError());
    }
    return run_groups(s, q_lo, m, g, m - g, 1, true, 0, 0, kmax);
}

}  // extern "C"
