// Shared by the two executors of a gate list: the register-segment passes
// (sv_fused.hip) and the matrix-core passes (sv_blocks.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "sv_device.h"
#include "sv_internal.h"

namespace sv {

enum OpType { OP_U = 0, OP_X = 1, OP_SWAP = 2, OP_PHASE = 3 };

constexpr int MAX_HI = 20;

// a tile: the lowest c index bits and r gathered ones
struct TileLayout {
    uint64_t nl_mask;      // the other bits (the tile number is deposited here)
    int k, c, r;           // k = c + r
    int hpos[MAX_HI];      // index positions of the gathered bits, ascending
};
// the tile of a pass with the local bits L, filled up to k bits
void tile_layout(int n, int k, uint64_t L, TileLayout &t);

struct FOp {
    int type;
    int p0, p1;            // tile positions of the target(s)
    int pad;
    uint64_t lmask, lval;  // condition on local bits (tile coordinates)
    uint64_t gmask, gval;  // condition on non-local bits (global coordinates)
    uint64_t turns;        // OP_PHASE: phase as a fraction of a turn, 2^-64 units
    double u[8];           // OP_U
};

// an op as a segment runs it: targets as register bits, its local condition
// split into the register part and the part fixed per thread
struct ROp {
    int type;
    int j0, j1;            // register bits of the target(s)
    uint32_t rmask, rval;  // condition on the register index
    uint32_t tmask, tval;  // condition on the tile bits outside the segment's set
    uint32_t onm;          // bit m set: register index m meets the register condition
    uint64_t gmask, gval;  // condition on non-local bits
    double u[8];           // OP_U matrix; OP_PHASE: (cos, sin) of the phase in u[0], u[1]
};

// global offset of tile coordinate t
__device__ __forceinline__ uint64_t scatter_t(uint32_t t, int c, int r, const int *__restrict__ hpos) {
    uint64_t g = t & ((1u << c) - 1u);
    uint32_t h = t >> c;
    for (int i = 0; i < r; ++i)
        if (h >> i & 1u) g |= 1ull << hpos[i];
    return g;
}

__device__ __forceinline__ uint32_t insert0(uint32_t p, int pos) {
    return ((p >> pos) << (pos + 1)) | (p & ((1u << pos) - 1u));
}

// LDS slot of tile coordinate t: the bank index (the low e = log2(256 B /
// elem) bits) is XOR-ed with the folded higher bits.  The segment tables
// are built on the host with the same function.
__host__ __device__ __forceinline__ uint32_t swz_e(uint32_t t, int e) {
    const uint32_t m = (1u << e) - 1u;
    const uint32_t h = t >> e;
    return t ^ ((h ^ (h >> e) ^ (h >> (2 * e))) & m);
}
template <typename R>
__device__ __forceinline__ uint32_t swz(uint32_t t) {
    return swz_e(t, sizeof(cvec<R>) == 8 ? 5 : 4);
}

// The register-bit condition of an op is uniform.  Without one every pair
// is updated (no branches, so the pairs interleave); with one, a uniform
// branch per pair (on the op's precomputed mask of the register indices
// that meet it) skips the pairs it leaves alone.
template <typename R, int RB, int J>
__device__ __forceinline__ void reg_u(cvec<R> (&v)[1 << RB], const ROp &f) {
    const cvec<R> u00 = cmake<R>((R)f.u[0], (R)f.u[1]), u01 = cmake<R>((R)f.u[2], (R)f.u[3]);
    const cvec<R> u10 = cmake<R>((R)f.u[4], (R)f.u[5]), u11 = cmake<R>((R)f.u[6], (R)f.u[7]);
    if (f.rmask == 0) {
#pragma unroll
        for (int m = 0; m < (1 << RB); ++m) {
            if (m & (1 << J)) continue;
            const cvec<R> a0 = v[m], a1 = v[m | (1 << J)];
            v[m] = cmac2<R>(u00, a0, u01, a1);
            v[m | (1 << J)] = cmac2<R>(u10, a0, u11, a1);
        }
    } else {
        const uint32_t on = f.onm;
#pragma unroll
        for (int m = 0; m < (1 << RB); ++m) {
            if (m & (1 << J)) continue;
            if (!(on >> m & 1u)) continue;
            const cvec<R> a0 = v[m], a1 = v[m | (1 << J)];
            v[m] = cmac2<R>(u00, a0, u01, a1);
            v[m | (1 << J)] = cmac2<R>(u10, a0, u11, a1);
        }
    }
}

// A conditional swap in place on the bits, d = (a ^ b) & mask, a ^= d,
// b ^= d: three instructions per pair of words (the AND folds into one
// three-input bit op), where selects of both words into fresh registers and
// moves back took four, with no register permutation for the compiler to resolve
__device__ __forceinline__ void cswap_bits(float &a, float &b, uint32_t mask) {
    const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    const uint32_t d = (x ^ y) & mask;
    a = __builtin_bit_cast(float, x ^ d);
    b = __builtin_bit_cast(float, y ^ d);
}
__device__ __forceinline__ void cswap_bits(double &a, double &b, uint32_t mask) {
    const uint64_t m64 = mask ? ~0ull : 0ull;
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const uint64_t d = (x ^ y) & m64;
    a = __builtin_bit_cast(double, x ^ d);
    b = __builtin_bit_cast(double, y ^ d);
}

template <typename R, int RB, int J>
__device__ __forceinline__ void reg_x(cvec<R> (&v)[1 << RB], const ROp &f) {
    const uint32_t on = f.onm;
#pragma unroll
    for (int m = 0; m < (1 << RB); ++m) {
        if (m & (1 << J)) continue;
        const uint32_t mask = 0u - (on >> m & 1u);
        cswap_bits(v[m].x, v[m | (1 << J)].x, mask);
        cswap_bits(v[m].y, v[m | (1 << J)].y, mask);
    }
}

template <typename R, int RB>
__device__ __forceinline__ void reg_phase(cvec<R> (&v)[1 << RB], const ROp &f) {
    const cvec<R> ph = cmake<R>((R)f.u[0], (R)f.u[1]);
    const uint32_t on = f.onm;
#pragma unroll
    for (int m = 0; m < (1 << RB); ++m)
        if (on >> m & 1u) v[m] = cmul<R>(v[m], ph);
}

template <typename R, int RB>
__device__ __forceinline__ void reg_apply(cvec<R> (&v)[1 << RB], const ROp &f) {
    switch (f.type) {
    case OP_PHASE: reg_phase<R, RB>(v, f); break;
    case OP_X:
        switch (f.j0) {
        case 0: reg_x<R, RB, 0>(v, f); break;
        case 1: reg_x<R, RB, 1 < RB ? 1 : 0>(v, f); break;
        case 2: reg_x<R, RB, 2 < RB ? 2 : 0>(v, f); break;
        case 3: reg_x<R, RB, 3 < RB ? 3 : 0>(v, f); break;
        default: reg_x<R, RB, 4 < RB ? 4 : 0>(v, f); break;
        }
        break;
    default:
        switch (f.j0) {
        case 0: reg_u<R, RB, 0>(v, f); break;
        case 1: reg_u<R, RB, 1 < RB ? 1 : 0>(v, f); break;
        case 2: reg_u<R, RB, 2 < RB ? 2 : 0>(v, f); break;
        case 3: reg_u<R, RB, 3 < RB ? 3 : 0>(v, f); break;
        default: reg_u<R, RB, 4 < RB ? 4 : 0>(v, f); break;
        }
        break;
    }
}

// LDS access by byte address.  The kernels that use these have no static LDS,
// so their dynamic area starts at address 0 (the host checks this): a slot's
// byte offset, formed by XOR, is then its address with no base added.
template <typename R> using v2r = R __attribute__((ext_vector_type(2)));
template <typename T> using lptr = __attribute__((address_space(3))) T *;
template <typename R>
__device__ __forceinline__ cvec<R> lds_ld(uint32_t a) {
    const v2r<R> x = *(lptr<v2r<R>>)(uintptr_t)a;
    return cmake<R>(x.x, x.y);
}
template <typename R>
__device__ __forceinline__ void lds_st(uint32_t a, cvec<R> v) {
    v2r<R> x;
    x.x = v.x;
    x.y = v.y;
    *(lptr<v2r<R>>)(uintptr_t)a = x;
}

struct PGate {
    int kind;          // 0 dense U, 1 X, 2 SWAP, 3 diagonal (phases)
    int t0, t1;
    uint64_t cmask, cval;
    uint64_t qubits;   // all qubits touched (targets + controls)
    uint64_t need;     // qubits that must be local
    double u[8];
};

// the ops of a gate on a tile with the local bits L
void emit_ops(const PGate &g, uint64_t L, std::vector<FOp> &ops);
// an op as ops on the register bits of the tile positions S; returns their number
int to_rops(const FOp &f, uint32_t S, int RB, std::vector<ROp> &rops);
// number of the ops a gate turns into (a diagonal gate: one phase per entry that is not 1)
int ops_of(const PGate &g);

// ---- planning (sv_plan.cpp) ------------------------------------------------
// A gate as the planners see it.
struct PlanItem {
    uint64_t order;            // gates that share one of these qubits keep their order
    uint64_t need;             // qubits that have to be in the window it runs in
    uint64_t ext;              // further qubits it reads from outside any window
    int ops;
};
struct PlanWindow {
    uint64_t set;              // the window's qubits
    std::vector<int> take;     // the gates it runs, in program order
};
// Cuts items into windows of at most `cap` qubits that contain `base`.  A gate
// may read at most item_out qubits from outside its window, a window's gates
// together at most window_out (< 0: no bound); at most max_ops ops per window.
// cap has to leave room for any one gate next to `base`.
void plan_windows(const std::vector<PlanItem> &items, int cap, uint64_t base, int item_out, int window_out,
                  int max_ops, std::vector<PlanWindow> &out);
// the same cut with windows that take the earliest gates until they are full
void plan_earliest(const std::vector<PlanItem> &items, int cap, uint64_t base, int max_ops,
                   std::vector<PlanWindow> &out);

// ---- matrix-core passes (sv_blocks.hip) -------------------------------------
// every gate is unitary and fits a block of four qubits, and one at least mixes amplitudes
bool blocks_eligible(sv_state s, const std::vector<PGate> &gates);
struct BlockPlan {
    int k, c, nblocks;
    std::vector<PlanWindow> wins;                  // the passes
    std::vector<std::vector<PlanWindow>> blocks;   // of each pass (gates: places in its window)
};
// on tiles of k qubits with the lowest c in them: 8 <= k <= 13, c <= k - 4, eligible gates
void plan_blocks(int n, const std::vector<PGate> &gates, int k, int c, BlockPlan &plan);
sv_status run_blocks(sv_state s, const std::vector<PGate> &gates, const BlockPlan &plan);
// the same for a configuration that may be pinned
sv_status run_blocks(sv_state s, const std::vector<PGate> &gates, int k, int c);

}  // namespace sv
