// LDS-fused passes: a circuit is cut into passes; each pass stages tiles of
// 2^k amplitudes (k "local" qubits) in LDS, applies every gate it can there
// and writes the tile back, so a run of gates costs one HBM round trip.
//
// Tile layout: the local qubits are the low c bits of the index plus a set
// of higher "gathered" bits.  The low bits keep HBM accesses contiguous
// (2^c amplitudes per segment); the gathered bits are the targets the pass
// needs.  All other bits are fixed per tile (the tile id is deposited into
// them), so controls and phases on them are uniform over a workgroup.
//
// Inside a tile the gates run from registers: the pass's gate list is cut
// into segments whose targets fall in at most RB tile positions S.  For a
// segment every thread holds the 2^RB amplitudes that differ only in S (its
// other tile bits come from the thread index), applies the segment's gates
// without any exchange, and hands the tile back through LDS.  The LDS
// layout is XOR-swizzled so that threads whose amplitudes sit 2^p apart hit
// distinct banks.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "sv_fused.h"

namespace sv {

constexpr int FUSE_BLOCK = 256;

constexpr int MAX_RB = 5;

struct FSeg {
    int pos[MAX_RB];       // tile positions held in registers (register bit i = pos[i]), ascending
    int nops, op_off;
    // LDS byte offsets (swz of the tile bits times the amplitude size) that
    // register index m is read from and written to.  They differ from the
    // slot of m itself where the segment's register permutations at its
    // start or end (register-controlled NOTs that commute there) were
    // folded into them.
    uint32_t off[1 << MAX_RB];
    uint32_t offw[1 << MAX_RB];
};

struct FPass {
    TileLayout t;
    int nseg, seg_off;
};

// One fused pass.  Blocks walk the tiles tile = block + i * (blocks in the
// grid): the grid is what the device holds at once, or one tile per block
// when that covers them all.  (Reading the next tile into registers during
// this tile's segments cost more in registers than it hid.)
template <typename R, int RB, int NT = FUSE_BLOCK>
__global__ __launch_bounds__(NT) void k_fused(cvec<R> *__restrict__ psi, const FPass *__restrict__ passes,
                                                       int pi, const FSeg *__restrict__ segs,
                                                       const ROp *__restrict__ ops, uint64_t ntiles) {
    extern __shared__ unsigned char smem_raw[];
    cvec<R> *tile = reinterpret_cast<cvec<R> *>(smem_raw);
    const FPass &P = passes[pi];
    const int k = P.t.k, c = P.t.c, r = P.t.r;
    const uint32_t T = 1u << k;
    const uint64_t tstride = (uint64_t)gridDim.x * gridDim.y;
    const int *hpos = P.t.hpos;

    // HBM <-> LDS with U loads in flight per thread.  scatter_t is a bit
    // deposit, so the thread's part (bits below log2 NT), the part of
    // the unrolled index u and that of the outer step t0 combine by OR; the
    // offsets of u's bits are formed once and combined per load (uniform
    // values: a table of all U combinations held 48 more vector registers
    // through the whole kernel).
    constexpr int U = sizeof(R) == 4 ? 16 : 8;
    constexpr int LB = NT == 512 ? 9 : 8, LU = sizeof(R) == 4 ? 4 : 3;      // log2 NT, log2 U
    const uint64_t gthr = scatter_t(threadIdx.x & (T - 1u), c, r, hpos);
    // swz is XOR-linear too: the LDS slot of t0 + u 256 + thread is
    // swz(thread) ^ swz(t0) ^ swz(u 256)
    const uint32_t sthr = swz<R>(threadIdx.x);
    const bool big = T >= NT * U;
    // the offsets of the bits of u (HBM and LDS), combined per load
    uint64_t hb[LU];
    uint32_t hs[LU];
#pragma unroll
    for (int i = 0; i < LU; ++i) {
        hb[i] = big ? scatter_t(1u << (LB + i), c, r, hpos) : 0;
        hs[i] = swz<R>(1u << (LB + i)) * (uint32_t)sizeof(cvec<R>);
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
    for (uint64_t tl = (uint64_t)blockIdx.x + (uint64_t)blockIdx.y * gridDim.x; tl < ntiles; tl += tstride) {
        const uint64_t base = pdep64(tl, P.t.nl_mask);
        if (big) {
            for (uint32_t t0 = 0; t0 < T; t0 += NT * U) {
                const uint64_t g0 = base | gthr | scatter_t(t0, c, r, hpos);
                const uint32_t s0 = (sthr ^ swz<R>(t0)) * (uint32_t)sizeof(cvec<R>);
                cvec<R> buf[U];
#pragma unroll
                for (int u = 0; u < U; ++u) buf[u] = psi[g0 | uoff(u)];
#pragma unroll
                for (int u = 0; u < U; ++u) lds_st<R>(s0 ^ uswz(u), buf[u]);
            }
        } else {
            for (uint32_t t = threadIdx.x; t < T; t += NT) tile[swz<R>(t)] = psi[base | scatter_t(t, c, r, hpos)];
        }
        __syncthreads();

        const uint32_t lines = T >> RB;                  // register lines per tile
        for (int sg = 0; sg < P.nseg; ++sg) {
            const FSeg &S = segs[P.seg_off + sg];
            // swz is XOR-linear and bt and the register bits are disjoint, so the
            // slot of bt | (bits of m) is swz(bt) ^ S.off[m] (the table is uniform,
            // in bytes, as the slot is used)
            uint32_t off[1 << RB];
#pragma unroll
            for (int m = 0; m < (1 << RB); ++m) off[m] = S.off[m];
            const ROp *op0 = ops + S.op_off;
            for (uint32_t line = threadIdx.x; line < lines; line += NT) {
                // the tile bits outside the register positions: the line index
                // with a zero inserted at each position, lowest first
                uint32_t bt = line;
#pragma unroll
                for (int i = 0; i < RB; ++i) bt = insert0(bt, S.pos[i]);
                const uint32_t sbt = swz<R>(bt) * (uint32_t)sizeof(cvec<R>);
                cvec<R> v[1 << RB];
#pragma unroll
                for (int m = 0; m < (1 << RB); ++m) v[m] = lds_ld<R>(sbt ^ off[m]);
                for (int o = 0; o < S.nops; ++o) {
                    const ROp &f = op0[o];
                    if ((base & f.gmask) != f.gval || (bt & f.tmask) != f.tval) continue;
                    reg_apply<R, RB>(v, f);
                }
#pragma unroll
                for (int m = 0; m < (1 << RB); ++m) lds_st<R>(sbt ^ S.offw[m], v[m]);
            }
            __syncthreads();
        }

        if (big) {
            for (uint32_t t0 = 0; t0 < T; t0 += NT * U) {
                const uint64_t g0 = base | gthr | scatter_t(t0, c, r, hpos);
                const uint32_t s0 = (sthr ^ swz<R>(t0)) * (uint32_t)sizeof(cvec<R>);
                cvec<R> buf[U];
#pragma unroll
                for (int u = 0; u < U; ++u) buf[u] = lds_ld<R>(s0 ^ uswz(u));
#pragma unroll
                for (int u = 0; u < U; ++u) psi[g0 | uoff(u)] = buf[u];
            }
        } else {
            for (uint32_t t = threadIdx.x; t < T; t += NT) psi[base | scatter_t(t, c, r, hpos)] = tile[swz<R>(t)];
        }
        // the next tile is written into the LDS this one was read from
        if (tl + tstride < ntiles) __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static int g_lds_limit = 0;
static bool g_fused_lds_at_0 = false;   // k_fused has no static LDS: its tile starts at address 0

static int lds_limit_bytes() {
    if (g_lds_limit) return g_lds_limit;
    int dev = 0;
    hipGetDevice(&dev);
    hipDeviceProp_t prop;
    int lim = 65536;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.sharedMemPerBlock > 0)
        lim = (int)prop.sharedMemPerBlock;
    if (lim > 147456) lim = 147456;   // the largest power-of-two tile (128 KiB) plus headroom
    bool ok = true;
    const void *fk[] = {(const void *)k_fused<float, 5>, (const void *)k_fused<float, 4>,
                        (const void *)k_fused<float, 4, 512>, (const void *)k_fused<float, 3>,
                        (const void *)k_fused<double, 4>, (const void *)k_fused<double, 3>};
    for (const void *f : fk) ok &= hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lim) == hipSuccess;
    bool at0 = true;
    for (const void *f : fk) {
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, f) != hipSuccess || fa.sharedSizeBytes != 0) at0 = false;
    }
    (void)hipGetLastError();
    if (!ok) lim = 65536;
    g_fused_lds_at_0 = at0;
    g_lds_limit = lim;
    return lim;
}

// low index bits every pass keeps local (contiguous HBM segments of 2^c
// amplitudes): 256-byte segments by default; SV_FUSED_LOWBITS (2..10) overrides
static int low_bits_for(sv_dtype dt) {
    if (const char *e = getenv("SV_FUSED_LOWBITS")) {
        const int v = atoi(e);
        if (v >= 2 && v <= 10) return v;
    }
    return dt == SV_C128 ? 4 : 5;
}

static int clamp_k(sv_state s, int max_local) {
    int k = max_local > 0 ? max_local : default_max_local(s->dt);
    const int bytes = (int)amp_bytes(s->dt);
    while (k > 1 && (1 << k) * bytes > lds_limit_bytes()) --k;
    if (k > s->n) k = s->n;
    return k;
}

static inline dim3 tile_grid(uint64_t tiles) {
    if (tiles <= 0x7fffffffull) return dim3((unsigned)tiles);
    return dim3(1u << 30, (unsigned)(tiles >> 30));
}

static bool unit_modulus(double re, double im) { return fabs(re * re + im * im - 1.0) < 1e-13; }

static uint64_t angle_turns(double re, double im) {
    // arg(re + i im) as a fraction of a turn in [-1/2, 1/2), rounded to 2^-64
    long double a = atan2l((long double)im, (long double)re) / (2.0L * 3.14159265358979323846264338327950288L);
    if (a >= 0.5L) a -= 1.0L;
    return (uint64_t)(int64_t)llroundl(ldexpl(a, 64));
}

static sv_status to_pgates(sv_state s, const sv_gate *gates, int n_gates, std::vector<PGate> &out) {
    out.clear();
    out.reserve(n_gates);
    for (int i = 0; i < n_gates; ++i) {
        const sv_gate &g = gates[i];
        PGate p;
        memset(&p, 0, sizeof p);
        if (g.n_ctrls < 0 || g.n_ctrls > SV_MAX_CTRLS) return fail(SV_EINVAL, "gate %d: n_ctrls out of range", i);
        int qs[2] = {g.target, g.target2};
        int nq = g.kind == SV_GATE_SWAP ? 2 : 1;
        if (g.kind != SV_GATE_U && g.kind != SV_GATE_X && g.kind != SV_GATE_SWAP)
            return fail(SV_EINVAL, "gate %d: unknown kind %d", i, g.kind);
        sv_status st = check_qubits(s, qs, nq, g.ctrls, g.ctrl_vals, g.n_ctrls, &p.cmask, &p.cval);
        if (st != SV_OK) return fail(st, "gate %d: %s", i, sv_last_error());
        p.t0 = g.target;
        p.t1 = nq == 2 ? g.target2 : -1;
        p.qubits = p.cmask | (1ull << g.target) | (nq == 2 ? 1ull << g.target2 : 0);
        if (g.kind == SV_GATE_X) {
            p.kind = 1;
            p.need = 1ull << g.target;
        } else if (g.kind == SV_GATE_SWAP) {
            p.kind = 2;
            p.need = (1ull << g.target) | (1ull << g.target2);
        } else {
            memcpy(p.u, g.u, sizeof p.u);
            for (int j = 0; j < 8; ++j)
                if (!isfinite(p.u[j])) return fail(SV_EINVAL, "gate %d: non-finite matrix entry", i);
            const bool diag = p.u[2] == 0 && p.u[3] == 0 && p.u[4] == 0 && p.u[5] == 0 &&
                              unit_modulus(p.u[0], p.u[1]) && unit_modulus(p.u[6], p.u[7]);
            p.kind = diag ? 3 : 0;
            p.need = diag ? 0 : 1ull << g.target;
        }
        out.push_back(p);
    }
    return SV_OK;
}

struct HostPass {
    FPass hdr;
    std::vector<FOp> ops;
};

int ops_of(const PGate &g) {
    if (g.kind != 3) return 1;
    int c = 0;
    if (!(g.u[0] == 1 && g.u[1] == 0)) ++c;
    if (!(g.u[6] == 1 && g.u[7] == 0)) ++c;
    return c;
}

void tile_layout(int n, int k, uint64_t L, TileLayout &t) {
    // fill the local set up to k with the lowest free bits
    for (int q = 0; q < n && popcount64(L) < k; ++q) L |= 1ull << q;
    int c = 0;
    while (c < n && (L >> c & 1)) ++c;
    t.c = c;
    t.k = popcount64(L);
    t.r = 0;
    for (int q = c; q < n; ++q)
        if (L >> q & 1) t.hpos[t.r++] = q;
    const uint64_t all = (n >= 64) ? ~0ull : ((1ull << n) - 1ull);
    t.nl_mask = all & ~L;
}

static int tile_pos(uint64_t L, int q) { return popcount64(L & ((1ull << q) - 1ull)); }

static uint64_t to_tile_mask(uint64_t L, uint64_t gm) {
    uint64_t r = 0;
    for (int q = 0; q < 64; ++q)
        if ((gm >> q & 1) && (L >> q & 1)) r |= 1ull << tile_pos(L, q);
    return r;
}

void emit_ops(const PGate &g, uint64_t L, std::vector<FOp> &ops) {
    FOp f;
    memset(&f, 0, sizeof f);
    const uint64_t lc = g.cmask & L, gc = g.cmask & ~L;
    f.lmask = to_tile_mask(L, lc);
    f.lval = to_tile_mask(L, g.cval & lc);
    f.gmask = gc;
    f.gval = g.cval & gc;
    if (g.kind == 3) {
        // diag(u00, u11): phase on target = 0 and on target = 1 (with the controls)
        const uint64_t tb = 1ull << g.t0;
        for (int b = 0; b < 2; ++b) {
            const double re = g.u[6 * b], im = g.u[6 * b + 1];
            if (re == 1 && im == 0) continue;
            FOp h = f;
            h.type = OP_PHASE;
            if (L & tb) {
                h.lmask |= 1ull << tile_pos(L, g.t0);
                if (b) h.lval |= 1ull << tile_pos(L, g.t0);
            } else {
                h.gmask |= tb;
                if (b) h.gval |= tb;
            }
            h.turns = angle_turns(re, im);
            ops.push_back(h);
        }
        return;
    }
    f.type = g.kind == 0 ? OP_U : g.kind == 1 ? OP_X : OP_SWAP;
    f.p0 = tile_pos(L, g.t0);
    f.p1 = g.kind == 2 ? tile_pos(L, g.t1) : 0;
    memcpy(f.u, g.u, sizeof f.u);
    ops.push_back(f);
}

// A pass's ops are interpreted one by one, so their number costs nothing by
// itself; the bound keeps the tables of a pass small.
constexpr int MAX_OPS_PER_PASS = 256;

// early: windows that take the earliest gates (the tuner's choice where their
// passes run as fast, see fusion_config)
static void plan(int n, int kmax, int c0, const std::vector<PGate> &gates, std::vector<HostPass> &passes,
                 bool early = false) {
    passes.clear();
    // a gate needs at most two local bits besides the low run, so every pass
    // takes at least the first gate left (callers pass c0 <= kmax - 2)
    c0 = std::max(0, std::min(c0, kmax - 2));
    std::vector<PlanItem> items;
    items.reserve(gates.size());
    for (const PGate &g : gates) items.push_back({g.qubits, g.need, 0, ops_of(g)});
    std::vector<PlanWindow> wins;
    const uint64_t low = (1ull << std::min(c0, n)) - 1ull;
    if (early) plan_earliest(items, kmax, low, MAX_OPS_PER_PASS, wins);
    else plan_windows(items, kmax, low, -1, -1, MAX_OPS_PER_PASS, wins);
    const uint64_t all = n >= 64 ? ~0ull : (1ull << n) - 1ull;
    for (const PlanWindow &w : wins) {
        HostPass hp;
        memset(&hp.hdr, 0, sizeof hp.hdr);
        tile_layout(n, kmax, w.set, hp.hdr.t);
        for (int i : w.take) emit_ops(gates[i], ~hp.hdr.t.nl_mask & all, hp.ops);
        if (!hp.ops.empty()) passes.push_back(std::move(hp));
    }
}

// tile positions a gate must hold in registers
static uint32_t op_targets(const FOp &f) {
    if (f.type == OP_PHASE) return 0;
    if (f.type == OP_SWAP) return (1u << f.p0) | (1u << f.p1);
    return 1u << f.p0;
}

static uint32_t compress_bits(uint32_t x, uint32_t S) {   // tile bits in S -> register bits
    uint32_t r = 0;
    int j = 0;
    for (int p = 0; p < 32; ++p)
        if (S >> p & 1) {
            if (x >> p & 1) r |= 1u << j;
            ++j;
        }
    return r;
}

// bit m set for the register indices m < 2^RB with (m & rmask) == rval
static uint32_t on_mask(uint32_t rmask, uint32_t rval, int RB) {
    uint32_t on = 0;
    for (uint32_t m = 0; m < (1u << RB); ++m)
        if ((m & rmask) == rval) on |= 1u << m;
    return on;
}

// a tile-level op as ops on the register bits of the positions S (its local
// conditions outside S become per-thread conditions); returns their number
int to_rops(const FOp &f, uint32_t S, int RB, std::vector<ROp> &rops) {
    ROp o;
    memset(&o, 0, sizeof o);
    o.type = f.type;
    o.j0 = f.type == OP_PHASE ? 0 : __builtin_ctz(compress_bits(1u << f.p0, S));
    o.j1 = f.type == OP_SWAP ? __builtin_ctz(compress_bits(1u << f.p1, S)) : 0;
    o.rmask = compress_bits((uint32_t)f.lmask & S, S);
    o.rval = compress_bits((uint32_t)f.lval & S, S);
    o.tmask = (uint32_t)f.lmask & ~S;
    o.tval = (uint32_t)f.lval & ~S;
    o.onm = on_mask(o.rmask, o.rval, RB);
    o.gmask = f.gmask;
    o.gval = f.gval;
    if (f.type == OP_PHASE) {
        const long double a = ldexpl((long double)(int64_t)f.turns, -64) * 2.0L * 3.14159265358979323846264338327950288L;
        o.u[0] = (double)cosl(a);
        o.u[1] = (double)sinl(a);
    } else {
        memcpy(o.u, f.u, sizeof o.u);
    }
    if (f.type != OP_SWAP) {
        rops.push_back(o);
        return 1;
    }
    // SWAP(a, b) = CX(a -> b) CX(b -> a) CX(a -> b), each an X on
    // a register bit controlled by the other
    const int a = o.j0, b = o.j1;
    ROp x = o;
    x.type = OP_X;
    for (int r = 0; r < 3; ++r) {
        const int tgt = r == 1 ? a : b, ctl = r == 1 ? b : a;
        x.j0 = tgt;
        x.j1 = 0;
        x.rmask = o.rmask | (1u << ctl);
        x.rval = o.rval | (1u << ctl);
        x.onm = on_mask(x.rmask, x.rval, RB);
        rops.push_back(x);
    }
    return 3;
}

// Register-controlled NOTs at either end of a segment permute the register
// indices only, so they need no arithmetic: those that commute to the start
// (with every op before them that is not moved) become the read offsets,
// those that commute to the end the write offsets, and both leave the op
// list.  A NOT moves only if its condition is on register bits alone (no
// tile or non-local control); an op touches its target and condition bits,
// a phase every register bit.  If P is the product of the leading NOTs in
// program order, register m holds the amplitude of P^-1(m) after them; if T
// is that of the trailing ones, the value in register m ends at T(m).
static void fold_permutations(FSeg &g, std::vector<ROp> &rops, int RB) {
    const size_t n = (size_t)g.nops, b0 = (size_t)g.op_off;
    const uint32_t all = (1u << RB) - 1u;
    auto movable = [](const ROp &f) { return f.type == OP_X && f.tmask == 0 && f.gmask == 0; };
    auto touched = [&](const ROp &f) { return f.type == OP_PHASE ? all : ((1u << f.j0) | f.rmask); };
    auto xmap = [](const ROp &f, uint32_t m) { return (m & f.rmask) == f.rval ? m ^ (1u << f.j0) : m; };
    std::vector<char> lead(n, 0), trail(n, 0);
    uint32_t blocked = 0;
    for (size_t i = 0; i < n; ++i) {
        const ROp &f = rops[b0 + i];
        if (movable(f) && !(touched(f) & blocked))
            lead[i] = 1;
        else
            blocked |= touched(f);
    }
    blocked = 0;
    for (size_t i = n; i-- > 0;) {
        const ROp &f = rops[b0 + i];
        if (lead[i]) continue;
        if (movable(f) && !(touched(f) & blocked))
            trail[i] = 1;
        else
            blocked |= touched(f);
    }
    uint32_t base[1 << MAX_RB];
    for (uint32_t m = 0; m <= all; ++m) base[m] = g.off[m];
    for (uint32_t m = 0; m <= all; ++m) {
        uint32_t p = m;      // P^-1(m): the leading NOTs from the last to the first
        for (size_t i = n; i-- > 0;)
            if (lead[i]) p = xmap(rops[b0 + i], p);
        uint32_t q = m;      // T(m), where the value in register m ends: the trailing NOTs from the first
        for (size_t i = 0; i < n; ++i)
            if (trail[i]) q = xmap(rops[b0 + i], q);
        g.off[m] = base[p];
        g.offw[m] = base[q];
    }
    size_t w = b0;
    for (size_t i = 0; i < n; ++i)
        if (!lead[i] && !trail[i]) rops[w++] = rops[b0 + i];
    rops.resize(w);
    g.nops = (int)(w - b0);
}

// cut a pass's gate list into register segments of at most RB target
// positions.  Gates that touch disjoint qubits commute, so a segment takes
// every gate that is ready (all earlier gates it does not commute with are
// placed) and whose targets fit, in program order, not only a contiguous run.
static void segment_pass(const HostPass &hp, int RB, int swz_bits, std::vector<FSeg> &segs, std::vector<ROp> &rops) {
    const int k = hp.hdr.t.k;
    const std::vector<FOp> &ops = hp.ops;
    const size_t n = ops.size();
    // conflict: a target of one is a target or a local control of the other
    // (controls on non-local bits never coincide with a target: targets are local)
    std::vector<std::vector<int>> pred(n);
    for (size_t b = 0; b < n; ++b) {
        const uint32_t tb = op_targets(ops[b]), qb = tb | (uint32_t)ops[b].lmask;
        for (size_t a = 0; a < b; ++a) {
            const uint32_t ta = op_targets(ops[a]), qa = ta | (uint32_t)ops[a].lmask;
            if ((ta & qb) || (tb & qa)) pred[b].push_back((int)a);
        }
    }
    std::vector<char> done(n, 0);
    size_t left = n;
    while (left) {
        uint32_t S = 0;
        std::vector<int> seg;
        for (bool progress = true; progress;) {
            progress = false;
            for (size_t b = 0; b < n; ++b) {
                if (done[b]) continue;
                bool ready = true;
                for (int a : pred[b])
                    if (!done[a]) {
                        ready = false;
                        break;
                    }
                if (!ready || popcount64(S | op_targets(ops[b])) > RB) continue;
                S |= op_targets(ops[b]);
                done[b] = 1;
                --left;
                seg.push_back((int)b);
                progress = true;
            }
        }
        // fill with the highest free positions: the threads of a wavefront then
        // differ in the low tile bits (contiguous LDS slots)
        for (int p = k - 1; p >= 0 && popcount64(S) < RB; --p) S |= 1u << p;
        FSeg g;
        memset(&g, 0, sizeof g);
        int npos = 0;
        for (int p = 0; p < k; ++p)
            if (S >> p & 1) g.pos[npos++] = p;
        for (int m = 0; m < (1 << RB); ++m) {
            uint32_t o = 0;
            for (int i = 0; i < RB; ++i)
                if (m >> i & 1) o |= 1u << g.pos[i];
            g.off[m] = swz_e(o, swz_bits) * (swz_bits == 5 ? 8u : 16u);   // bytes
        }
        g.op_off = (int)rops.size();
        g.nops = 0;
        for (int q : seg) g.nops += to_rops(ops[q], S, RB, rops);
        fold_permutations(g, rops, RB);
        segs.push_back(g);
    }
}

// amplitudes per thread in a segment: 2^5 (complex64) or 2^4 (complex128);
// SV_FUSED_RB (3..5, complex128 at most 4) overrides
static int reg_bits_for(sv_dtype dt, int k) {
    int rb = dt == SV_C128 ? 4 : 5;
    if (const char *e = getenv("SV_FUSED_RB")) {
        const int v = atoi(e);
        if (v >= 3 && v <= (dt == SV_C128 ? 4 : 5)) rb = v;
    }
    return rb < k ? rb : k;
}

// persistent fused passes (the blocks the device holds at once walk the
// tiles); SV_FUSED_PERSIST=0 launches one block per tile
static int fused_persist_env() {
    static int v = -1;
    if (v < 0) {
        const char *e = getenv("SV_FUSED_PERSIST");
        v = (e && atoi(e) == 0) ? 0 : 1;
    }
    return v;
}

template <typename R, int RB, int NT = FUSE_BLOCK>
static void launch_fused(uint64_t tiles, size_t lds, hipStream_t st, cvec<R> *psi, const FPass *dp, int i,
                         const FSeg *ds, const ROp *dops) {
    dim3 grid = tile_grid(tiles);
    if (fused_persist_env()) {
        int dev = 0, cus = 0, per = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, (const void *)k_fused<R, RB, NT>, NT, lds);
        (void)hipGetLastError();
        const uint64_t slots = (uint64_t)(cus > 0 ? cus : 1) * (uint64_t)(per > 0 ? per : 1);
        if (slots < tiles) grid = dim3((unsigned)slots);
    }
    hipLaunchKernelGGL((k_fused<R, RB, NT>), grid, dim3(NT), lds, st, psi, dp, i, ds, dops, tiles);
}

// rb_req: amplitudes per thread in a segment as 2^rb_req (the fusion tuner's
// choice), 0 for the default of reg_bits_for
template <typename R>
static sv_status launch_passes(sv_state s, std::vector<HostPass> &passes, int rb_req = 0) {
    if (passes.empty()) return SV_OK;
    lds_limit_bytes();
    if (!g_fused_lds_at_0) return fail(SV_EDEVICE, "the fused-pass kernels carry static LDS; their tile addressing needs none");
    int RB = reg_bits_for(s->dt, passes[0].hdr.t.k);
    if (rb_req > 0) {
        if (rb_req < 3 || rb_req > (sizeof(R) == 4 ? 5 : 4)) return fail(SV_EINVAL, "%d register bits per segment line", rb_req);
        RB = std::min(rb_req, passes[0].hdr.t.k);
    }
    if (RB < 3) return fail(SV_EUNSUPPORTED, "state too small for fused passes");
    std::vector<FSeg> segs;
    std::vector<ROp> rops;
    for (auto &p : passes) {
        if (p.hdr.t.k < RB) return fail(SV_EDEVICE, "pass with %d local qubits (< %d)", p.hdr.t.k, RB);
        p.hdr.seg_off = (int)segs.size();
        segment_pass(p, RB, sizeof(R) == 4 ? 5 : 4, segs, rops);
        p.hdr.nseg = (int)segs.size() - p.hdr.seg_off;
    }
    const size_t hbytes = passes.size() * sizeof(FPass);
    const size_t sbytes = std::max<size_t>(segs.size(), 1) * sizeof(FSeg);
    const size_t obytes = std::max<size_t>(rops.size(), 1) * sizeof(ROp);
    const size_t soff = (hbytes + 255) & ~(size_t)255, ooff = (soff + sbytes + 255) & ~(size_t)255;
    std::vector<unsigned char> blob(ooff + obytes, 0);
    for (size_t i = 0; i < passes.size(); ++i) memcpy(blob.data() + i * sizeof(FPass), &passes[i].hdr, sizeof(FPass));
    memcpy(blob.data() + soff, segs.data(), segs.size() * sizeof(FSeg));
    memcpy(blob.data() + ooff, rops.data(), rops.size() * sizeof(ROp));
    void *dev = nullptr;
    SV_HIP(hipMallocAsync(&dev, blob.size(), s->stream));
    sv_status st = upload_plan(s, dev, blob.data(), blob.size());
    if (st != SV_OK) {
        hipFreeAsync(dev, s->stream);
        return st;
    }
    const FPass *dp = (const FPass *)dev;
    const FSeg *ds = (const FSeg *)((unsigned char *)dev + soff);
    const ROp *dops = (const ROp *)((unsigned char *)dev + ooff);
    for (size_t i = 0; i < passes.size(); ++i) {
        const FPass &h = passes[i].hdr;
        const uint64_t tiles = dim_of(s->n - h.t.k);
        const size_t lds = ((size_t)1 << h.t.k) * sizeof(cvec<R>);
        TraceScope _ts(s->stream, "fused_pass", 2.0 * (double)dim_of(s->n) * sizeof(cvec<R>), 0.0);
        cvec<R> *psi = (cvec<R> *)s->data;
        // complex64 lines of 16 amplitudes on tiles of 2^13 or more: 512
        // threads, so that each has one line per segment and two workgroups
        // of a 64 KiB tile keep four waves on every SIMD
        if (RB == 5 && sizeof(R) == 4) launch_fused<float, 5>(tiles, lds, s->stream, (cvec<float> *)psi, dp, (int)i, ds, dops);
        else if (RB >= 4 && sizeof(R) == 4 && (1u << (h.t.k - 4)) >= 512u)
            launch_fused<float, 4, 512>(tiles, lds, s->stream, (cvec<float> *)psi, dp, (int)i, ds, dops);
        else if (RB >= 4) launch_fused<R, 4>(tiles, lds, s->stream, psi, dp, (int)i, ds, dops);
        else launch_fused<R, 3>(tiles, lds, s->stream, psi, dp, (int)i, ds, dops);
    }
    hipError_t e = hipGetLastError();
    hipFreeAsync(dev, s->stream);
    if (e != hipSuccess) return hip_fail(e, "k_fused launch");
    return SV_OK;
}

sv_status run_hadamards(sv_state s, int lo, int m, uint64_t fix_mask, uint64_t fix_val) {
    // a layer of Hadamards restricted to (i & fix_mask) == fix_val, as fused passes
    std::vector<PGate> gs;
    const double h = 0.70710678118654752440;
    for (int j = 0; j < m; ++j) {
        PGate p;
        memset(&p, 0, sizeof p);
        p.kind = 0;
        p.t0 = lo + j;
        p.t1 = -1;
        p.cmask = fix_mask;
        p.cval = fix_val;
        p.qubits = (1ull << (lo + j)) | fix_mask;
        p.need = 1ull << (lo + j);
        const double u[8] = {h, 0, h, 0, h, 0, -h, 0};
        memcpy(p.u, u, sizeof u);
        gs.push_back(p);
    }
    const int k = clamp_k(s, 0);
    std::vector<HostPass> passes;
    plan(s->n, k, std::min(low_bits_for(s->dt), k - 2), gs, passes);
    return s->dt == SV_C64 ? launch_passes<float>(s, passes) : launch_passes<double>(s, passes);
}

// rb of a configuration that runs as matrix-core blocks (sv_blocks.hip)
constexpr int RB_BLOCKS = 1;

// the environment names the vector passes' own parameters
static bool fusion_pinned() { return getenv("SV_FUSED_LOWBITS") || getenv("SV_FUSED_RB"); }

// The configuration without tuning, for states below 2^22 amplitudes (larger
// ones: the vector passes).  Times here are launches, latencies and the serial
// run of a tile's gates, and blocks shorten the last.  Fitted to 684 circuits (1
// to 8 layers, 4 to 300 mixed gates, 20 to 150 NOTs and swaps or 8 to 200 phases
// with 1 to 20 dense gates, 8 to 21 qubits, both types), in us: a dense gate
// costs the vector passes 1.0, a NOT or swap 0.6, a phase 0.3; blocks cost 16
// for the build and its gap, 2 per further pass (8 where the vector passes' tile
// holds the whole state) and, where they fill the chip, their arithmetic: 3 per
// block on 21 qubits in complex128, 0.5 in complex64, half of it per qubit less
// (complex128 from 19 qubits on: and at least three gates per block; 600 mixed
// gates on 20 qubits, two and a half per block, 1240 against 1153).
// The rule's pick takes 0.5 % longer than the faster one on average, at most 24 %
// (13 of 55 us); always blocks: 6 % and 75 %.  Examples (blocks,
// vector passes): 8 layers on 14 qubits, complex128, 105 and 304 us; 80 mixed
// gates on 18 qubits, complex64, 123 and 153; one dense gate and 60 phases on 21
// qubits, complex128, 107 and 63; 16 mixed gates on 14 qubits 43 and 36.
// The tile grows with the state, so that small states still spread over many
// compute units: 14 qubits, complex64, k = 8 .. 13: 72 71 54 56 57 71 us; 20
// qubits: 337 243 179 122 119 117 us.
static bool fusion_default(sv_state s, const std::vector<PGate> &pg, BlockPlan &plan) {
    if (s->n >= 22 || fusion_pinned() || !blocks_eligible(s, pg)) return false;
    const bool wide = s->dt == SV_C128;
    double saved = -16.0;
    for (const PGate &g : pg) saved += g.kind == 0 ? 1.0 : g.kind == 3 ? 0.3 : 0.6;
    if (saved <= 0.0) return false;
    plan_blocks(s->n, pg, std::min(wide ? 12 : 13, std::max(std::min(s->n, 10), s->n / 2 + (wide ? 2 : 3))), 3, plan);
    saved -= (s->n <= default_max_local(s->dt) ? 8.0 : 2.0) * ((double)plan.wins.size() - 1.0);
    if (wide && s->n >= 19 && plan.nblocks * 3 > (int)pg.size()) return false;
    return saved > ldexp(wide ? 3.0 : 0.5, s->n - 21) * plan.nblocks;
}

// The fusion autotuner (sv_apply_circuit with max_local = 0, states of 2^22
// amplitudes and more): the candidates are k local qubits in {K-1, K} (K the
// default, bounded by the LDS) times c contiguous low bits in {C-1, C, C+1}
// (C the default, c <= k - 2) times rb register bits per segment line (the
// default and one fewer) times the planner (windows, and windows of the
// earliest gates where those come to at most a fifth more passes), and
// matrix-core blocks where every gate fits one.  Each candidate's first passes
// are timed on a scratch copy of the state (the state itself is not touched):
// the first pass, plus the mean of up to eight others spread over the plan times
// their number; the best few run their whole plan, and the fastest is kept.  A first call costs about 30 runs of the circuit (28
// qubits, complex64: 6 layers 0.31 s, 120 mixed gates 0.33 s; 0.55 and 0.33 with
// a warm-up for every run and the first planner and the vector passes alone).  Cached per dtype,
// size and circuit structure (gate kinds and qubits, not angles) as (k, c, rb),
// with a fourth value 1 for windows of the earliest gates; an entry of (k, c)
// takes the default rb, rb = 1 stands for blocks.  SV_FUSED_LOWBITS pins c and
// skips the tuning.
static uint64_t circuit_signature(const std::vector<PGate> &pg) {
    uint64_t h = 1469598103934665603ull;
    auto mix = [&](uint64_t v) {
        for (int i = 0; i < 8; ++i) {
            h ^= (v >> (8 * i)) & 0xff;
            h *= 1099511628211ull;
        }
    };
    mix(pg.size());
    for (const PGate &g : pg) {
        mix((uint64_t)g.kind);
        mix((uint64_t)(int64_t)g.t0);
        mix((uint64_t)(int64_t)g.t1);
        mix(g.cmask);
        mix(g.cval);
        mix(g.need);
    }
    return h;
}

sv_status fusion_config(sv_state s, const std::vector<PGate> &pg, int &k, int &c, int &rb, bool &early) {
    if (s->n < 22 || getenv("SV_FUSED_LOWBITS")) return SV_OK;
    char sig[32];
    snprintf(sig, sizeof sig, "%016llx", (unsigned long long)circuit_signature(pg));
    const std::string key = std::string("fused/") + (s->dt == SV_C64 ? "c64/" : "c128/") + std::to_string(s->n) + "/" + sig;
    std::vector<int> cached;
    if (tune_lookup(key, cached) && cached.size() >= 2 && cached.size() <= 4) {
        k = cached[0];
        c = cached[1];
        rb = cached.size() >= 3 ? cached[2] : 0;
        early = cached.size() == 4 && cached[3] == 1;
        return SV_OK;
    }
    if (!autotune_enabled()) return SV_OK;
    const size_t bytes = dim_of(s->n) * amp_bytes(s->dt);
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || free_b < bytes + bytes / 16) return SV_OK;
    void *scratch = nullptr;
    if (hipMalloc(&scratch, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return SV_OK;
    }
    sv_state t = new sv_state_s();
    t->n = s->n;
    t->dt = s->dt;
    t->data = scratch;
    t->owned = false;
    t->stream = s->stream;
    t->device = s->device;
    sv_status st = SV_OK;
    if (hipMemcpyAsync(scratch, s->data, bytes, hipMemcpyDeviceToDevice, s->stream) != hipSuccess)
        st = fail(SV_EDEVICE, "scratch copy for the fusion tuner");
    // Candidates: tile depth k, contiguous low bits c and register bits per
    // segment line rb.  Fewer register bits mean more segments but far fewer
    // registers, so a smaller tile can run three or more workgroups per CU.
    // Circuits of few gates per qubit come to as many passes, or nearly, with
    // windows of the earliest gates, and those may run a little faster (25
    // qubits, complex64: 106 mixed gates 1217 us in 10 passes against 1249 in 9,
    // 77 gates 922 against 942, 7 passes each; 120 gates 1285 in 9 against 1233
    // in 7; 28 qubits, complex128, 120 gates: 24.2 against 24.8 ms, with another
    // c): where they are at most a fifth more they are candidates too.
    // A plan's time is estimated from its first pass (which holds the most
    // ops) plus a sample of the others scaled to their number.  The runs are
    // queued one behind the other, so that the host plans the next while they
    // run; below 27 qubits, where a run may be shorter than its planning, an
    // untimed one goes ahead of each.
    const int K = k, C = c, RB0 = s->dt == SV_C64 ? 5 : 4;
    struct Cand {
        float est;
        int k, c, rb;
        bool early;
        float scale1;              // est = ms of span 0 + scale1 x ms of span 1
        size_t ev;                 // first of its three events
    };
    std::vector<Cand> cands;
    std::vector<hipEvent_t> ev;
    auto mark = [&]() -> sv_status {
        hipEvent_t x = nullptr;
        SV_HIP(hipEventCreate(&x));
        ev.push_back(x);
        SV_HIP(hipEventRecord(x, s->stream));
        return SV_OK;
    };
    auto run_plan = [&](std::vector<HostPass> &p, int r) {
        return s->dt == SV_C64 ? launch_passes<float>(t, p, r) : launch_passes<double>(t, p, r);
    };
    // the estimates of the candidates from `from` on
    auto read_times = [&](size_t from) -> sv_status {
        SV_HIP(hipStreamSynchronize(s->stream));
        for (size_t i = from; i < cands.size(); ++i) {
            float ms[2] = {0.f, 0.f};
            for (int q = 0; q < 2; ++q) SV_HIP(hipEventElapsedTime(&ms[q], ev[cands[i].ev + q], ev[cands[i].ev + q + 1]));
            cands[i].est = ms[0] + cands[i].scale1 * ms[1];
        }
        return SV_OK;
    };
    const bool brief = s->n < 27;
    auto tune = [&]() -> sv_status {
        bool warm = false;
        for (int rr = RB0; rr >= RB0 - 1; --rr)
            for (int kk = K - 1; kk <= K; ++kk)
                for (int cc = std::max(0, C - 1); cc <= C + 1; ++cc) {
                    if (kk < 3 || kk < rr || cc > kk - 2) continue;
                    std::vector<HostPass> p[2];
                    for (int e = 0; e < 2; ++e) plan(s->n, kk, cc, pg, p[e], e == 1);
                    for (int e = 0; e < 2; ++e) {
                        const size_t N = p[e].size();
                        if (!N || (e && N * 5 > p[0].size() * 6)) continue;
                        // the first pass, and up to eight of the others spread evenly
                        // over the plan (pass times vary several-fold along it)
                        const size_t S = N - 1 < 8 ? N - 1 : 8;
                        std::vector<HostPass> first(p[e].begin(), p[e].begin() + 1), sample;
                        for (size_t j = 0; j < S; ++j) sample.push_back(p[e][1 + j * (N - 1) / S]);
                        if (brief || !warm) SV_TRY(run_plan(first, rr));
                        warm = true;
                        cands.push_back({0.f, kk, cc, rr, e == 1, S ? (float)(N - 1) / (float)S : 0.f, ev.size()});
                        SV_TRY(mark());
                        SV_TRY(run_plan(first, rr));
                        SV_TRY(mark());
                        if (S) SV_TRY(run_plan(sample, rr));
                        SV_TRY(mark());
                    }
                }
        SV_TRY(read_times(0));
        // matrix-core blocks: the whole circuit, or on large states a prefix of it
        // (at least four gates per qubit), scaled, behind a few gates that load the
        // kernels; a second tile only where the first comes within a third of the
        // vector passes
        if (!fusion_pinned() && blocks_eligible(s, pg)) {
            const size_t part = s->n <= 28 ? pg.size() : std::min(pg.size(), (size_t)(4 * s->n));
            const std::vector<PGate> head(pg.begin(), pg.begin() + (long)part);
            const std::vector<PGate> few(pg.begin(), pg.begin() + (long)std::min<size_t>(part, 8));
            float vec = 1e30f;
            for (const Cand &q : cands) vec = std::min(vec, q.est);
            for (int cc = s->dt == SV_C64 ? 3 : 2, e = cc + 1; cc <= e && blocks_eligible(s, head); ++cc) {
                if (brief) SV_TRY(run_blocks(t, head, K, cc));
                else if (cc < e && blocks_eligible(s, few)) SV_TRY(run_blocks(t, few, K, cc));
                cands.push_back({0.f, K, cc, RB_BLOCKS, false, (float)pg.size() / (float)part, ev.size()});
                SV_TRY(mark());
                SV_TRY(mark());
                SV_TRY(run_blocks(t, head, K, cc));
                SV_TRY(mark());
                SV_TRY(read_times(cands.size() - 1));
                if (cands.back().est > 1.33f * vec) break;
            }
        }
        if (cands.empty()) return SV_OK;
        // The samples tell estimates apart to about 2 % (6 % below half a
        // millisecond; to 10 % between the kinds: windows, windows of the earliest
        // gates, blocks): the best few within that run their whole plan, in turn,
        // and the fastest is kept.
        std::sort(cands.begin(), cands.end(), [](const Cand &x, const Cand &y) { return x.est < y.est; });
        const bool tiny = cands[0].est < 0.5f;
        std::vector<size_t> fin;
        for (size_t i = 0; i < cands.size() && cands[i].est <= 1.1f * cands[0].est; ++i) {
            bool seen = false;
            for (size_t j : fin) seen |= (cands[j].rb == RB_BLOCKS) == (cands[i].rb == RB_BLOCKS) && cands[j].early == cands[i].early;
            if (!seen || (fin.size() < (tiny ? 7 : 4) && cands[i].est <= (tiny ? 1.06f : 1.02f) * cands[0].est)) fin.push_back(i);
        }
        size_t best = 0;
        if (fin.size() > 1) {
            std::vector<std::vector<HostPass>> p(fin.size());
            for (size_t i = 0; i < fin.size(); ++i)
                if (cands[fin[i]].rb != RB_BLOCKS) plan(s->n, cands[fin[i]].k, cands[fin[i]].c, pg, p[i], cands[fin[i]].early);
            auto whole = [&](size_t i) -> sv_status {
                const Cand &q = cands[fin[i]];
                return q.rb == RB_BLOCKS ? run_blocks(t, pg, q.k, q.c) : run_plan(p[i], q.rb);
            };
            const size_t e0 = ev.size(), n = fin.size(), runs = n * (tiny ? 4 : 1);
            if (brief) SV_TRY(whole(n - 1));
            SV_TRY(mark());
            for (size_t j = 0; j < runs; ++j) {
                SV_TRY(whole(j % n));
                SV_TRY(mark());
            }
            SV_HIP(hipStreamSynchronize(s->stream));
            float least = 1e30f;
            for (size_t j = 0; j < runs; ++j) {
                float m = 0.f;
                SV_HIP(hipEventElapsedTime(&m, ev[e0 + j], ev[e0 + j + 1]));
                if (m < least) {
                    least = m;
                    best = fin[j % n];
                }
            }
        }
        k = cands[best].k;
        c = cands[best].c;
        rb = cands[best].rb;
        early = cands[best].early;
        return SV_OK;
    };
    if (st == SV_OK) st = tune();
    hipStreamSynchronize(s->stream);
    for (hipEvent_t x : ev) (void)hipEventDestroy(x);
    sv_free(t);
    hipFree(scratch);
    if (st != SV_OK) return st;
    if (early) tune_store(key, {k, c, rb, 1});
    else tune_store(key, {k, c, rb});
    return SV_OK;
}

}  // namespace sv

using namespace sv;

extern "C" {

int sv_plan_passes(int n_qubits, sv_dtype dt, const sv_gate *gates, int n_gates, int max_local) {
    sv_state_s tmp;
    tmp.n = n_qubits;
    tmp.dt = dt;
    tmp.data = (void *)1;
    std::vector<PGate> pg;
    if (to_pgates(&tmp, gates, n_gates, pg) != SV_OK) return -1;
    int k = max_local > 0 ? max_local : default_max_local(dt);
    if (k > n_qubits) k = n_qubits;
    const int c = std::min(low_bits_for(dt), k - 2);
    BlockPlan blocks;
    if (max_local == 0 && fusion_default(&tmp, pg, blocks)) return (int)blocks.wins.size();
    std::vector<HostPass> passes;
    plan(n_qubits, k, c, pg, passes);
    return (int)passes.size();
}

sv_status sv_apply_circuit(sv_state s, const sv_gate *gates, int n_gates, int max_local) {
    clear_error();
    SV_TRY(check_state(s));
    if (n_gates < 0 || (n_gates && !gates)) return fail(SV_EINVAL, "bad gate list");
    if (!n_gates) return SV_OK;
    std::vector<PGate> pg;
    SV_TRY(to_pgates(s, gates, n_gates, pg));
    SV_TRY(refuse_capture(s));
    int k = clamp_k(s, max_local);
    if (k < 3) return fail(SV_EUNSUPPORTED, "state too small for fused passes");
    int c = std::max(0, std::min(low_bits_for(s->dt), k - 2)), rb = 0;
    bool early = false;
    if (max_local == 0) {
        BlockPlan blocks;
        if (fusion_default(s, pg, blocks)) return run_blocks(s, pg, blocks);
        SV_TRY(fusion_config(s, pg, k, c, rb, early));
    }
    if (rb == RB_BLOCKS) return run_blocks(s, pg, k, c);
    std::vector<HostPass> passes;
    plan(s->n, k, c, pg, passes, early);
    return s->dt == SV_C64 ? launch_passes<float>(s, passes, rb) : launch_passes<double>(s, passes, rb);
}

}  // extern "C"
