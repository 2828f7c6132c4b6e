// The gfx950 kernel of one explicit-implicit step (eq. (8)).
//
// Layout.  Inside the library a field is [nz][np] with np = 64 * rpl and each
// line stored lane-major: row i = lane * rpl + reg lives at reg * 64 + lane.
// One wave (64 lanes) owns one radial line; lane k owns the contiguous rows
// k*rpl .. k*rpl+rpl-1, so every load and store of a line is coalesced and
// the r-neighbours across chunk ends come from the adjacent lane.
//
// Step (delta form).  For the line j each row gets coefficients from the old
// field (eq. (13) capacity rows, eq. (18) interface rows, eq. (15) or held
// boundary rows) and the right-hand side is the explicit residual, so the
// unknown is the increment dT = T^ - T:
//   A dT_{i-1} + B dT_i + C dT_{i+1} = Lambda_i[T] + Lambda_j[T] + X.
// The rows are solved in scaled form (same solution): capacity rows times
// eta^2, so the axial faces take the radial law, and interface rows divided
// by the outer layer's law at the node, so they need one ratio law; the
// plan's forward tables (fgw, fge, finfo, flaws) hold that form.
// The tridiagonal system is solved by partition: every lane eliminates its
// chunk down to two unknowns (first and last row), the 128 chunk-end unknowns
// are reduced to one per lane, and parallel cyclic reduction across the wave
// solves those; lanes then back-substitute their chunk.
#pragma once

#include "device_common.h"

namespace cryo {

// Rows per lane from which a scheduling barrier follows every row.
constexpr int ROW_FENCE = 10;

// Couplings that the step's line solves leave out (solve_tail), of the largest
// increment on the line: below the last place that any temperature beside it is
// held to.  FP64: 2^-17 of its rounding.  FP32 pairs: temperatures lie in
// [2^-4, 2^20) K, so no increment exceeds 2^20 K, and the smallest are held to
// 2^-52 K (in the residual).  A pass squares the couplings, so 2^-41, a float's
// rounding and not the pair's, saves a pass at most (1 to 3 % of a step), and
// cost the quiet rows beside a hot layer up to 200 times their last place.
template <typename R>
constexpr R STEP_DROP = sizeof(R) == 8 ? (R)0x1p-70 : (R)0x1p-74;

// A barrier that orders LDS accesses only: loads of the next lines stay in
// flight across it.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Rows r of one plane of a line at a uniform address: f(r, pointer to this
// lane's row), the address kept in scalar registers and renewed where the
// instructions' 4 KiB offset range ends (left alone, the compiler forms a
// vector register per row past it).
template <typename P, int RPL, int NL, class F>
__device__ inline void each_row(P *base, int lg, F f) {
    constexpr int CH = NL * (int)sizeof(P) < 4096 ? 4096 / (NL * (int)sizeof(P)) : 1;
    // (global, said outright: the compiler no longer sees it past the asm)
    typedef __attribute__((address_space(1))) P *GP;
    GP p = (GP)base;
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if (r % CH == 0) {
            p = (GP)base + r * NL;
            asm volatile("" : "+s"(p));
        }
        f(r, p + (r % CH) * NL + lg);
    }
}

// Rows of this lane's chunk that belong to the line (nodes 0..nr-1); the rest is
// padding.  A step leaves padding rows as they are: they have no radial
// coupling, and every line's hold the same value (pad_value), so no axial flux
// either.  That holds for the z-boundary lines too, which is why a held value
// is written to the line's own rows only.  (Formed where it is used, a cold
// path, from the lane's number anew: hoisted out of it the comparisons take a
// register pair per row, and a lane number kept for it a register.)
template <typename R, int RPL>
__device__ inline int own_rows(const StepArgs<R> &a, int wig) {
    unsigned all = ~0u;
    asm volatile("" : "+s"(all));
    const int lane = __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
    return (a.surf_lane - wig * WAVE - lane) * RPL + a.surf_reg + 1;
}

// One step of eq. (8).  A line is spread over G waves (NL = 64 G lanes, each
// lane a chunk of RPL rows); a workgroup of STEP_WAVES waves runs NG =
// STEP_WAVES / G lines side by side.  Two forms: one line per line group
// (step_shared), and blocks of several (step_march).
//
// CUBE: every capacity law has exponent 3 (c(T) by multiplication).
// POLY: polynomial laws (eqs. (23), (24)), interface rows as the quotient
// of two laws, and the optional Joule source (eq. (25)).
// STEPPED: the stepped domain of eq. (9).  Lines above z_full end at the
// terminal's wall, node nr_top - 1 (rows past it are identity rows), the axial
// face between lines z_full and z_full + 1 is closed from that node on, the
// held outer wall belongs to the layered lines, and the surface mean covers
// lines 0..z_full.

// The step with one line per group (lpw 1).
//
// Axial fluxes (eq. (11)): the flux through the face between two lines enters
// the capacity rows of both.  Each group first evaluates its line's face to
// the next one (independent rows: no elimination chain, few registers) and
// puts it into an LDS slot; after a barrier it reads the slot of the group
// before, so a capacity row costs two conductivities (east r-face, axial
// face).  The face below the workgroup's lines is spread over all waves.
//
// Nothing is decoded per row: a capacity row, by far the most common, takes
// its two faces from one law, whose constants stay in registers from row to
// row; interface rows are found from a bit per row and lane, walls and the
// terminal by position.  Any FP32 shape fits 128 registers that way, and FP64
// with the cube or polynomial laws up to 8 rows per lane (general laws up to 7:
// 130 at 8 rows), so that two or more workgroups share a compute unit: one loads
// its lines while another computes.  One line per wave either way, step_march ->
// here: 512 x 2048 FP64 9.2 -> 9.1 us a step, FP32 7.2 -> 6.6, 631 x 1201 FP64
// 10.6 -> 9.8, 1024 x 2050 15.8 -> 15.0, 512 x 8194 FP64 32.1 -> 23.4; against
// step_march with 2 and 4 lines: 512 x 8194 FP32 17.5, 19.5 -> 14.8.  16 FP64
// rows take 184 registers and 110 KB, one workgroup per unit, and step_march's
// blocks win there once there are more lines than waves (pick_lpw).
//
// MULTI (one wave per line): K steps in one launch.  A workgroup owns the
// middle NG - 2 (K - 1) of its lines; the others are its neighbours', stepped
// here too as long as the owned ones need them (a line less on each side per
// step), and a line passes from step to step in registers, to its neighbours
// through an LDS slot.  Groups past either end of the grid hold the z-boundary
// line (and real lines, discarded).  Owned lines' steps are what single steps
// give, bit for bit.
template <typename R, int RPL, int G, bool CUBE, bool POLY, bool STEPPED, bool MULTI>
__device__ inline void step_shared(const StepArgs<R> &a, const int blk, const R *__restrict__ Tin,
                                   R *__restrict__ Tout, const MultiRun<R> &run, double *partial) {
    constexpr bool PAIR = Pair<R>::on;
    constexpr int NPL = PAIR ? 2 : 1;                 // planes per line (pairs: hi, lo)
    constexpr int NL = WAVE * G;                      // lanes per line
    constexpr int NP = RPL * NL;                      // rows per line (a.np)
    constexpr int NG = STEP_WAVES / G;                // lines per round
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double wsum[STEP_WAVES];
    __shared__ R xchg[NG][9 * G];
    const int L = a.L;
    const unsigned lb = (unsigned)step_law_bytes<R>(L, CUBE, POLY);
    // (the full lines' gw, ge follow the laws in the image)
    stage_tables(a.img, lb, a.img + law_bytes<R>(L, POLY), (unsigned)geom_bytes<R>(NP), smem);
    const auto law = staged_laws<R, POLY>(smem, L);
    const R *sgw = (const R *)(smem + lb), *sge = sgw + NP;
    R *flux = (R *)(smem + lb + geom_bytes<R>(NP));
    const int t = threadIdx.x;
    // the wave index is uniform: line indices and bases live in scalar registers
    const int lane = t & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(t / WAVE);
    const int grp = wv / G, wig = wv % G, lg = wig * WAVE + lane;
    const LaneWord word = ((const LaneWord *)(a.img + a.lanes))[lg];
    constexpr size_t LS = (size_t)NP * NPL;               // line stride
    constexpr size_t LO = PAIR ? (size_t)NP : 0;          // offset of the low plane
    const int K = MULTI ? run.K : 1;
    const int jf = 1 + blk * (NG - 2 * (K - 1)) - (K - 1);   // the workgroup's first line
    const int jr = jf + grp;                              // the group's, or past either end
    const bool active = jr >= 1 && jr < a.nz - 1 && grp >= K - 1 && grp <= NG - K;
    // (past the end: on a real line, discarded)
    const int j = MULTI ? min(max(jr, 0), a.nz - 1) : min(jr, a.nz - 2);
    R *xch = xchg[grp];
    // neighbour rows across the chunk ends (the row itself at the line ends)
    const int qW = lg > 0 ? (RPL - 1) * NL + lg - 1 : 0;
    const int qE = lg < NL - 1 ? lg + 1 : (RPL - 1) * NL + lg;
    // the terminal's lines: this lane's rows from the wall on
    const int nin = STEPPED ? min(max(a.nr_top - 1 - lg * RPL, 0), RPL) : RPL;
    const uint32_t past = STEPPED ? ~((1u << nin) - 1u) : 0u;
    // the group's slot, after the one of the group before (slot 0: the face
    // below the workgroup's lines)
    R *own = flux + (grp + 1) * NP + lg;
    const R *before = own - NP;
    auto face = [&](const auto &S, R Ta, R La, R Tb, R Lb) {   // flux into a from b
#pragma clang fp contract(off)
        return law.at(S, Ta + Tb) * dif<R>(Tb, Lb, Ta, La);
    };
    unsigned off = 0;                                     // see LawLds::off_range
    double sv = 0.0;
    R Tc[RPL], Lc[RPL], Tn[RPL], Ln[RPL];
    R TwF, TeL, LwF = 0, LeL = 0;
    auto load_line = [&](int j, R (&T_)[RPL], R (&L_)[RPL]) {
        const R *b = Tin + (size_t)j * LS;
        each_row<const R, RPL, NL>(b, lg, [&](int r, auto *p) { T_[r] = *p; });
        if constexpr (PAIR) {
            each_row<const R, RPL, NL>(b + LO, lg, [&](int r, auto *p) { L_[r] = *p; });
        } else {
#pragma unroll
            for (int r = 0; r < RPL; ++r) L_[r] = (R)0;
        }
    };
    // a stepped domain's closed face (between lines z_full and z_full + 1)
    auto open_face = [&](int lower, uint32_t bits, int r, R F) {
        if constexpr (STEPPED)
            if (lower == a.z_full && ((bits >> r) & 1)) return (R)0;
        return F;
    };
    // (before the lines' loads: waiting for both at once cost 3 to 5 % of a
    // step, the lines being slower to arrive than the tables)
    stage_wait();
    load_line(j, Tc, Lc);
    load_line(MULTI ? min(j + 1, a.nz - 1) : j + 1, Tn, Ln);
    {
        const R *b = Tin + (size_t)j * LS;
        TwF = b[qW];
        TeL = b[qE];
        if constexpr (PAIR) {
            LwF = b[LO + qW];
            LeL = b[LO + qE];
        }
    }
    // the face below the workgroup's lines: its rows dealt to the groups
    constexpr int NF = (RPL + NG - 1) / NG;
    R Ta[NF], La[NF], Tb[NF], Lb[NF];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
        const R *b = Tin + (size_t)(MULTI ? max(jf - 1, 0) : jf - 1) * LS +
                     min(grp + k * NG, RPL - 1) * NL + lg;
        Ta[k] = b[0];
        La[k] = PAIR ? b[LO] : (R)0;
        Tb[k] = b[LS];
        Lb[k] = PAIR ? b[LS + LO] : (R)0;
    }
    R *pass = flux + (NG + 1) * NP;                       // MULTI: a slot per line
    for (int s = 0; s < K; ++s) {
        const R X = run.X[s];
        // an input value is looked at once, by the group that owns its line
        const bool watch = !MULTI || active || (s == 0 && (jr == 0 || jr == a.nz - 1));
        if (MULTI && !PAIR && s == 1) {
            if (a.held[2]) off = max(off, law.off_range(a.val[2]));
            if (a.held[3]) off = max(off, law.off_range(a.val[3]));
        }
        if (MULTI && s > 0) {
            // the line after, and the chunk ends; z-boundary lines follow the
            // line next to them (insulated) or are held
            const R *mine = pass + grp * NPL * NP, *next = mine + (grp + 1 < NG ? NPL * NP : 0);
            const bool top = jr == a.nz - 2;
            const R *src = top ? mine : next;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                Tn[r] = src[r * NL + lg];
                Ln[r] = PAIR ? src[NP + r * NL + lg] : (R)0;
            }
            // (a held value goes to the line's own rows, as below)
            if (top && a.held[3]) {
                const int n = own_rows<R, RPL>(a, wig);
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    Tn[r] = r < n ? a.val[3] : Tn[r];
                    Ln[r] = r < n ? (R)0 : Ln[r];
                }
            }
            if (jr == 0) {
                const int n = a.held[2] ? own_rows<R, RPL>(a, wig) : 0;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    Tc[r] = r < n ? a.val[2] : Tn[r];
                    Lc[r] = r < n ? (R)0 : Ln[r];
                }
            }
            TwF = mine[qW];
            TeL = mine[qE];
            if constexpr (PAIR) {
                LwF = mine[NP + qW];
                LeL = mine[NP + qE];
            }
        }
        // flux into the line from the next one
        R Fr[RPL];
        {
            auto S = law.set((int)word.law);
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                if ((a.m.iface >> r) & 1)
                    if ((word.iface >> r) & 1) law.next(S);
                // every face mean lies between two nodes: one range check per node
                if (!PAIR && watch) off = max(off, law.off_range(Tc[r]));
                Fr[r] = open_face(j, past, r, face(S, Tc[r], Lc[r], Tn[r], Ln[r]));
                asm volatile("" : "+v"(Fr[r]));              // evaluated here
                own[r * NL] = Fr[r];
                if (r & 1) __builtin_amdgcn_sched_barrier(0);   // register pressure
            }
        }
        if (s == 0) {
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                const int r = grp + k * NG;
                if (r >= RPL) break;
                const auto S = law.set((int)word.law + __popc(word.iface & ((2u << r) - 1u)));
                if constexpr (!PAIR && !MULTI) off = max(off, law.off_range(Ta[k]));
                flux[r * NL + lg] = open_face(jf - 1, past, r, face(S, Ta[k], La[k], Tb[k], Lb[k]));
            }
        }
        if (!PAIR && !MULTI && j + 1 == a.nz - 1) {
#pragma unroll
            for (int r = 0; r < RPL; ++r) off = max(off, law.off_range(Tn[r]));
        }
        lds_barrier();
        const size_t base = (size_t)j * LS;
        const bool up = STEPPED && j > a.z_full;
        const uint32_t wif = word.iface, wheat = up ? word.heat & ~past : word.heat;
        // The rows and the forward elimination of each lane's chunk.
        R a0 = 0, b0 = 1, c0 = 0, d0 = 0;
        R al[RPL], ga[RPL], de[RPL];
        {
            // the outer wall's row (uniform; a terminal line has its own)
            const int hrow = __builtin_amdgcn_readfirstlane(up ? -1 : a.surf_reg);
            const uint32_t heat = X != (R)0 ? a.m.heat : 0u;
            auto S = law.set((int)word.law);
            // west face of the chunk's first row: east face of the previous row
            R lamW = law.at(S, TwF + Tc[0]);
            R dW = dif<R>(TwF, LwF, Tc[0], Lc[0]);
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
#pragma clang fp contract(off)                    // both forms round alike
                const int q = r * NL + lg;
                const R gw = sgw[q], ge = sge[q];
                const R Fb = before[r * NL];         // (into the line before, from this one)
                const R T = Tc[r], Tl = Lc[r];
                const R Te = (r < RPL - 1) ? Tc[r + 1] : TeL;
                const R Le = (r < RPL - 1) ? Lc[r + 1] : LeL;
                // interface rows (eq. (18)): west coefficient the ratio of the
                // inner to the outer layer's law at the node (the row divided
                // by the outer law), east one h_i; no other terms
                const bool some = (a.m.iface >> r) & 1;            // uniform
                const bool ifc = some && ((wif >> r) & 1);
                R v = (R)1;
                if (some)
                    if (ifc) {
                        v = law.ratio(S, T + T);
                        law.next(S);
                    }
                // laws are evaluated from the sum of the two values they average
                const R lamE = law.at(S, T + Te);
                R rc = law.template cap<CUBE>(S, T);
                const R dE = dif<R>(Te, Le, T, Tl);
                R fw = gw * lamW, fe = ge * lamE, ax = Fr[r] - Fb;
                if (some)
                    if (ifc) {
                        fw = gw * v;
                        fe = ge;
                        rc = ax = (R)0;
                    }
                // walls: unit rows with dT = value - T where held
                if (r == 0 && lg == 0) {
                    fe = ge;
                    rc = a.held[0] ? (R)1 : (R)0;
                    ax = a.held[0] ? dif<R>(a.val[0], (R)0, T, Tl) : (R)0;
                }
                if (r == hrow) {
                    asm volatile("" ::: "memory");                  // keeps the branch
                    if (lg == a.surf_lane) {
                        fw = gw;
                        rc = a.held[1] ? (R)1 : (R)0;
                        ax = a.held[1] ? dif<R>(a.val[1], (R)0, T, Tl) : (R)0;
                    }
                }
                if constexpr (STEPPED)
                    if (up)
                        if ((past >> r) & 1) {                     // the terminal's wall, and past it
                            const bool wall = lg * RPL + r == a.nr_top - 1;
                            fw = wall ? (R)1 : (R)0;
                            rc = wall ? (R)0 : (R)1;
                            fe = ax = (R)0;
                        }
                R dd = fma(fe, dE, fw * dW) + ax;
                if ((heat >> r) & 1) {                             // heater rows
                    const R h = (R)((wheat >> r) & 1);
                    if constexpr (POLY) dd = fma(h, a.joule ? X * rsqrt(T) : X, dd);   // eq. (25)
                    else dd = fma(h, X, dd);
                }
                lamW = lamE;
                dW = -dE;
                const R aa = -fw, bb = fw + fe + rc, cc = -fe;
                if (r == 0) {
                    a0 = aa;
                    b0 = bb;
                    c0 = cc;
                    d0 = dd;
                } else {
                    elim_row<R, RPL>(r, aa, bb, cc, dd, al, ga, de);
                    // eliminate here, not where the results are first used
                    // (the solve): sinking it would keep every row's
                    // coefficients live
                    asm volatile("" : "+v"(al[r]), "+v"(ga[r]), "+v"(de[r]));
                }
                // keep the scheduler from hoisting every row's law evaluations
                // at once (register pressure); rows still overlap pairwise
                if (RPL >= ROW_FENCE || (r & 1)) __builtin_amdgcn_sched_barrier(0);
            }
        }
        R x[RPL];
        // the line solve is the step's longest dependent chain (the cyclic
        // reduction's exchanges): a wave inside it issues before a wave still
        // in its rows, whose independent work fills the gaps (measured: 1 %
        // on the 1024 x 4096 FP64 step, results bit for bit the same)
        __builtin_amdgcn_s_setprio(2);
        solve_tail<R, RPL, G>(a0, b0, c0, d0, al, ga, de, x, lane, wig, xch, STEP_DROP<R>);
        __builtin_amdgcn_s_setprio(0);
        // new state: T + dT (pairs: error-free sum, then renormalise)
        R Hn[RPL], Lnw[RPL];
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            if constexpr (PAIR) {
                const R xr = x[r], h = Tc[r];
                const R s = h + xr;
                const R bp = s - h;
                const R err = (h - (s - bp)) + (xr - bp);
                const R lo = Lc[r] + err;
                const R h2 = s + lo;
                Hn[r] = h2;
                Lnw[r] = lo - (h2 - s);
            } else {
                Hn[r] = Tc[r] + x[r];
                Lnw[r] = (R)0;
            }
        }
        if (active && s == K - 1) {
            each_row<R, RPL, NL>(Tout + base, lg, [&](int r, auto *p) { *p = Hn[r]; });
            if constexpr (PAIR)
                each_row<R, RPL, NL>(Tout + base + LO, lg, [&](int r, auto *p) { *p = Lnw[r]; });
            // z-boundary lines: copied (insulated) or held, after the solve
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const bool mine = side == 0 ? j == 1 : j == a.nz - 2;
                if (!mine) continue;
                // (held: the line's own rows, see own_rows)
                const int n = a.held[2 + side] ? own_rows<R, RPL>(a, wig) : 0;
                // formed here (cold path), not hoisted out of the line loop
                size_t ob = side == 0 ? (size_t)0 : (size_t)(a.nz - 1) * LS;
                asm volatile("" : "+v"(ob));
                R *o = Tout + ob;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    o[r * NL + lg] = r < n ? a.val[2 + side] : Hn[r];
                    if constexpr (PAIR) o[LO + r * NL + lg] = r < n ? (R)0 : Lnw[r];
                }
            }
        }
        if (partial && active && lg == a.surf_lane) {
            // the surface row's register is uniform: one scalar test per
            // register, and only the matching register's value is read
            int sreg = __builtin_amdgcn_readfirstlane(a.surf_reg);
            asm volatile("" : "+s"(sreg));               // cold path: no hoisting
            double v = 0.0;
#pragma unroll
            for (int r = 0; r < RPL; ++r)
                if (r == sreg) {
                    asm volatile("" ::: "memory");       // keeps the branch
                    v = (double)Hn[r] + (double)Lnw[r];
                }
            if constexpr (STEPPED) {                    // lines 0..z_full
                sv += j < a.z_full ? a.wz_mid * v : j == a.z_full ? a.wz_end * v : 0.0;
                if (j == 1) sv += a.wz_end * (a.held[2] ? (double)a.val[2] : v);
            } else {
                sv += a.wz_mid * v;
                if (j == 1) sv += a.wz_end * (a.held[2] ? (double)a.val[2] : v);
                if (j == a.nz - 2) sv += a.wz_end * (a.held[3] ? (double)a.val[3] : v);
            }
            if (a.surf_cols > 0) {           // a value per line
                partial[(size_t)s * a.surf_cols + j - 1] = sv;
                sv = 0.0;
            }
        }
        if (MULTI && s + 1 < K) {
            R *mine = pass + grp * NPL * NP;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                Tc[r] = Hn[r];
                Lc[r] = Lnw[r];
                mine[r * NL + lg] = Hn[r];
                if constexpr (PAIR) mine[NP + r * NL + lg] = Lnw[r];
            }
            lds_barrier();
        }
    }
    if (__any(off >= POW_HN)) {
        if (lane == 0) atomicOr(a.flag, 2);
    }
    if (partial && a.surf_cols == 0) {
        if (lane == (a.surf_lane & (WAVE - 1))) wsum[wv] = sv;
        __syncthreads();
        if (t == 0) {
            double s = 0.0;
            for (int w = 0; w < STEP_WAVES; ++w) s += wsum[w];
            partial[blk] = s;
        }
    }
}

// The step over blocks of lpw lines.  Each line group marches through its
// block (up or down), keeping the flux through the face between the current
// and the next line: the flux into line j from line j+1 is minus the flux into
// line j+1 from line j (eq. (11)), so a capacity row evaluates two
// conductivities per line (east r-face, the face towards the next line)
// instead of three.  Rows are decoded from their words (STEPPED: a terminal
// line has its own row tables).
template <typename R, int RPL, int G, bool CUBE, bool POLY, bool STEPPED>
__device__ inline void step_march(const StepArgs<R> &a, const int blk, const R *__restrict__ Tin,
                                 R *__restrict__ Tout, const R X, double *partial) {
    constexpr bool PAIR = Pair<R>::on;
    constexpr int NPL = PAIR ? 2 : 1;                 // planes per line (pairs: hi, lo)
    constexpr int NL = WAVE * G;                      // lanes per line
    constexpr int NG = STEP_WAVES / G;                // lines per workgroup
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double wsum[STEP_WAVES];
    __shared__ R xchg[NG][9 * G];
    const int L = a.L;
    const size_t tbytes = tables_bytes<R>(L, a.np, POLY, STEPPED);
    stage_tables(a.img, (unsigned)tbytes, nullptr, 0, smem);
    const auto law = staged_laws<R, POLY>(smem, L);
    // per-row tables of the line (shared by every line) after the law tables,
    // with the terminal's (STEPPED)
    const R *sgw = (const R *)(smem + law_bytes<R>(L, POLY));
    const R *sge = sgw + a.np;
    const R *sgw2 = sgw + (STEPPED ? 2 * a.np : 0), *sge2 = sgw2 + a.np;
    const uint32_t *sinf = (const uint32_t *)(smem + info_offset<R>(L, a.np, POLY, STEPPED));
    const uint32_t *sinf2 = sinf + (STEPPED ? a.np : 0);
    const int t = threadIdx.x;
    // the wave index is uniform: line indices and bases live in scalar registers
    const int lane = t & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(t / WAVE);
    const int grp = wv / G, wig = wv % G, lg = wig * WAVE + lane;
    const int j0 = 1 + (blk * NG + grp) * a.lpw;
    const int j1 = min(j0 + a.lpw, a.nz - 1);             // exclusive
    // Line order: even line groups march up, odd ones down, so that the
    // halo line two neighbouring groups share is read by both at about the
    // same time (both at their start or both at their end) and stays in L2.
    // The LDS line ring marches up only.  dir is uniform.
    constexpr bool RING_ = ring_used<R>(RPL);
    const int dir = (!RING_ && ((blk * NG + grp) & 1)) ? -1 : 1;
    // line of iteration it, clamped: active iterations first (it < j1 - j0),
    // then inactive ones on real lines (results discarded)
    auto line_at = [&](int it) {
        const int jr = dir > 0 ? j0 + it : j1 - 1 - it;
        return min(max(jr, 1), a.nz - 2);
    };
    const size_t LS = (size_t)a.np * NPL;                 // line stride
    const size_t LO = PAIR ? (size_t)a.np : 0;            // offset of the low plane
    R *xch = xchg[grp];
    // neighbour rows across the chunk ends (the row itself at the line ends)
    const int qW = lg > 0 ? (RPL - 1) * NL + lg - 1 : 0;
    const int qE = lg < NL - 1 ? lg + 1 : (RPL - 1) * NL + lg;
    double sv = 0.0;
    int bad = 0;
    // Line ring (FP32 pairs, ring_used): two LDS slots per wave hold the wave's
    // part of the next line and of the line after it, loaded straight from
    // memory into LDS (no registers in flight) one iteration ahead.  Slot
    // layout: element (row r, plane p, lane) at (r NPL + p) WAVE + lane.  Other
    // cases read the next line from memory directly.  Groups past the last
    // line march on clamped line indices (real lines, results discarded).
    constexpr int SLOT = RPL * NPL * WAVE;
    constexpr bool RING = ring_used<R>(RPL);
    constexpr int EPL = 16 / (int)sizeof(R);              // elements per lane per load
    constexpr int LPS = WAVE / EPL;                       // lanes per row-plane
    R *ring = (R *)(smem + tbytes) + (size_t)wv * 2 * SLOT;
    auto prefetch = [&](int slot, size_t lbase) {
        if constexpr (!RING) return;
        R *dst = ring + slot * SLOT;
        const int sub = lane / LPS, e0 = EPL * (lane % LPS);
#pragma unroll
        for (int i = 0; i < RPL * NPL / EPL; ++i) {
            const int rp = i * EPL + sub;                 // row-plane of this lane
            const R *src = Tin + lbase + (size_t)(rp % NPL) * LO + (size_t)(rp / NPL) * NL +
                           wig * WAVE + e0;
            __builtin_amdgcn_global_load_lds((const void *)src,
                                             (__attribute__((address_space(3))) void *)(dst + i * EPL * WAVE),
                                             16, 0, 0);
        }
    };
    // carried south-face fluxes: registers, or (FP64, 10+ rows per lane) LDS
    constexpr bool FS_LDS = fs_in_lds<R>(RPL);
    R FSr[FS_LDS ? 1 : RPL];
    R *fsl = (R *)(smem + tbytes) + (size_t)wv * RPL * WAVE + lane;
    auto fs_get = [&](int r) -> R {
        if constexpr (FS_LDS) return fsl[r * WAVE];
        else return FSr[r];
    };
    auto fs_set = [&](int r, R v) {
        if constexpr (FS_LDS) fsl[r * WAVE] = v;
        else FSr[r] = v;
    };
    R Tc[RPL], Lc[RPL];
    R TwF, TeL, LwF = 0, LeL = 0;
    {
        const int jb = line_at(0);
        const size_t bc = (size_t)jb * LS;
        const size_t bp = (size_t)(jb - dir) * LS;       // the line before it
        const uint32_t *tinf = (STEPPED && jb > a.z_full) ? sinf2 : sinf;
        const bool trans = STEPPED && min(jb, jb - dir) == a.z_full;
        // (before the lines' loads: waiting for both at once cost 3 to 5 % of
        // a step, the lines being slower to arrive than the tables)
        stage_wait();
        prefetch(1, bc + LS);
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int q = r * NL + lg;
            Tc[r] = Tin[bc + q];
            Lc[r] = PAIR ? Tin[bc + LO + q] : (R)0;
        }
        TwF = Tin[bc + qW];
        TeL = Tin[bc + qE];
        if constexpr (PAIR) {
            LwF = Tin[bc + LO + qW];
            LeL = Tin[bc + LO + qE];
        }
        // axial flux into the block's first line from the line before it
        // (capacity rows); that line is loaded up front
        R Tpv[RPL], Tplv[RPL];
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            Tpv[r] = Tin[bp + r * NL + lg];
            Tplv[r] = PAIR ? Tin[bp + LO + r * NL + lg] : (R)0;
        }
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int q = r * NL + lg;
            const R Tp = Tpv[r], Tpl = Tplv[r];
            const uint32_t inf_r = tinf[q];
            const bool cap = (inf_r & 7) == K_CAP;
            const int l2 = (inf_r >> 12) & 63;
            if constexpr (!PAIR) bad |= !law.in_range(Tp);
            const R lamS = law.lawm(cap ? l2 : law_zero(L), Tc[r] + Tp);
            R Fs = lamS * dif<R>(Tp, Tpl, Tc[r], Lc[r]);
            if constexpr (STEPPED)                          // the step face
                if (trans && (sinf2[q] & 7) != K_CAP) Fs = (R)0;
            fs_set(r, Fs);
            if (r & 1) __builtin_amdgcn_sched_barrier(0);      // register pressure
        }
        // the next line's slot must have landed before the first row reads it
        if constexpr (RING) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    // the first rows of the line above the current one, loaded one line ahead
    constexpr int PF = 2;
    R TnQ[PF], LnQ[PF];
    if constexpr (!RING) {
        const size_t bq = (size_t)(line_at(0) + dir) * LS;
#pragma unroll
        for (int r = 0; r < PF && r < RPL; ++r) {
            TnQ[r] = Tin[bq + r * NL + lg];
            LnQ[r] = PAIR ? Tin[bq + LO + r * NL + lg] : (R)0;
        }
    }
    for (int it = 0; it < a.lpw; ++it) {
        const bool active = it < j1 - j0;
        const int j = line_at(it);
        const size_t base = (size_t)j * LS;
        const size_t bo = (size_t)(j + dir) * LS;        // the other line: the next one
        // stepped domain: this line's tables, and whether its face with the
        // other line is the one at the step
        const bool up = STEPPED && j > a.z_full;
        const bool trans = STEPPED && min(j, j + dir) == a.z_full;
        const R *tgw = up ? sgw2 : sgw, *tge = up ? sge2 : sge;
        const uint32_t *tinf = up ? sinf2 : sinf;
        const R *sn = ring + ((it + 1) & 1) * SLOT;      // line j+1
        // the other slot (line j, already read into registers) takes line j+2;
        // its reads must have completed before the load overwrites it
        if constexpr (RING) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            prefetch(it & 1, (size_t)min(j + 2, a.nz - 1) * LS);
        }
        R TwP, TeP, LwP = 0, LeP = 0;                      // next line's chunk-end neighbours
        {
            const size_t bn = (size_t)line_at(it + 1) * LS;
            TwP = Tin[bn + qW];
            TeP = Tin[bn + qE];
            if constexpr (PAIR) {
                LwP = Tin[bn + LO + qW];
                LeP = Tin[bn + LO + qE];
            }
        }
        // west face of the chunk's first row: east face of the previous row
        R lamW = law.lawm((tinf[qW] >> 6) & 63, TwF + Tc[0]);
        R a0 = 0, b0 = 1, c0 = 0, d0 = 0;
        R al[RPL], ga[RPL], de[RPL];
        // without the ring: the next line's values come from memory two rows
        // ahead of their use (software pipelined across the rows' regions);
        // the first two were loaded before the previous line's solve
        R TnP[RPL], LnP[RPL];
        if constexpr (!RING) {
#pragma unroll
            for (int r = 0; r < PF && r < RPL; ++r) {
                TnP[r] = TnQ[r];
                LnP[r] = LnQ[r];
            }
        }
        // the held outer wall's row (uniform; -1 for none): its test below is
        // a scalar branch per row, not a select kept in registers for every row
        int hrow = (a.held[1] && !up) ? a.surf_reg : -1;
        hrow = __builtin_amdgcn_readfirstlane(hrow);
        const bool hlane = lg == a.surf_lane;
        // the rows' info words, one row ahead (they head each row's chain of
        // table lookups)
        uint32_t infn = tinf[lg];
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
#pragma clang fp contract(off)                    // both forms round alike
            const int q = r * NL + lg;
            const uint32_t inf_r = infn;
            if (r + 1 < RPL) infn = tinf[q + NL];
            if constexpr (!RING) {
                if (r + PF < RPL) {
                    TnP[r + PF] = Tin[bo + q + PF * NL];
                    LnP[r + PF] = PAIR ? Tin[bo + LO + q + PF * NL] : (R)0;
                }
            }
            const uint32_t kind = inf_r & 7;
            const bool cap = kind == K_CAP;
            const R T = Tc[r], Tl = Lc[r];
            R Tnr, Lnr = 0;
            if constexpr (RING) {
                Tnr = sn[r * NPL * WAVE + lane];
                if constexpr (PAIR) Lnr = sn[(r * NPL + 1) * WAVE + lane];
            } else {
                Tnr = TnP[r];
                if constexpr (PAIR) Lnr = LnP[r];
            }
            // the carried flux into this line from the previous line, read
            // unconditionally at the row's start (a read under the capacity
            // test becomes a branch that waits for it at once)
            const R Fc = fs_get(r);
            const R Tw = (r > 0) ? Tc[r - 1] : TwF;
            const R Te = (r < RPL - 1) ? Tc[r + 1] : TeL;
            const R Lw = (r > 0) ? Lc[r - 1] : LwF;
            const R Le = (r < RPL - 1) ? Lc[r + 1] : LeL;
            const int le = (inf_r >> 6) & 63, l2 = (inf_r >> 12) & 63;
            const int lc = (inf_r >> 24) & 63;
            // every face mean lies between two nodes: one range check per node
            if constexpr (!PAIR) bad |= !law.in_range(T);
            // laws are evaluated from the sum of the two values they average
            const R lamE = law.lawm(le, T + Te);
            // slot 2: the north axial face of a capacity row (the row's radial
            // law: capacity rows are scaled by eta^2), the ratio of the inner
            // to the outer layer's law at an interface node (its row divided
            // by the outer law), or unit (boundary, a terminal line past its
            // wall)
            R lam2 = law.lawm(l2, T + (cap ? Tnr : T));
            if constexpr (POLY) lam2 = lam2 / law.lawm((inf_r >> 18) & 63, T + T);
            R rc;
            if constexpr (CUBE) rc = law.cube(lc, T);
            else rc = law.lawm(lc, T + T);
            const R fw = tgw[q] * (cap ? lamW : lam2);
            const R fe = tge[q] * (cap ? lamE : (R)1);
            // flux into this line from the next one (carried on, negated), and
            // the line's two axial fluxes; not contracted, so that results do
            // not depend on the direction, and equal step_shared's
            R Fo = lam2 * dif<R>(Tnr, Lnr, T, Tl);
            if constexpr (STEPPED)                          // the step face
                if (trans && (sinf2[q] & 7) != K_CAP) Fo = (R)0;
            const R ax = Fo + Fc;
            R dd = fma(fe, dif<R>(Te, Le, T, Tl), fw * dif<R>(Tw, Lw, T, Tl)) + (cap ? ax : (R)0);
            const R h = (R)((inf_r >> 3) & 1);                 // heater capacity rows
            if constexpr (POLY) dd = fma(h, a.joule ? X * rsqrt(T) : X, dd);   // eq. (25)
            else dd = fma(h, X, dd);
            // held walls: rows 0 and nr - 1 are unit rows with dT = value - T
            if (r == 0 && a.held[0]) dd = lg == 0 ? dif<R>(a.val[0], (R)0, T, Tl) : dd;
            if (r == hrow) {
                asm volatile("" ::: "memory");               // keeps the branch
                dd = hlane ? dif<R>(a.val[1], (R)0, T, Tl) : dd;
            }
            fs_set(r, -Fo);
            lamW = lamE;
            const R aa = -fw, bb = fw + fe + rc, cc = -fe;
            if (r == 0) {
                a0 = aa;
                b0 = bb;
                c0 = cc;
                d0 = dd;
            } else {
                elim_row<R, RPL>(r, aa, bb, cc, dd, al, ga, de);
                // eliminate here, not where the results are first used (the
                // solve): sinking it would keep every row's coefficients live
                asm volatile("" : "+v"(al[r]), "+v"(ga[r]), "+v"(de[r]));
            }
            // keep the scheduler from hoisting every row's law evaluations
            // at once (register pressure); rows still overlap pairwise
            if (RPL >= 10 || (r & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!RING) {
            // the next iteration's first rows of its other line (a boundary
            // line only for inactive iterations)
            const size_t bq = (size_t)(line_at(it + 1) + dir) * LS;
#pragma unroll
            for (int r = 0; r < PF && r < RPL; ++r) {
                TnQ[r] = Tin[bq + r * NL + lg];
                LnQ[r] = PAIR ? Tin[bq + LO + r * NL + lg] : (R)0;
            }
        }
        R X[RPL];
        // the line solve is the step's longest dependent chain (the cyclic
        // reduction's exchanges): a wave inside it issues before a wave still
        // in its rows, whose independent work fills the gaps (measured: 1 %
        // on the 1024 x 4096 FP64 step, results bit for bit the same)
        __builtin_amdgcn_s_setprio(2);
        solve_tail<R, RPL, G>(a0, b0, c0, d0, al, ga, de, X, lane, wig, xch, STEP_DROP<R>);
        __builtin_amdgcn_s_setprio(0);
        // the line after next (slot) and the next neighbours have landed
        if constexpr (RING) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (active) {
            // new state: T + dT (pairs: error-free sum, then renormalise)
            R Hn[RPL], Lnw[RPL];
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                if constexpr (PAIR) {
                    const R x = X[r], h = Tc[r];
                    const R s = h + x;
                    const R bp = s - h;
                    const R err = (h - (s - bp)) + (x - bp);
                    const R lo = Lc[r] + err;
                    const R h2 = s + lo;
                    Hn[r] = h2;
                    Lnw[r] = lo - (h2 - s);
                } else {
                    Hn[r] = Tc[r] + X[r];
                    Lnw[r] = (R)0;
                }
                Tout[base + r * NL + lg] = Hn[r];
                if constexpr (PAIR) Tout[base + LO + r * NL + lg] = Lnw[r];
            }
            // z-boundary lines: copied (insulated) or held, after the solve
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const bool mine = side == 0 ? j == 1 : j == a.nz - 2;
                if (!mine) continue;
                // (held: the line's own rows, see own_rows)
                const int n = a.held[2 + side] ? own_rows<R, RPL>(a, wig) : 0;
                // formed here (cold path), not hoisted out of the line loop
                size_t ob = side == 0 ? (size_t)0 : (size_t)(a.nz - 1) * LS;
                asm volatile("" : "+v"(ob));
                R *o = Tout + ob;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    o[r * NL + lg] = r < n ? a.val[2 + side] : Hn[r];
                    if constexpr (PAIR) o[LO + r * NL + lg] = r < n ? (R)0 : Lnw[r];
                }
            }
            if (partial && lg == a.surf_lane) {
                // the surface row's register is uniform: one scalar test per
                // register, and only the matching register's value is read
                int sreg = __builtin_amdgcn_readfirstlane(a.surf_reg);
                asm volatile("" : "+s"(sreg));               // cold path: no hoisting
                double v = 0.0;
#pragma unroll
                for (int r = 0; r < RPL; ++r)
                    if (r == sreg) {
                        asm volatile("" ::: "memory");       // keeps the branch
                        v = (double)Hn[r] + (double)Lnw[r];
                    }
                if constexpr (STEPPED) {                    // lines 0..z_full
                    sv += j < a.z_full ? a.wz_mid * v : j == a.z_full ? a.wz_end * v : 0.0;
                    if (j == 1) sv += a.wz_end * (a.held[2] ? (double)a.val[2] : v);
                } else {
                    sv += a.wz_mid * v;
                    if (j == 1) sv += a.wz_end * (a.held[2] ? (double)a.val[2] : v);
                    if (j == a.nz - 2) sv += a.wz_end * (a.held[3] ? (double)a.val[3] : v);
                }
            }
        }
        // next line: registers from its ring slot, or the values the rows
        // read as their north neighbours (line j + 1; past the last interior
        // line only inactive iterations use them)
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            if constexpr (RING) {
                Tc[r] = sn[r * NPL * WAVE + lane];
                Lc[r] = PAIR ? sn[(r * NPL + 1) * WAVE + lane] : (R)0;
            } else {
                Tc[r] = TnP[r];
                Lc[r] = LnP[r];
            }
        }
        TwF = TwP;
        TeL = TeP;
        LwF = LwP;
        LeL = LeP;
    }
    if (__any(bad)) {
        if (lane == 0) atomicOr(a.flag, 2);
    }
    if (partial) {
        if (lane == (a.surf_lane & (WAVE - 1))) wsum[wv] = sv;
        __syncthreads();
        if (t == 0) {
            double s = 0.0;
            for (int w = 0; w < STEP_WAVES; ++w) s += wsum[w];
            partial[blk] = s;
        }
    }
}

// Workgroups are dealt to the 8 XCDs in turn (workgroup b on XCD b mod 8);
// each XCD gets a contiguous range of line groups, so that the lines shared by
// neighbouring groups meet in the same L2.  A bijection of 0..nb-1.
__device__ inline int xcd_block(int b, int nb) {
    const int x = b & 7, i = b >> 3, per = nb >> 3, rem = nb & 7;
    return x * per + min(x, rem) + i;
}

template <typename R, int RPL, int G, bool CUBE, bool POLY, bool STEPPED, bool SHARED>
__global__ __launch_bounds__(STEP_WAVES *WAVE) void k_step(StepArgs<R> a) {
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    if constexpr (SHARED)
        step_shared<R, RPL, G, CUBE, POLY, STEPPED, false>(a, blk, a.Tin, a.Tout, {1, {a.X}},
                                                           a.partial);
    else
        step_march<R, RPL, G, CUBE, POLY, STEPPED>(a, blk, a.Tin, a.Tout, a.X, a.partial);
}

// K steps in one launch (step_shared's MULTI)
template <typename R, int RPL, bool CUBE, bool POLY, bool STEPPED>
__global__ __launch_bounds__(STEP_WAVES *WAVE) void k_step_multi(StepArgs<R> a, MultiRun<R> run) {
    step_shared<R, RPL, 1, CUBE, POLY, STEPPED, true>(a, xcd_block(blockIdx.x, gridDim.x), a.Tin,
                                                      a.Tout, run, a.partial);
}

// Pulse average over step k (eq. (4)), step units; the host's schedule.
__device__ inline double source_fraction_dev(const Pulse &p, int64_t k) {
    if (!(p.W > 0)) return 0.0;
    const double lo = (double)k, hi = lo + 1.0;
    double s = 0.0;
    int64_t n = (int64_t)floor((lo - p.b0 - p.W) / p.P);
    if (n < 0) n = 0;
    for (int guard = 0; guard < 64; ++guard, ++n) {
        const double b = p.b0 + (double)n * p.P;
        if (b >= hi) break;
        const double o = fmin(hi, b + p.W) - fmax(lo, b);
        if (o > 0) s += o;
    }
    return s;
}

// One step of many instances: workgroup -> (instance, workgroup of that
// instance); global step k = *k0 + n; buffers by the parity of n.
template <typename R, int RPL, int G, bool CUBE, bool POLY, bool STEPPED, bool SHARED>
__global__ __launch_bounds__(STEP_WAVES *WAVE) void k_step_batch(const StepArgs<R> *descs,
                                                                 const int2 *wg_map, int64_t n,
                                                                 const int64_t *k0) {
    const int2 m = wg_map[blockIdx.x];
    const StepArgs<R> &a = descs[m.x];
    double X = a.pulse.amplitude * source_fraction_dev(a.pulse, *k0 + n);
    if constexpr (POLY) X *= a.jsq;                 // the Joule source's sqrt(T_J)
    double *part = a.partial ? a.partial + (size_t)(n % SURF_CHUNK) * a.groups : nullptr;
    const R *in = a.buf[n & 1];
    R *out = a.buf[(n + 1) & 1];
    if constexpr (SHARED)
        step_shared<R, RPL, G, CUBE, POLY, STEPPED, false>(a, m.y, in, out, {1, {(R)X}}, part);
    else
        step_march<R, RPL, G, CUBE, POLY, STEPPED>(a, m.y, in, out, (R)X, part);
}

// One launch of the kernel of a plan's shape and options; false if the shape
// is not built.
template <typename R, bool CUBE, bool POLY, bool STEPPED, bool SHARED>
inline bool launch_step_kind(int key, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> &a) {
    switch (key) {
#define STEP_CASE(RP, GW) \
    case RP * 10 + GW: \
        hipLaunchKernelGGL((k_step<R, RP, GW, CUBE, POLY, STEPPED, SHARED>), g, \
                           dim3(STEP_WAVES *WAVE), lds, s, a); \
        return true;
        CRYO_FOR_SHAPES(STEP_CASE)
#undef STEP_CASE
    }
    return false;
}
template <typename R, bool CUBE, bool POLY, bool STEPPED, bool SHARED>
inline bool launch_batch_kind(int key, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> *d,
                              const int2 *map, int64_t n, const int64_t *k0) {
    switch (key) {
#define BATCH_CASE(RP, GW) \
    case RP * 10 + GW: \
        hipLaunchKernelGGL((k_step_batch<R, RP, GW, CUBE, POLY, STEPPED, SHARED>), g, \
                           dim3(STEP_WAVES *WAVE), lds, s, d, map, n, k0); \
        return true;
        CRYO_FOR_SHAPES(BATCH_CASE)
#undef BATCH_CASE
    }
    return false;
}

// The launches of one field type, domain and sharing, each in a source file
// of its own (they compile side by side); `laws` 0: cube capacity, 1: general
// power laws, 2: polynomial.
template <typename R, bool STEPPED, bool SHARED>
struct StepLaunch {
    static bool step(int laws, int key, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> &a);
    static bool batch(int laws, int key, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> *d,
                      const int2 *map, int64_t n, const int64_t *k0);
};
#define CRYO_STEP_LAUNCH(R, STEPPED, SHARED) \
    template <> \
    bool StepLaunch<R, STEPPED, SHARED>::step(int laws, int key, dim3 g, size_t lds, \
                                              hipStream_t s, const StepArgs<R> &a) { \
        return laws == 2 ? launch_step_kind<R, false, true, STEPPED, SHARED>(key, g, lds, s, a) \
             : laws == 1 ? launch_step_kind<R, false, false, STEPPED, SHARED>(key, g, lds, s, a) \
                         : launch_step_kind<R, true, false, STEPPED, SHARED>(key, g, lds, s, a); \
    } \
    template <> \
    bool StepLaunch<R, STEPPED, SHARED>::batch(int laws, int key, dim3 g, size_t lds, \
                                               hipStream_t s, const StepArgs<R> *d, \
                                               const int2 *map, int64_t n, const int64_t *k0) { \
        return laws == 2 ? launch_batch_kind<R, false, true, STEPPED, SHARED>(key, g, lds, s, d, \
                                                                              map, n, k0) \
             : laws == 1 ? launch_batch_kind<R, false, false, STEPPED, SHARED>(key, g, lds, s, d, \
                                                                               map, n, k0) \
                         : launch_batch_kind<R, true, false, STEPPED, SHARED>(key, g, lds, s, d, \
                                                                              map, n, k0); \
    }


// K-step launches, one wave per line
template <typename R, bool CUBE, bool POLY, bool STEPPED>
inline bool launch_multi_kind(int rpl, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> &a,
                              const MultiRun<R> &run) {
    switch (rpl) {
#define MULTI_CASE(RP) \
    case RP: \
        hipLaunchKernelGGL((k_step_multi<R, RP, CUBE, POLY, STEPPED>), g, dim3(STEP_WAVES *WAVE), \
                           lds, s, a, run); \
        return true;
        MULTI_CASE(2) MULTI_CASE(3) MULTI_CASE(4) MULTI_CASE(5) MULTI_CASE(6) MULTI_CASE(7)
        MULTI_CASE(8) MULTI_CASE(10)
#undef MULTI_CASE
    }
    return false;
}
template <typename R, bool STEPPED>
struct MultiLaunch {
    static bool step(int laws, int rpl, dim3 g, size_t lds, hipStream_t s, const StepArgs<R> &a,
                     const MultiRun<R> &run);
};
#define CRYO_MULTI_LAUNCH(R, STEPPED) \
    template <> \
    bool MultiLaunch<R, STEPPED>::step(int laws, int rpl, dim3 g, size_t lds, hipStream_t s, \
                                       const StepArgs<R> &a, const MultiRun<R> &run) { \
        return laws == 2 ? launch_multi_kind<R, false, true, STEPPED>(rpl, g, lds, s, a, run) \
             : laws == 1 ? launch_multi_kind<R, false, false, STEPPED>(rpl, g, lds, s, a, run) \
                         : launch_multi_kind<R, true, false, STEPPED>(rpl, g, lds, s, a, run); \
    }

}  // namespace cryo
