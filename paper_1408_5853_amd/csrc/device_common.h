// Device code shared by the stepping and adjoint kernels: law evaluation
// from LDS tables, compensated FP32 pairs, wave shuffles and the partitioned
// tridiagonal solve.
#pragma once

#include <math.h>
#include <string.h>

#include <type_traits>

#include "internal.h"

namespace cryo {

// reciprocal: hardware estimate (relative error below 5e-8 on gfx950)
// refined by one Newton step (below 3e-15).  The step's solves work in delta
// form, so a pivot off by that much perturbs only the increment, by a
// relative 3e-15; the adjoint's uses (transposed solves, derivative factors)
// carry it into the gradient at the same relative size.
__device__ inline double rcp(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ inline float rcp(float x) {
    float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.0f), r, r);
}

// Law evaluation K[id] * T^e[id] from tables staged in LDS.  A Set holds one
// radial law's constants in a lane's registers, `at` evaluates it at the mean
// of two values given their sum, `next` moves on to the next layer's, `ratio`
// is the quotient of this layer's law and the next one's at s / 2, and `cap`
// the layer's capacity law at T (CUBE: every exponent is 3).
template <typename R>
struct LawLds;

template <>
struct LawLds<double> {
    const double *blk;      // law blocks (POW_BLK doubles per law id)
    int L;
    struct Set {
        const double *B;
        double e, k;         // exponent; the layer's cube multiplier
        double2 c23, c45, c67;
    };
    static __device__ inline Set load(const double *B) {
        Set s;
        s.B = B;
        const double2 ek = *(const double2 *)(B + POW_BE);
        s.e = ek.x;
        s.k = ek.y;
        s.c23 = *(const double2 *)(B + POW_BE + 2);
        s.c45 = *(const double2 *)(B + POW_BE + 4);
        s.c67 = *(const double2 *)(B + POW_BE + 6);
        return s;
    }
    __device__ inline Set set(int id) const { return load(blk + id * POW_BLK); }
    __device__ inline void next(Set &s) const { s = load(s.B + POW_BLK); }
    // T on the table range [2^POW_EMIN, 2^(POW_EMIN+POW_NE)) K: the high
    // words' distance from the lower end, as an unsigned number (NaN and
    // negative values are far above)
    static __device__ inline unsigned off_range(double x) {
        return (unsigned)(__double_as_longlong(x) >> 32) - POW_HLO;
    }
    static __device__ inline bool in_range(double x) { return off_range(x) < POW_HN; }
    __device__ inline double expo(int id) const { return blk[id * POW_BLK + POW_BE]; }
    // the law at x, and at s / 2 (halving only moves the binade); an argument
    // off the table range reads some binade's slot, so callers check the
    // range themselves
    __device__ inline double lawc(int id, double x) const { return pw<1>(set(id), x); }
    __device__ inline double lawm(int id, double s) const { return pw<2>(set(id), s); }
    static __device__ inline double at(const Set &c, double s) { return pw<2>(c, s); }
    template <int SH>
    static __device__ inline double pw(const Set &c, double x) {
#pragma clang fp contract(off)                    // (a value does not depend on its use)
        const double mh = __builtin_amdgcn_frexp_mant(x);          // x = mh 2^xe, mh in [1/2, 1)
        const unsigned hi = (unsigned)(__double_as_longlong(x) >> 32);
        const unsigned jm = __builtin_amdgcn_ubfe(hi, 20 - POW_MBITS, POW_MBITS);
        // the argument's binade is its biased exponent less 1023, the mean's
        // one lower; 1024 is 0 mod NX
        const unsigned xc = SH == 2 ? __builtin_amdgcn_ubfe(hi, 20, 5)
                                    : ((hi >> 20) + 1) & (POW_NX - 1);
        const double2 mm = *(const double2 *)(c.B + 2 * jm);
        const double u = fma(mh, mm.y, -1.0);                   // m / m0 - 1
        // (1 + u)^e, |u| <= 2^-(POW_MBITS+1), by Estrin's scheme (depth 4,
        // against 7 dependent steps for Horner's)
        const double u2 = u * u, u4 = u2 * u2;
        const double p01 = fma(c.e, u, 1.0), p23 = fma(c.c23.y, u, c.c23.x);
        const double p45 = fma(c.c45.y, u, c.c45.x), p67 = fma(c.c67.y, u, c.c67.x);
        const double s = fma(fma(p67, u2, p45), u4, fma(p23, u2, p01));
        return (c.B[POW_BX + xc] * mm.x) * s;
    }
    __device__ inline double ratio(const Set &s, double x) const {
        return at(load(s.B + L * POW_BLK), x);
    }
    template <bool CUBE>
    __device__ inline double cap(const Set &s, double T) const {
#pragma clang fp contract(off)
        if constexpr (CUBE) return s.k * (T * T * T);
        else return at(load(s.B + 2 * L * POW_BLK), T + T);
    }
    // capacity of a row by its capacity law's id (K T^3 + A): a layer's, or the
    // zero and unit laws of other rows
    __device__ inline double cube(int id, double x) const {
        const double2 k = *(const double2 *)(blk + (3 * L + 2) * POW_BLK + 2 * id);
        return fma(k.x, x * x * x, k.y);
    }
    __device__ inline double cubek(int id) const { return blk[(3 * L + 2) * POW_BLK + 2 * id]; }
};

// Polynomial laws (eqs. (23), (24)): sum_k c_k x^k, k <= 4, by Horner's
// rule, from POLY_BLK numbers per law id staged in LDS in place of the power
// tables (c_0 .. c_4, one pad); FP32 holds the coefficients rounded to float.
template <typename R>
struct LawPoly {
    using R2 = std::conditional_t<sizeof(R) == 8, double2, float2>;
    const R *c;
    int L;
    struct Set {
        const R *B;
        R2 k01, k23;
        R k4;
    };
    static __device__ inline Set load(const R *p) {
        return Set{p, *(const R2 *)p, *(const R2 *)(p + 2), p[4]};
    }
    __device__ inline Set set(int id) const { return load(c + POLY_BLK * id); }
    __device__ inline void next(Set &s) const { s = load(s.B + POLY_BLK); }
    static __device__ inline unsigned off_range(R x) { return LawLds<double>::off_range(x); }
    static __device__ inline bool in_range(R x) { return LawLds<double>::in_range(x); }
    static __device__ inline R horner(const Set &s, R x) {
        return fma(fma(fma(fma(s.k4, x, s.k23.y), x, s.k23.x), x, s.k01.y), x, s.k01.x);
    }
    __device__ inline R lawc(int id, R x) const { return horner(set(id), x); }
    __device__ inline R lawm(int id, R s) const { return lawc(id, (R)0.5 * s); }
    static __device__ inline R at(const Set &c, R s) { return horner(c, (R)0.5 * s); }
    __device__ inline R ratio(const Set &s, R x) const {
        return at(s, x) / at(load(s.B + POLY_BLK), x);
    }
    template <bool CUBE>
    __device__ inline R cap(const Set &s, R T) const {
        return horner(load(s.B + 2 * L * POLY_BLK), T);
    }
};

// FP32: 2^(e log2 s + lk); the stepping kernel's tables hold lk = log2 K - e,
// so that s is the sum of the two values whose mean the law is taken at, with
// e and the layer's cube multiplier, one float4 per law.
// The hardware log2 and exp2 instructions serve directly: s is a sum of two
// temperatures (a normal float); only law values below 1e-38, which no law
// here reaches, could differ from the library functions, which add a
// rescaling for subnormal arguments and results around the same instructions
// (six more instructions per law).
template <>
struct LawLds<float> {
    const float4 *t;
    int L;
    struct Set {
        const float4 *B;
        float lk, e, k;
    };
    static __device__ inline Set load(const float4 *B) {
        const float4 v = *B;
        return Set{B, v.x, v.y, v.z};
    }
    __device__ inline Set set(int id) const { return load(t + id); }
    __device__ inline void next(Set &s) const { s = load(s.B + 1); }
    static __device__ inline unsigned off_range(float) { return 0; }
    __device__ inline float lawm(int id, float s) const { return at(set(id), s); }
    __device__ inline float cube(int id, float x) const {
        const float4 v = t[id];
        return fmaf(v.z, x * x * x, v.w);
    }
    static __device__ inline float at(const Set &c, float s) {
        return __builtin_amdgcn_exp2f(fmaf(c.e, __builtin_amdgcn_logf(s), c.lk));
    }
    __device__ inline float ratio(const Set &s, float x) const { return at(load(s.B + L), x); }
    template <bool CUBE>
    __device__ inline float cap(const Set &s, float T) const {
#pragma clang fp contract(off)
        if constexpr (CUBE) return s.k * (T * T * T);
        else return at(load(s.B + 2 * L), T + T);
    }
};

template <typename R>
struct StepArgs {
    const R *Tin;             // single plan: this step's input and output
    R *Tout;
    R *buf[2];                // batch: ping-pong buffers (step n reads buf[n & 1])
    const unsigned char *img; // table image (tables_bytes), staged in LDS
    int L;                    // layers
    int cube;                 // every capacity exponent is 3
    int nz, np;
    int lpw;                  // lines per wave (a contiguous block)
    RowMasks m;               // of a line
    unsigned lanes;           // byte offset of the image's lane words
    R X;                      // amplitude * pulse average of this step
    int held[4];              // r_inner, r_outer, z_low, z_high
    R val[4];
    double *partial;          // nullable: per-workgroup surface partial sums
    int *flag;                // error word: bit 1 = temperature off the law tables
    double wz_end, wz_mid;    // trapezoid weights of the surface mean
    int surf_lane, surf_reg;
    int surf_cols;            // partial sums: one per line (its count), or 0: per workgroup
    int groups;               // workgroups of one step of this instance
    Pulse pulse;              // batch: schedule evaluated on the device
    int joule;                // heater source times X / sqrt(T) (eq. (25)), X holding sqrt(T_J)
    // stepped domain (eq. (9)): lines above z_full take the terminal's row
    // tables (nz - 1 when there is none)
    int z_full, nr_top;
    double jsq;               // sqrt(T_J) with the Joule source, else 1 (batch
                              // and adjoint kernels form their source with it)
};

// The steps of one launch: their sources (amplitude * pulse average).
template <typename R>
struct MultiRun {
    int K;
    R X[MULTI_MAX];
};

constexpr int STEP_WAVES = STEP_WAVES_HOST;

// v of lane (idx4 / 4) mod 64: the permute takes address bits 7:2 as the
// source lane, so idx4 = 4 lane + (256 - 4 s) reads lane - s around the wave
// and the constant folds into the instruction's offset field
__device__ inline float lane_read(float v, int idx4) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(idx4, __builtin_bit_cast(int, v)));
}
__device__ inline double lane_read(double v, int idx4) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_ds_bpermute(idx4, (int)b);
    const int hi = __builtin_amdgcn_ds_bpermute(idx4, (int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
template <typename R>
__device__ inline R shfl_up1(R v, int s, int lane) {
    R u = __shfl_up(v, s, WAVE);
    return lane >= s ? u : (R)0;
}
template <typename R>
__device__ inline R shfl_dn1(R v, int s, int lane) {
    R u = __shfl_down(v, s, WAVE);
    return lane + s < WAVE ? u : (R)0;
}

// Forward elimination of one row r >= 1 of a lane's chunk, with a fill-in
// column on the chunk's first row x_0:  al_r x_0 + x_r + ga_r x_{r+1} = de_r
template <typename R, int RPL>
__device__ inline void elim_row(int r, R aa, R bb, R cc, R dd, R (&al)[RPL], R (&ga)[RPL],
                                R (&de)[RPL]) {
    if (r == 1) {
        const R inv = rcp(bb);
        al[1] = aa * inv;
        ga[1] = cc * inv;
        de[1] = dd * inv;
    } else {
        const R inv = rcp(bb - aa * ga[r - 1]);
        al[r] = -aa * al[r - 1] * inv;
        ga[r] = cc * inv;
        de[r] = (dd - aa * de[r - 1]) * inv;
    }
}

// Rest of the partitioned solve, after every lane has eliminated rows 1..RPL-1
// of its chunk (elim_row).  A line is spread over G waves (64 G lanes, lane
// lg = wig * 64 + lane owns rows lg*RPL .. lg*RPL+RPL-1):
//  1. back-eliminate each chunk onto its ends x_0, x_e;
//  2. eliminate x_0 with the first row, leaving one unknown x_e per lane and a
//     tridiagonal reduced system across the 64 G lanes;
//  3. each wave solves its 64 unknowns by parallel cyclic reduction, with the
//     couplings to the neighbouring waves' unknowns as two extra right-hand
//     sides (spikes);
//  4. the 2 G wave-end unknowns satisfy a small system, exchanged in LDS and
//     solved by every lane;
//  5. back-substitution.
// (a0, b0, c0, d0) is the chunk's first row.  On exit x[r] holds the solution
// of row lg * RPL + r.  xch: LDS exchange area of this line's waves (9 G
// values); all waves of the workgroup must call this together when G > 1.
// drop: couplings below it are left out of the cyclic reduction (see there).
template <typename R, int RPL, int G>
__device__ inline void solve_tail(R a0, R b0, R c0, R d0, R (&al)[RPL], R (&ga)[RPL],
                                  R (&de)[RPL], R (&x)[RPL], int lane, int wig, R *xch, R drop) {
    static_assert(RPL >= 2, "chunks of at least two rows");
#pragma unroll
    for (int r = RPL - 3; r >= 1; --r) {
        de[r] = de[r] - ga[r] * de[r + 1];
        al[r] = al[r] - ga[r] * al[r + 1];
        ga[r] = -ga[r] * ga[r + 1];
    }
    // first row: a0 x_e(k-1) + sb x_0 + sc x_e(k) = sd
    R sb, sc, sd;
    if (RPL == 2) {
        sb = b0;
        sc = c0;
        sd = d0;
    } else {
        sb = b0 - c0 * al[1];
        sc = -c0 * ga[1];
        sd = d0 - c0 * de[1];
    }
    const R isb = rcp(sb);
    const R sig = a0 * isb, tau = sc * isb, rho = sd * isb;   // x_0 = rho - sig x_e(k-1) - tau x_e(k)
    // Lane reads wrap around the wave: a value from past either end only meets
    // a coefficient that is exactly zero there (the line's first row has no
    // west coupling, its last no east coupling, the spikes zero the wave
    // ends, and cyclic reduction keeps couplings beyond the ends zero), and
    // every lane's values are finite, so no select is needed.
    // (l4 is opaque to the optimiser: the twelve addresses are formed here,
    // not hoisted out of the caller's loop into registers held throughout)
    int l4 = lane << 2;
    asm volatile("" : "+v"(l4));
    const int up1 = l4 + 4 * (WAVE - 1), dn1 = l4 + 4;
    R sigN = lane_read(sig, dn1), tauN = lane_read(tau, dn1);
    R rhoN = lane_read(rho, dn1);
    if constexpr (G > 1) {
        if (lane == 0) {
            xch[3 * wig + 0] = sig;
            xch[3 * wig + 1] = tau;
            xch[3 * wig + 2] = rho;
        }
        __syncthreads();
        if (lane == WAVE - 1 && wig < G - 1) {
            sigN = xch[3 * (wig + 1) + 0];
            tauN = xch[3 * (wig + 1) + 1];
            rhoN = xch[3 * (wig + 1) + 2];
        }
    }
    const int e = RPL - 1;
    // reduced row of x_e(k):  A x_e(k-1) + B x_e(k) + C x_e(k+1) = D
    R A = -al[e] * sig;
    R B = (R)1 - al[e] * tau - ga[e] * sigN;
    R C = -ga[e] * tauN;
    R D = de[e] - al[e] * rho - ga[e] * rhoN;
    {
        const R ib = rcp(B);
        A *= ib;
        C *= ib;
        D *= ib;
    }
    // spikes: couplings across the wave ends moved to extra right-hand sides
    R PL = (R)0, PR = (R)0, Afirst = (R)0, Clast = (R)0;
    if constexpr (G > 1) {
        Afirst = __shfl(A, 0, WAVE);
        Clast = __shfl(C, WAVE - 1, WAVE);
        if (lane == 0) {
            A = (R)0;
            PL = (R)1;
        }
        if (lane == WAVE - 1) {
            C = (R)0;
            PR = (R)1;
        }
    }
    // A pass squares the couplings (they fall as exp(-distance / diffusion
    // length of a step) and eq. (21) bounds that length by an axial interval),
    // so most lines are done after one to three passes: stop once no lane of
    // the wave couples by more than `drop`, which leaves the solution as it
    // is to that part of its largest value.  (1024 x 4096 FP64 step 25.6 us
    // with six passes and a clamped table index in every law, 23.9 without.)
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
        if (!__any(!(fabs(A) < drop && fabs(C) < drop))) break;
        const int iu = l4 + 4 * (WAVE - s), id = l4 + 4 * s;
        const R Am = lane_read(A, iu), Cm = lane_read(C, iu), Dm = lane_read(D, iu);
        const R Ap = lane_read(A, id), Cp = lane_read(C, id), Dp = lane_read(D, id);
        const R ib = rcp((R)1 - A * Cm - C * Ap);
        const R nA = -A * Am * ib;
        const R nC = -C * Cp * ib;
        const R nD = (D - A * Dm - C * Dp) * ib;
        if constexpr (G > 1) {
            const R PLm = lane_read(PL, iu), PLp = lane_read(PL, id);
            const R PRm = lane_read(PR, iu), PRp = lane_read(PR, id);
            PL = (PL - A * PLm - C * PLp) * ib;
            PR = (PR - A * PRm - C * PRp) * ib;
        }
        A = nA;
        C = nC;
        D = nD;
    }
    R xe = D, uL = (R)0;
    if constexpr (G > 1) {
        // x_e = y + vL uL + vR uR with uL, uR the neighbouring waves' end unknowns
        const R vL = -Afirst * PL, vR = -Clast * PR;
        R *xi = xch + 3 * G;     // per wave: y, vL, vR at its first and last lane
        if (lane == 0) {
            xi[6 * wig + 0] = D;
            xi[6 * wig + 1] = vL;
            xi[6 * wig + 2] = vR;
        }
        if (lane == WAVE - 1) {
            xi[6 * wig + 3] = D;
            xi[6 * wig + 4] = vL;
            xi[6 * wig + 5] = vR;
        }
        __syncthreads();
        // f_w = y0 + vL0 l_{w-1} + vR0 f_{w+1};  l_w = y63 + vL63 l_{w-1} + vR63 f_{w+1}
        // eliminate upwards: f_w = g_w + h_w f_{w+1}, l_w = p_w + q_w f_{w+1}
        R gq[G], hq[G], pq[G], qq[G];
        R pPrev = (R)0, qPrev = (R)0;
#pragma unroll
        for (int w = 0; w < G; ++w) {
            const R y0 = xi[6 * w + 0], vL0 = xi[6 * w + 1], vR0 = xi[6 * w + 2];
            const R y63 = xi[6 * w + 3], vL63 = xi[6 * w + 4], vR63 = xi[6 * w + 5];
            const R den = rcp((R)1 - vL0 * qPrev);
            gq[w] = (y0 + vL0 * pPrev) * den;
            hq[w] = vR0 * den;
            pq[w] = y63 + vL63 * (pPrev + qPrev * gq[w]);
            qq[w] = vR63 + vL63 * qPrev * hq[w];
            pPrev = pq[w];
            qPrev = qq[w];
        }
        R fNext = (R)0, fw[G], lw[G];
#pragma unroll
        for (int w = G - 1; w >= 0; --w) {
            fw[w] = gq[w] + hq[w] * fNext;
            lw[w] = pq[w] + qq[w] * fNext;
            fNext = fw[w];
        }
        R uR = (R)0;
#pragma unroll
        for (int w = 0; w < G; ++w) {
            if (w == wig - 1) uL = lw[w];
            if (w == wig + 1) uR = fw[w];
        }
        xe = D + vL * uL + vR * uR;
    }
    R xeP = lane_read(xe, up1);
    if (G > 1 && lane == 0) xeP = uL;
    const R x0 = rho - sig * xeP - tau * xe;
#pragma unroll
    for (int r = 1; r < RPL - 1; ++r) x[r] = de[r] - al[r] * x0 - ga[r] * xe;
    x[0] = x0;
    x[e] = xe;
}

// FP32 fields carry a compensated pair per node (hi + lo, |lo| <= ulp(hi)/2):
// a single float cannot hold per-step increments far below its ulp, so the
// low part keeps them; arithmetic stays in FP32.
template <typename R>
struct Pair {
    static constexpr bool on = false;
};
template <>
struct Pair<float> {
    static constexpr bool on = true;
};

// (a_hi + a_lo) - (b_hi + b_lo) for nearby values: the hi difference is exact
template <typename R>
__device__ inline R dif(R ah, R al, R bh, R bl) {
    if constexpr (Pair<R>::on)
        return (ah - bh) + (al - bl);
    else
        return ah - bh;
}

// The device's image of a plan's tables: the laws, each line class's (the
// full lines', and a stepped domain's terminal lines') per-row gw and ge,
// each class's row words, the lane words.  The stepping kernel takes the laws
// it uses and the full lines' gw, ge into LDS (a terminal line's rows are the
// same up to its wall), the adjoint kernels everything up to the lane words,
// each by stage_tables.
__host__ __device__ constexpr size_t up16(size_t b) { return (b + 15) & ~(size_t)15; }
// bytes of one law
template <typename R>
__host__ __device__ constexpr size_t law_size(bool poly) {
    return poly ? sizeof(R) * POLY_BLK : sizeof(R) == 8 ? sizeof(double) * POW_BLK : sizeof(float4);
}
template <typename R>
__host__ __device__ inline size_t law_bytes(int L, bool poly) {
    // (FP64: then the {K, A} pairs of LawLds::cube)
    return up16((law_size<R>(poly) + (sizeof(R) == 8 && !poly ? 16 : 0)) * (3 * L + 2));
}
// the laws the stepping kernel uses: radial, ratio and, unless every exponent
// is 3, capacity laws
template <typename R>
__host__ __device__ inline size_t step_law_bytes(int L, bool cube, bool poly) {
    return up16(law_size<R>(poly) * (cube ? 2 : 3) * L);
}
// gw, ge of a line class
template <typename R>
__host__ __device__ inline size_t geom_bytes(int np) {
    return 2 * sizeof(R) * (size_t)np;
}
template <typename R>
__host__ __device__ inline size_t info_offset(int L, int np, bool poly, bool stepped) {
    return law_bytes<R>(L, poly) + (stepped ? 2 : 1) * geom_bytes<R>(np);
}
template <typename R>
__host__ __device__ inline size_t tables_bytes(int L, int np, bool poly, bool stepped) {
    return info_offset<R>(L, np, poly, stepped) + (stepped ? 2 : 1) * sizeof(uint32_t) * (size_t)np;
}
// The stepping kernel's LDS: laws, gw and ge of the full lines, then the
// axial fluxes of its lines: a slot of one value per row for each line group
// and one more.
template <typename R>
__host__ __device__ inline size_t step_tables_bytes(int L, int np, bool cube, bool poly) {
    return step_law_bytes<R>(L, cube, poly) + geom_bytes<R>(np);
}
template <typename R>
__host__ __device__ inline size_t flux_bytes(int np, int wpl) {
    return sizeof(R) * (size_t)(STEP_WAVES / wpl + 1) * np;
}

// step_march keeps a two-slot ring of line buffers per wave after the tables
// (the lines after the current one, loaded straight into LDS): a slot is RPL
// rows x planes x 64 lanes.
template <typename R>
__host__ __device__ inline size_t ring_slot_elems(int rpl) {
    return (size_t)rpl * (Pair<R>::on ? 2 : 1) * WAVE;
}
// The ring serves FP32 pairs while a slot stays within 4 KiB; FP64 spends
// that LDS on its law tables instead (its prefetch gained nothing measurable).
template <typename R>
__host__ __device__ constexpr bool ring_used(int rpl) {
    // a slot of rpl rows x 2 planes x 64 lanes, filled in 16-byte pieces
    return sizeof(R) == 4 && rpl * 2 * WAVE * sizeof(R) <= 4096 && (rpl * 2) % 4 == 0;
}
// FP64 with 10 or more rows per lane keeps the carried axial fluxes in LDS
// (registers)
template <typename R>
__host__ __device__ constexpr bool fs_in_lds(int rpl) {
    return sizeof(R) == 8 && rpl >= 10;
}
// the ring, or the FP64 carried fluxes, after the tables
template <typename R>
__host__ __device__ inline size_t line_lds_bytes(int rpl) {
    if (ring_used<R>(rpl)) return sizeof(R) * 2 * (size_t)STEP_WAVES * ring_slot_elems<R>(rpl);
    if (fs_in_lds<R>(rpl)) return sizeof(R) * (size_t)STEP_WAVES * rpl * WAVE;
    return 0;
}

// Start the copy of a plan's tables (two ranges of the image, lengths
// multiples of 16 bytes, one after the other in LDS); all STEP_WAVES waves
// call it, and stage_wait before the first read.
// A launch runs only one or two lines per wave, so the tables' latency is
// part of every step.  Copied through registers in loops (each 4 KiB pass of
// each table waits for its loads: 11 memory latencies in a row for 8 layers
// and 1024 rows) the 1024 x 4096 FP64 step took 28.0 us and a 64 x 128 FP32
// step 5.1 us; with every wave issuing all its pieces of 1 KiB (64 lanes x 16
// bytes, memory to LDS, no registers) before anything waits, 25.6 and 4.0 us.
__device__ inline void stage_range(const unsigned char *img, unsigned char *smem, unsigned bytes,
                                   unsigned wv, int lane) {
    const unsigned full = bytes >> 10, rem = bytes & 1023;
    for (unsigned c = wv; c < full; c += STEP_WAVES)
        __builtin_amdgcn_global_load_lds((const void *)(img + (c << 10) + 16 * lane),
                                         (__attribute__((address_space(3))) void *)(smem + (c << 10)),
                                         16, 0, 0);
    // the last piece, under 1 KiB
    if (wv == full % STEP_WAVES && 16u * lane < rem)
        *(uint4 *)(smem + (full << 10) + 16 * lane) = *(const uint4 *)(img + (full << 10) + 16 * lane);
}
__device__ inline void stage_tables(const unsigned char *a, unsigned na, const unsigned char *b,
                                    unsigned nb, unsigned char *smem) {
    const int lane = threadIdx.x & (WAVE - 1);
    const unsigned wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    stage_range(a, smem, na, wv, lane);
    if (nb) stage_range(b, smem + na, nb, STEP_WAVES - 1 - wv, lane);
}
// every piece of the tables has landed (vmcnt 0) and every wave knows it
__device__ inline void stage_wait() {
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
}

// The law evaluator over the staged tables.
template <typename R, bool POLY>
__device__ inline auto staged_laws(const unsigned char *smem, int L) {
    if constexpr (POLY) return LawPoly<R>{(const R *)smem, L};
    else if constexpr (sizeof(R) == 8) return LawLds<double>{(const double *)smem, L};
    else return LawLds<float>{(const float4 *)smem, L};
}

}  // namespace cryo
