// Launches of the stepping kernel, the layout conversions around it, and the
// table image it reads.
#include <math.h>
#include <string.h>

#include "step_kernel.h"

namespace cryo {

// the launches of step_f64*.hip and step_f32*.hip
#define CRYO_STEP_EXTERN(R, STEPPED, SHARED) \
    template <> \
    bool StepLaunch<R, STEPPED, SHARED>::step(int, int, dim3, size_t, hipStream_t, \
                                              const StepArgs<R> &); \
    template <> \
    bool StepLaunch<R, STEPPED, SHARED>::batch(int, int, dim3, size_t, hipStream_t, \
                                               const StepArgs<R> *, const int2 *, int64_t, \
                                               const int64_t *);
CRYO_STEP_EXTERN(double, false, false)
CRYO_STEP_EXTERN(double, false, true)
CRYO_STEP_EXTERN(double, true, false)
CRYO_STEP_EXTERN(double, true, true)
CRYO_STEP_EXTERN(float, false, false)
CRYO_STEP_EXTERN(float, false, true)
CRYO_STEP_EXTERN(float, true, false)
CRYO_STEP_EXTERN(float, true, true)
#define CRYO_MULTI_EXTERN(R, STEPPED) \
    template <> \
    bool MultiLaunch<R, STEPPED>::step(int, int, dim3, size_t, hipStream_t, const StepArgs<R> &, \
                                       const MultiRun<R> &);
CRYO_MULTI_EXTERN(double, false)
CRYO_MULTI_EXTERN(double, true)
CRYO_MULTI_EXTERN(float, false)
CRYO_MULTI_EXTERN(float, true)

// Layout conversions: the ABI field (row major; FP32 two planes [2][nz][nr],
// rounded value and residual) and the internal lines ([nz][np], FP32
// [nz][2][np], lane-major).  One wave per line and plane: both sides are read
// and written 64 rows at a time, and the wave turns the line over in LDS (one
// element of padding per chunk, so that the chunks' rows fall on different
// banks).  Bound by memory: 1024 x 4096 in and out 22 us FP64, 25 us FP32 pairs
// (40 and 59 us with an element per thread, its other side a cache line apart
// from its neighbour's, and 64-bit divisions); the 256-cell sweep's fields, one
// launch each way, 0.66 ms (2.4 ms with a launch per cell).
constexpr int CONV_WAVES = 4;
template <typename R>
struct ConvArgs {
    R *T;              // ABI field
    R *Ti;             // internal lines
    int nz, nr, np, rpl, nl;
    R pad;
    int *flag;
};
template <typename R>
__host__ __device__ constexpr int planes() { return Pair<R>::on ? 2 : 1; }
__host__ __device__ inline int conv_lds_rows(int np, int nl) { return np + nl; }

// line p = j planes + plane; buf: this wave's LDS
template <typename R>
__device__ inline void line_in(const ConvArgs<R> &c, int p, R *buf, int lane) {
    constexpr int U = 8;
    const int j = p / planes<R>(), plane = p % planes<R>();
    const R *src = c.T + ((size_t)plane * c.nz + j) * c.nr;
    R *dst = c.Ti + (size_t)p * c.np;
    const R pad = plane == 0 ? c.pad : (R)0;
    for (int i0 = lane; i0 < c.np; i0 += U * WAVE) {
        R v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * WAVE;
            v[u] = i < c.nr ? src[i] : pad;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * WAVE;
            if (i < c.np) buf[i + i / c.rpl] = v[u];
        }
    }
    __builtin_amdgcn_wave_barrier();
    // position q = reg nl + lg holds row lg rpl + reg
    for (int lg = lane; lg < c.nl; lg += WAVE)
        for (int r = 0; r < c.rpl; ++r) dst[r * c.nl + lg] = buf[lg * (c.rpl + 1) + r];
    __builtin_amdgcn_wave_barrier();
}

template <typename R>
__device__ inline int line_out(const ConvArgs<R> &c, int p, R *buf, int lane) {
    constexpr int U = 8;
    const int j = p / planes<R>(), plane = p % planes<R>();
    const R *src = c.Ti + (size_t)p * c.np;
    R *dst = c.T + ((size_t)plane * c.nz + j) * c.nr;
    for (int lg = lane; lg < c.nl; lg += WAVE)
        for (int r0 = 0; r0 < c.rpl; r0 += U) {
            R v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = r0 + u < c.rpl ? src[(r0 + u) * c.nl + lg] : (R)0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (r0 + u < c.rpl) buf[lg * (c.rpl + 1) + r0 + u] = v[u];
        }
    __builtin_amdgcn_wave_barrier();
    int bad = 0;
    for (int i = lane; i < c.nr; i += WAVE) {
        const R v = buf[i + i / c.rpl];
        dst[i] = v;
        bad |= !isfinite(v);
    }
    __builtin_amdgcn_wave_barrier();
    return bad;
}

template <typename R>
__global__ __launch_bounds__(CONV_WAVES *WAVE) void k_to_internal(ConvArgs<R> c) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    R *buf = (R *)smem + (size_t)wv * conv_lds_rows(c.np, c.nl);
    if (blockIdx.x == 0 && threadIdx.x == 0 && c.flag) *c.flag = 0;
    for (int p = blockIdx.x * CONV_WAVES + wv; p < c.nz * planes<R>(); p += gridDim.x * CONV_WAVES)
        line_in(c, p, buf, lane);
}

template <typename R>
__global__ __launch_bounds__(CONV_WAVES *WAVE) void k_from_internal(ConvArgs<R> c) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    R *buf = (R *)smem + (size_t)wv * conv_lds_rows(c.np, c.nl);
    int bad = 0;
    for (int p = blockIdx.x * CONV_WAVES + wv; p < c.nz * planes<R>(); p += gridDim.x * CONV_WAVES)
        bad |= line_out(c, p, buf, lane);
    if (bad) atomicOr(c.flag, 1);
}

// The same for every instance of a batch in one launch: line numbers run over
// the instances (first[i] .. first[i + 1] - 1), each wave takes a contiguous
// run of them.
template <typename R, bool IN>
__global__ __launch_bounds__(CONV_WAVES *WAVE) void k_batch_convert(const BatchConv *inst,
                                                                    const int64_t *first, int n,
                                                                    R *T, int par, int buf_rows) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    R *buf = (R *)smem + (size_t)wv * buf_rows;
    if constexpr (IN)
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
            *inst[i].flag = 0;
    const int64_t waves = (int64_t)gridDim.x * CONV_WAVES, w = blockIdx.x * CONV_WAVES + wv;
    const int64_t total = first[n], per = (total + waves - 1) / waves;
    int64_t p = w * per;
    const int64_t end = min(p + per, total);
    if (p >= end) return;
    int lo = 0, hi = n;                          // the instance of line p
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (first[mid] <= p) lo = mid;
        else hi = mid;
    }
    for (int i = lo; p < end; ++i) {
        const BatchConv b = inst[i];
        const ConvArgs<R> c = {T + b.off, (R *)b.buf[par], b.nz, b.nr, b.np, b.rpl, b.nl,
                               (R)b.pad, b.flag};
        const int64_t stop = min(end, first[i + 1]);
        int bad = 0;
        for (; p < stop; ++p) {
            if constexpr (IN) line_in(c, (int)(p - first[i]), buf, lane);
            else bad |= line_out(c, (int)(p - first[i]), buf, lane);
        }
        if (bad) atomicOr(c.flag, 1);
    }
}

template <typename R>
__global__ void k_fill(R *T, size_t n, R v, size_t n_lo) {
    for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n + n_lo;
         idx += (size_t)gridDim.x * blockDim.x)
        T[idx] = idx < n ? v : (R)0;
}

// S[k] = sum over workgroups of the step-k partial sums, a wave per step: each
// lane its strided terms in order, then a fixed tree (one thread per step
// waited for its G loads in a row)
__global__ __launch_bounds__(WAVE) void k_surf_reduce(const double *part, int G, double *out) {
    const int k = blockIdx.x;
    double s = 0.0;
    for (int g = threadIdx.x; g < G; g += WAVE) s += part[(size_t)k * G + g];
    for (int w = WAVE / 2; w > 0; w >>= 1) s += __shfl_down(s, w, WAVE);
    if (threadIdx.x == 0) out[k] = s;
}

static int blocks_for(size_t n) {
    size_t b = (n + 255) / 256;
    return (int)std::min<size_t>(b, 65536);
}

static cryo_status launch_check(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CRYO_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
    return CRYO_OK;
}

// whether a plan's lines share their axial fluxes (see step_shared in step_kernel.h)
bool step_shared(const cryo_plan *p) { return p->lpw == 1; }

static size_t multi_lds(const cryo_plan *p) {
    return step_lds(p) + 8 * (size_t)STEP_WAVES * p->np;     // a slot per line (FP32: two planes)
}
static int multi_grid(const cryo_plan *p, int K) {
    const int own = STEP_WAVES - 2 * (K - 1);
    return (p->nz - 2 + own - 1) / own;
}

// Steps that one launch takes: on a grid that leaves compute units idle a
// workgroup steps its neighbours' lines too, as far as it needs them, and
// saves launches (2.4 us each with the latency of the tables and lines).  As
// many as leave at most one workgroup per unit; us per step at 1, 2, 3, 4
// steps, 512 rows (FP64 | FP32):
//     514 lines   8.1  6.6  6.1  5.9    | 5.5  4.2  3.7  3.5   (4 taken)
//     1026        8.3  6.8  6.3  11.2   | 5.8  4.4  3.8  5.1   (3)
//     1538        8.7  7.0  11.6  16.5  | 6.1  4.6  5.5  7.4   (2)
//     2050        8.9  12.6  11.8  21.9 | 6.5  6.2  5.6  9.2   (1 | 3)
// FP32 with short chunks fits two workgroups on a unit: three steps gain up to
// 25 % there (128 rows: 4.1 -> 3.1), 10 rows per lane lose 15 % (7.9 -> 9.1,
// general laws).  Beyond, at 3074 lines, two steps would gain too (8.5 -> 6.5 at
// 8 rows per lane, 10.8 -> 10.0 at 10); the rule does not take them.
int step_multi(const cryo_plan *p) {
    if (!step_shared(p) || p->wpl != 1 || p->rpl > 10 || multi_lds(p) > MAX_STEP_LDS) return 1;
    for (int K = MULTI_MAX; K > 1; --K)
        if (multi_grid(p, K) <= N_CU) return K;
    return p->dtype == CRYO_F32 && p->rpl <= 8 && multi_grid(p, 3) <= 2 * N_CU ? 3 : 1;
}

// (a value per line where steps share a launch: the mean must not depend on
// how they are grouped)
int surf_cols(const cryo_plan *p) { return step_multi(p) > 1 ? p->nz - 2 : step_grid(p); }

static int grid_of(const cryo_plan *p, int lpw) {
    const int groups = (p->nz - 2 + lpw - 1) / lpw;
    const int per_wg = STEP_WAVES / p->wpl;
    return (groups + per_wg - 1) / per_wg;
}
int step_grid(const cryo_plan *p) { return grid_of(p, p->lpw); }

// FP32 pairs at their default of one line per wave run up to 8 workgroups per
// compute unit; their sums take the memory of the balanced grid's, so that a
// large grid's workspace (and what fits cryo_forward_noalloc's array) does not
// grow by a second part: 512 x 8194 66.0 MiB, 72.0 with all workgroups' sums.
int surf_grid(const cryo_plan *p) {
    const bool one = one_line_shape(p->dtype, p->rpl) && p->lpw == 1;
    return grid_of(p, one ? balanced_lpw(p->nz, p->wpl) : p->lpw);
}

// Steps per surface reduction: what fits the memory of SURF_CHUNK rows of one
// value per workgroup of surf_grid; with values per line an eighth of it (whole
// launches of 2, 3 or 4 steps).
int surf_chunk(const cryo_plan *p) {
    const int c = (int)std::min<int64_t>((int64_t)SURF_CHUNK * surf_grid(p) / surf_cols(p), SURF_CHUNK);
    return step_multi(p) > 1 ? std::min(c, SURF_CHUNK / STEP_WAVES) / 12 * 12 : c;
}

template <typename R>
static ConvArgs<R> conv_args(const cryo_plan *p, const void *T, const void *Ti, int *flag) {
    return ConvArgs<R>{(R *)T, (R *)Ti, p->nz, p->nr, p->np, p->rpl, WAVE * p->wpl,
                       (R)pad_value(p), flag};
}
template <typename R>
static void launch_convert(const cryo_plan *p, bool in, const void *T, const void *Ti, int *flag,
                           hipStream_t s) {
    const ConvArgs<R> c = conv_args<R>(p, T, Ti, flag);
    const int lines = c.nz * planes<R>();
    const dim3 g(std::min((lines + CONV_WAVES - 1) / CONV_WAVES, 65536)), b(CONV_WAVES * WAVE);
    const size_t lds = sizeof(R) * CONV_WAVES * conv_lds_rows(c.np, c.nl);
    if (in) hipLaunchKernelGGL(k_to_internal<R>, g, b, lds, s, c);
    else hipLaunchKernelGGL(k_from_internal<R>, g, b, lds, s, c);
}

cryo_status launch_to_internal(const cryo_plan *p, const void *T, void *Ti, int *flag,
                               hipStream_t s) {
    if (p->dtype == CRYO_F64) launch_convert<double>(p, true, T, Ti, flag, s);
    else launch_convert<float>(p, true, T, Ti, flag, s);
    return launch_check("to_internal");
}

cryo_status launch_from_internal(const cryo_plan *p, const void *Ti, void *T, int *flag,
                                 hipStream_t s) {
    if (p->dtype == CRYO_F64) launch_convert<double>(p, false, T, Ti, flag, s);
    else launch_convert<float>(p, false, T, Ti, flag, s);
    return launch_check("from_internal");
}

// a batch's fields between the caller's packed buffer T and the instances'
// internal buffers `par`
cryo_status launch_batch_convert(cryo_dtype dt, bool in, const BatchConv *inst,
                                 const int64_t *first, int n, int64_t lines, int buf_rows, void *T,
                                 int par, hipStream_t s) {
    // up to 16 waves a compute unit, one line each at least
    const dim3 g((unsigned)std::min<int64_t>((lines + CONV_WAVES - 1) / CONV_WAVES, 4096));
    const dim3 b(CONV_WAVES * WAVE);
    const size_t lds = (dt == CRYO_F64 ? 8 : 4) * (size_t)CONV_WAVES * buf_rows;
    if (dt == CRYO_F64 && in)
        hipLaunchKernelGGL((k_batch_convert<double, true>), g, b, lds, s, inst, first, n,
                           (double *)T, par, buf_rows);
    else if (dt == CRYO_F64)
        hipLaunchKernelGGL((k_batch_convert<double, false>), g, b, lds, s, inst, first, n,
                           (double *)T, par, buf_rows);
    else if (in)
        hipLaunchKernelGGL((k_batch_convert<float, true>), g, b, lds, s, inst, first, n,
                           (float *)T, par, buf_rows);
    else
        hipLaunchKernelGGL((k_batch_convert<float, false>), g, b, lds, s, inst, first, n,
                           (float *)T, par, buf_rows);
    return launch_check("batch convert");
}

cryo_status launch_fill(const cryo_plan *p, void *T, hipStream_t s) {
    size_t n = (size_t)p->nz * p->nr;
    if (p->dtype == CRYO_F64)
        hipLaunchKernelGGL(k_fill<double>, dim3(blocks_for(n)), dim3(256), 0, s, (double *)T, n,
                           p->prob.T_init, (size_t)0);
    else
        hipLaunchKernelGGL(k_fill<float>, dim3(blocks_for(2 * n)), dim3(256), 0, s, (float *)T, n,
                           (float)p->prob.T_init, n);
    return launch_check("fill");
}

// Arguments of the stepping kernel (its row tables and laws: capacity rows
// scaled by eta^2, so the source is too); the adjoint kernels take the same.
template <typename R>
static StepArgs<R> step_args(const cryo_plan *p, const void *Tin, void *Tout, double X,
                             double *partial, int *flag) {
    StepArgs<R> a;
    const double xs = p->eta * p->eta;
    a.flag = flag;
    a.Tin = (const R *)Tin;
    a.Tout = (R *)Tout;
    a.img = p->d_tab;
    a.L = p->L;
    a.cube = p->flaws.cube;
    a.nz = p->nz;
    a.np = p->np;
    a.lpw = p->lpw;
    a.m = p->masks;
    a.lanes = (unsigned)tables_bytes<R>(p->L, p->np, p->poly, p->stepped);
    a.joule = p->poly && p->joule_tref > 0;
    a.jsq = a.joule ? sqrt(p->joule_tref) : 1.0;
    a.X = (R)(X * xs * a.jsq);
    for (int s = 0; s < 4; ++s) {
        a.held[s] = p->prob.bc.kind[s] == CRYO_HELD;
        a.val[s] = (R)p->prob.bc.value[s];
    }
    a.partial = partial;
    a.wz_mid = 1.0 / (p->nz - 1);
    a.wz_end = 0.5 / (p->nz - 1);
    a.surf_lane = p->surf_lane;
    a.surf_reg = p->surf_reg;
    // stepped domain: the surface over lines 0..z_full
    a.z_full = p->stepped ? p->z_full : p->nz - 1;
    a.nr_top = p->stepped ? p->nr_top : p->nr;
    if (p->stepped) {
        a.wz_mid = 1.0 / p->z_full;
        a.wz_end = 0.5 / p->z_full;
    }
    a.surf_cols = step_multi(p) > 1 ? p->nz - 2 : 0;
    a.groups = step_grid(p);
    a.pulse = p->pulse;
    a.pulse.amplitude *= xs;
    a.buf[0] = a.buf[1] = nullptr;
    return a;
}

template <typename R>
static cryo_status step_t(const cryo_plan *p, const void *Tin, void *Tout, double X,
                          double *partial, int *flag, hipStream_t s) {
    StepArgs<R> a = step_args<R>(p, Tin, Tout, X, partial, flag);
    const dim3 g(step_grid(p));
    const size_t lds = step_lds(p);
    const int key = p->rpl * 10 + p->wpl, laws = p->poly ? 2 : a.cube ? 0 : 1;
    const bool shared = step_shared(p);
    const bool built =
        p->stepped ? (shared ? StepLaunch<R, true, true>::step(laws, key, g, lds, s, a)
                             : StepLaunch<R, true, false>::step(laws, key, g, lds, s, a))
                   : (shared ? StepLaunch<R, false, true>::step(laws, key, g, lds, s, a)
                             : StepLaunch<R, false, false>::step(laws, key, g, lds, s, a));
    if (!built) return fail(CRYO_ERR_UNSUPPORTED, "radial chunk shape");
    return launch_check("step");
}

cryo_status launch_step(const cryo_plan *p, const void *Tin, void *Tout, double X,
                        double *partial, int *flag, hipStream_t s) {
    return p->dtype == CRYO_F64 ? step_t<double>(p, Tin, Tout, X, partial, flag, s)
                                : step_t<float>(p, Tin, Tout, X, partial, flag, s);
}

template <typename R>
static cryo_status steps_t(const cryo_plan *p, const void *Tin, void *Tout, int K,
                           const double *X, double *partial, int *flag, hipStream_t s) {
    const StepArgs<R> a = step_args<R>(p, Tin, Tout, 0.0, partial, flag);
    MultiRun<R> run = {};
    run.K = K;
    for (int k = 0; k < K; ++k) run.X[k] = (R)(X[k] * (p->eta * p->eta) * a.jsq);
    const dim3 g(multi_grid(p, K));
    const int laws = p->poly ? 2 : a.cube ? 0 : 1;
    const bool built =
        p->stepped ? MultiLaunch<R, true>::step(laws, p->rpl, g, multi_lds(p), s, a, run)
                   : MultiLaunch<R, false>::step(laws, p->rpl, g, multi_lds(p), s, a, run);
    if (!built) return fail(CRYO_ERR_UNSUPPORTED, "radial chunk shape");
    return launch_check("steps");
}

// K steps (at most step_multi) in one launch; X: their sources, partial: the
// first one's partial sums
cryo_status launch_steps(const cryo_plan *p, const void *Tin, void *Tout, int K, const double *X,
                         double *partial, int *flag, hipStream_t s) {
    if (K == 1) return launch_step(p, Tin, Tout, X[0], partial, flag, s);
    return p->dtype == CRYO_F64 ? steps_t<double>(p, Tin, Tout, K, X, partial, flag, s)
                                : steps_t<float>(p, Tin, Tout, K, X, partial, flag, s);
}

cryo_status launch_surf_reduce(const cryo_plan *p, const double *partial, int nsteps,
                               double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_surf_reduce, dim3(nsteps), dim3(WAVE), 0, s, partial, surf_cols(p), out);
    return launch_check("surf_reduce");
}

}  // namespace cryo

namespace cryo {

// ---- batch support -------------------------------------------------------
size_t step_desc_bytes(cryo_dtype dt) {
    return dt == CRYO_F64 ? sizeof(StepArgs<double>) : sizeof(StepArgs<float>);
}

template <typename R>
static size_t step_lds_t(const cryo_plan *p) {
    if (!step_shared(p))
        return tables_bytes<R>(p->L, p->np, p->poly, p->stepped) + line_lds_bytes<R>(p->rpl);
    const bool cube = p->flaws.cube && !p->poly;
    return step_tables_bytes<R>(p->L, p->np, cube, p->poly) + flux_bytes<R>(p->np, p->wpl);
}
size_t step_lds(const cryo_plan *p) {
    return p->dtype == CRYO_F64 ? step_lds_t<double>(p) : step_lds_t<float>(p);
}
// (the acceptance rule of earlier kernels, so that what is accepted does not
// change; step_lds stays within the hardware's LDS for all that it accepts)
template <typename R>
static size_t tables_reserve_t(const cryo_plan *p) {
    const size_t rows = up16((2 * sizeof(R) + sizeof(uint32_t)) * (size_t)p->np);
    return up16((sizeof(R) == 8 ? LAW_RESERVE_F64 : LAW_RESERVE_F32) * (3 * p->L + 2)) +
           (p->stepped ? 2 : 1) * rows;
}
size_t tables_reserve(const cryo_plan *p) {
    return p->dtype == CRYO_F64 ? tables_reserve_t<double>(p) : tables_reserve_t<float>(p);
}
size_t step_lds_reserve(const cryo_plan *p) {
    return tables_reserve(p) + (p->dtype == CRYO_F64 ? line_lds_bytes<double>(p->rpl)
                                                     : line_lds_bytes<float>(p->rpl));
}

// The image that ensure_device uploads once.
template <typename R>
static std::vector<unsigned char> table_image_t(const cryo_plan *p) {
    const size_t nl = p->lanes.size(), nc = p->stepped ? 2 : 1;
    const size_t lo = tables_bytes<R>(p->L, p->np, p->poly, p->stepped);
    std::vector<unsigned char> img(lo + nl * sizeof(LaneWord), 0);
    const int nlaw = 3 * p->L + 2;
    R *law = (R *)img.data();
    if (p->poly) {
        for (int i = 0; i < POLY_BLK * nlaw; ++i) law[i] = (R)p->fpow_blob[i];
    } else if constexpr (sizeof(R) == 8) {
        memcpy(law, p->fpow_blob.data(), sizeof(double) * pow_blob_doubles(p->L));
    } else {
        const Laws &l = p->flaws;
        for (int i = 0; i < nlaw; ++i) {
            law[4 * i] = (R)l.lk[i];
            law[4 * i + 1] = (R)l.e[i];
            const bool capl = i >= 2 * p->L && i < 3 * p->L;
            law[4 * i + 2] = i < p->L ? (R)l.K[2 * p->L + i] : capl ? (R)l.K[i] : (R)0;
            law[4 * i + 3] = i == law_unit(p->L) ? (R)1 : (R)0;
        }
    }
    R *g = (R *)(img.data() + law_bytes<R>(p->L, p->poly));
    uint32_t *info = (uint32_t *)(img.data() + info_offset<R>(p->L, p->np, p->poly, p->stepped));
    for (size_t c = 0; c < nc; ++c) {
        for (int i = 0; i < p->np; ++i) {
            g[(2 * c) * p->np + i] = (R)(c ? p->tfgw : p->fgw)[i];
            g[(2 * c + 1) * p->np + i] = (R)(c ? p->tfge : p->fge)[i];
        }
        memcpy(info + c * p->np, (c ? p->tfinfo : p->finfo).data(), sizeof(uint32_t) * p->np);
    }
    memcpy(img.data() + lo, p->lanes.data(), nl * sizeof(LaneWord));
    return img;
}
std::vector<unsigned char> table_image(const cryo_plan *p) {
    return p->dtype == CRYO_F64 ? table_image_t<double>(p) : table_image_t<float>(p);
}

void step_desc_fill(const cryo_plan *p, void *out, void *buf0, void *buf1, int *flag) {
    if (p->dtype == CRYO_F64) {
        StepArgs<double> a = step_args<double>(p, nullptr, nullptr, 0.0, nullptr, flag);
        a.buf[0] = (double *)buf0;
        a.buf[1] = (double *)buf1;
        memcpy(out, &a, sizeof(a));
    } else {
        StepArgs<float> a = step_args<float>(p, nullptr, nullptr, 0.0, nullptr, flag);
        a.buf[0] = (float *)buf0;
        a.buf[1] = (float *)buf1;
        memcpy(out, &a, sizeof(a));
    }
}

template <typename R>
static cryo_status step_batch_t(int rpl, int wpl, bool cube, bool poly, bool stepped, bool shared,
                                const void *desc, const int2 *map, int nwg, size_t lds,
                                int64_t n, const int64_t *k0, hipStream_t s) {
    const StepArgs<R> *d = (const StepArgs<R> *)desc;
    const dim3 g(nwg);
    const int key = rpl * 10 + wpl, laws = poly ? 2 : cube ? 0 : 1;
    const bool built =
        stepped ? (shared ? StepLaunch<R, true, true>::batch(laws, key, g, lds, s, d, map, n, k0)
                          : StepLaunch<R, true, false>::batch(laws, key, g, lds, s, d, map, n, k0))
                : (shared ? StepLaunch<R, false, true>::batch(laws, key, g, lds, s, d, map, n, k0)
                          : StepLaunch<R, false, false>::batch(laws, key, g, lds, s, d, map, n, k0));
    if (!built) return fail(CRYO_ERR_UNSUPPORTED, "radial chunk shape");
    return launch_check("step_batch");
}

cryo_status launch_step_batch(cryo_dtype dt, int rpl, int wpl, bool cube, bool poly,
                              bool stepped, bool shared, const void *desc, const int2 *map,
                              int nwg, size_t lds, int64_t n, const int64_t *k0, hipStream_t s) {
    return dt == CRYO_F64 ? step_batch_t<double>(rpl, wpl, cube, poly, stepped, shared, desc, map,
                                                 nwg, lds, n, k0, s)
                          : step_batch_t<float>(rpl, wpl, cube, poly, stepped, shared, desc, map,
                                                nwg, lds, n, k0, s);
}

__global__ void k_set_i64(int64_t *p, int64_t v) { *p = v; }
__global__ void k_add_i64(int64_t *p, int64_t v) { *p += v; }

cryo_status launch_set_i64(int64_t *ptr, int64_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, ptr, v);
    return launch_check("set_i64");
}

cryo_status launch_add_i64(int64_t *ptr, int64_t v, hipStream_t s) {
    hipLaunchKernelGGL(k_add_i64, dim3(1), dim3(1), 0, s, ptr, v);
    return launch_check("add_i64");
}

}  // namespace cryo

namespace cryo {
StepArgs<double> step_args_f64(const cryo_plan *p, int *flag) {
    return step_args<double>(p, nullptr, nullptr, 0.0, nullptr, flag);
}
}  // namespace cryo
