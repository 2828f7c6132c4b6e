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

// ABI field -> internal lines.  FP32 fields are two planes [2][nz][nr]
// (rounded value, residual) and become [nz][2][np] internally.
template <typename R>
__global__ void k_to_internal(const R *T, R *Ti, int nz, int nr, int np, int rpl, R pad,
                              int *flag) {
    constexpr int NPL = Pair<R>::on ? 2 : 1;
    size_t n = (size_t)nz * NPL * np;
    size_t start = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (start == 0 && flag) *flag = 0;
    for (size_t idx = start; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        int j = (int)(idx / ((size_t)NPL * np));
        int rem = (int)(idx % ((size_t)NPL * np));
        int plane = rem / np, q = rem % np;
        const int nl = np / rpl;                      // lanes per line
        int i = (q % nl) * rpl + q / nl;
        R v = plane == 0 ? pad : (R)0;
        if (i < nr) v = T[((size_t)plane * nz + j) * nr + i];
        Ti[idx] = v;
    }
}

template <typename R>
__global__ void k_from_internal(const R *Ti, R *T, int nz, int nr, int np, int rpl, int *flag) {
    constexpr int NPL = Pair<R>::on ? 2 : 1;
    size_t n = (size_t)NPL * nz * nr;
    int bad = 0;
    for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
        int plane = (int)(idx / ((size_t)nz * nr));
        size_t rem = idx % ((size_t)nz * nr);
        int j = (int)(rem / nr), i = (int)(rem % nr);
        const int nl = np / rpl;
        R v = Ti[((size_t)j * NPL + plane) * np + (i % rpl) * nl + i / rpl];
        T[idx] = v;
        bad |= !isfinite(v);
    }
    if (bad) atomicOr(flag, 1);
}

template <typename R>
__global__ void k_fill(R *T, size_t n, R v, size_t n_lo) {
    for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n + n_lo;
         idx += (size_t)gridDim.x * blockDim.x)
        T[idx] = idx < n ? v : (R)0;
}

// S[k] = sum over workgroups of the step-k partial sums, in a fixed order
__global__ void k_surf_reduce(const double *part, int nsteps, int G, double *out) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nsteps) return;
    double s = 0.0;
    for (int g = 0; g < G; ++g) s += part[(size_t)k * G + g];
    out[k] = s;
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

// whether a plan's lines share their axial fluxes (see step_body)
bool step_shared(const cryo_plan *p) { return p->lpw == 1; }

int step_grid(const cryo_plan *p) {
    const int groups = (p->nz - 2 + p->lpw - 1) / p->lpw;
    const int per_wg = STEP_WAVES / p->wpl;
    return (groups + per_wg - 1) / per_wg;
}

template <typename R>
static cryo_status to_internal_t(const cryo_plan *p, const void *T, void *Ti, int *flag,
                                 hipStream_t s) {
    size_t n = (size_t)p->nz * p->np * (Pair<R>::on ? 2 : 1);
    hipLaunchKernelGGL(k_to_internal<R>, dim3(blocks_for(n)), dim3(256), 0, s, (const R *)T,
                       (R *)Ti, p->nz, p->nr, p->np, p->rpl, (R)p->prob.T_init, flag);
    return launch_check("to_internal");
}

cryo_status launch_to_internal(const cryo_plan *p, const void *T, void *Ti, int *flag,
                               hipStream_t s) {
    return p->dtype == CRYO_F64 ? to_internal_t<double>(p, T, Ti, flag, s)
                                : to_internal_t<float>(p, T, Ti, flag, s);
}

cryo_status launch_from_internal(const cryo_plan *p, const void *Ti, void *T, int *flag,
                                 hipStream_t s) {
    size_t n = (size_t)p->nz * p->nr * (p->dtype == CRYO_F32 ? 2 : 1);
    if (p->dtype == CRYO_F64)
        hipLaunchKernelGGL(k_from_internal<double>, dim3(blocks_for(n)), dim3(256), 0, s,
                           (const double *)Ti, (double *)T, p->nz, p->nr, p->np, p->rpl, flag);
    else
        hipLaunchKernelGGL(k_from_internal<float>, dim3(blocks_for(n)), dim3(256), 0, s,
                           (const float *)Ti, (float *)T, p->nz, p->nr, p->np, p->rpl, flag);
    return launch_check("from_internal");
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

cryo_status launch_surf_reduce(const cryo_plan *p, const double *partial, int nsteps,
                               double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_surf_reduce, dim3((nsteps + 255) / 256), dim3(256), 0, s, partial,
                       nsteps, step_grid(p), out);
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
