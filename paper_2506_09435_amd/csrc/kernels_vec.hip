// Vector kernels of the preconditioned conjugate-gradient solve (paper Sec. 4: CG for the
// Laplace system) and its FP64/FP32 defect correction.
//
// All reductions are deterministic: grid-stride kernels whose grid depends on the mesh only write
// one FP64 partial per block (wave64 shuffle reduction, then the block's waves in order).  The
// kernel that needs the sum adds the partials in a fixed order in every block, and its first block
// stores the device scalars (alpha, r.z, convergence flag); the p.Ap partials of large meshes, and
// the sums at a solve's start, are added by a single-block kernel.  Once `done` is set, every later
// kernel of the iteration leaves its vectors alone, so the host may check convergence only every few
// iterations without changing the result.
//
// Vectors hold all n_v volume nodes; the free-surface level [top*n_s, n_v) of r, p, q and
// dinv is kept at zero, so the iteration acts on the non-surface unknowns only.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "deferred.h"
#include "fnpf_internal.h"
#include "reduce.h"

namespace fnpf {

namespace {

__global__ void k_set_lift(double *v, const double *phis, int64_t n_v, int64_t top0) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_v; i += (int64_t)gridDim.x * blockDim.x)
    v[i] = i >= top0 ? phis[i - top0] : 0.0;
}

__global__ void k_copy_top(double *x, const double *phis, int64_t n_s, int64_t top0) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_s; i += (int64_t)gridDim.x * blockDim.x)
    x[top0 + i] = phis[i];
}

__global__ void k_fill(double *v, double val, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    v[i] = val;
}

__global__ void k_zero_i32(int32_t *v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) v[i] = 0;
}

__global__ void k_cast_f32(const double *a, float *b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = (float)a[i];
}

// ||b||^2 with b = f - A [0; phi_s] (y = A [0; phi_s], surface rows masked to 0).
__global__ __launch_bounds__(kVecThreads) void k_bnorm(const double *f, const double *y, int64_t n_v, int64_t top0,
                                                       double *partial) {
  double v[1] = {0.0};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < top0; i += (int64_t)gridDim.x * blockDim.x) {
    double b = (f ? f[i] : 0.0) - y[i];
    v[0] += b * b;
  }
  block_partials<1>(v, partial);
}

__global__ __launch_bounds__(kVecThreads) void k_fin_bnorm(const double *partial, int np, PcgScalars *sc, double rtol,
                                                           double atol) {
  double s[1];
  final_sums<1>(partial, np, s);
  if (threadIdx.x == 0) {
    sc->bnorm2 = s[0];
    sc->tol2 = fmax(rtol * rtol * s[0], atol * atol);
  }
}

// r = f - A x (surface rows 0), z = dinv r, p = z; partial sums (r.z, r.r).
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_pcg_init(const double *f, const T *Ax, T *r, T *p, const T *dinv,
                                                          int64_t n_v, int64_t top0, double *partial) {
  double v[2] = {0.0, 0.0};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_v; i += (int64_t)gridDim.x * blockDim.x) {
    T ri = i < top0 ? (T)((f ? f[i] : 0.0) - (double)Ax[i]) : T(0);
    T zi = dinv[i] * ri;
    r[i] = ri;
    p[i] = zi;
    v[0] += (double)ri * (double)zi;
    v[1] += (double)ri * (double)ri;
  }
  block_partials<2>(v, partial);
}

__global__ __launch_bounds__(kVecThreads) void k_fin_init(const double *partial, int np, PcgScalars *sc, int relative,
                                                          double inner_rtol) {
  double s[2];
  final_sums<2>(partial, np, s);
  if (threadIdx.x == 0) {
    sc->rz2 = s[0];
    sc->rr = s[1];
    sc->rr0 = s[1];
    if (relative) sc->tol2 = inner_rtol * inner_rtol * s[1];
    sc->iters = 0;
    sc->breakdown = (s[1] == s[1] && s[1] <= 1e300) ? 0 : 2;
    sc->done = (sc->breakdown != 0 || s[1] <= sc->tol2) ? 1 : 0;
    sc->alpha = 0.0;
  }
}

// Outer residual of the mixed solve: r64 = f - A64 x (surface 0); r32 = (float) r64; the
// inner FP32 PCG starts from d = 0: z = dinv32 r32, p = z.  Partials (r64.r64, r32.z, r32.r32).
__global__ __launch_bounds__(kVecThreads) void k_resid_to32(const double *f, const double *Ax, float *r, float *p,
                                                            float *d, const float *dinv, int64_t n_v, int64_t top0,
                                                            double *partial) {
  double v[3] = {0.0, 0.0, 0.0};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_v; i += (int64_t)gridDim.x * blockDim.x) {
    double r64 = i < top0 ? (f ? f[i] : 0.0) - Ax[i] : 0.0;
    float r32 = (float)r64;
    float z = dinv[i] * r32;
    r[i] = r32;
    p[i] = z;
    d[i] = 0.0f;
    v[0] += r64 * r64;
    v[1] += (double)r32 * (double)z;
    v[2] += (double)r32 * (double)r32;
  }
  block_partials<3>(v, partial);
}

// The inner FP32 solve stops at its relative reduction or, earlier, once its residual is below
// this fraction of the outer tolerance: the FP64 test that follows then passes unless the FP32
// rounding of the correction is larger, so iterations past that point would be wasted.
constexpr double kInnerFloor = 0.5;

__global__ __launch_bounds__(kVecThreads) void k_fin_outer(const double *partial, int np, PcgScalars *outer,
                                                           PcgScalars *inner, double inner_rtol) {
  double s[3];
  final_sums<3>(partial, np, s);
  if (threadIdx.x == 0) {
    outer->rr = s[0];
    outer->breakdown = (s[0] == s[0] && s[0] <= 1e300) ? 0 : 2;
    outer->done = (outer->breakdown != 0 || s[0] <= outer->tol2) ? 1 : 0;
    inner->rz2 = s[1];
    inner->rr = s[2];
    inner->rr0 = s[2];
    inner->tol2 = fmax(inner_rtol * inner_rtol * s[2], kInnerFloor * kInnerFloor * outer->tol2);
    inner->iters = 0;
    inner->breakdown = 0;
    inner->alpha = 0.0;
    inner->done = (outer->done || s[2] <= inner->tol2) ? 1 : 0;
  }
}

__global__ __launch_bounds__(kVecThreads) void k_fin_pq(const double *partial, int np, PcgScalars *sc) {
  if (sc->done) return;
  double s[1];
  final_sums<1>(partial, np, s);
  if (threadIdx.x == 0) cg_set_alpha(sc, s[0], sc->rz2);
}

// x += alpha p ; r -= alpha q ; partial sums (r.z, r.r) with z = dinv r.  q comes straight from
// the apply's first pass and is assembled here.  Bound by HBM on large meshes (seven vector
// accesses and the slots), by launches on small ones.
template <typename T>
struct PcgLoads { T x, r, p, d; };
// np > 0: alpha from the np partials of p.q, else as k_fin_pq left it
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads, LV == 1 ? 8 : 1) void k_pcg_update(T *x, T *r, const T *p, Deferred<T> q, const T *dinv,
                                                            int64_t n_s, double *partial, PcgScalars *sc,
                                                            const double *pq, int np) {
  const int dn = sc->done;
  const double rz = sc->rz2;
  double alpha = sc->alpha;
  const PartialLoads<1> pv(pq, np);
  bool live = dn == 0;
  T a = T(0);
  double v[2] = {0.0, 0.0};
  for_nodes<LV>(q, n_s, [&](int64_t i) { return PcgLoads<T>{x[i], r[i], p[i], dinv[i]}; },
            [&] {
              if (np > 0) live = cg_alpha(pv, dn != 0, rz, sc, alpha);
              a = (T)alpha;
              return live;
            },
            [&](int64_t i, const PcgLoads<T> &l, T qi) {
              x[i] = l.x + a * l.p;
              const T ri = l.r - a * qi;
              r[i] = ri;
              const T zi = l.d * ri;
              v[0] += (double)ri * (double)zi;
              v[1] += (double)ri * (double)ri;
            });
  if (!live) return;
  block_partials<2>(v, partial);
}

// after an iteration: the new r.z and r.r, convergence
__device__ __forceinline__ void pcg_store(PcgScalars *sc, double rz, double rr) {
  sc->rz2 = rz;
  sc->rr = rr;
  sc->iters += 1;
  if (!(rr == rr) || !(rr <= 1e300)) {
    sc->breakdown = 2;
    sc->done = 1;
  } else if (rr <= sc->tol2) {
    sc->done = 1;
  }
}

template <typename T>
struct Vec16;
template <>
struct Vec16<double> {
  using type = double2;
  static constexpr int W = 2;
};
template <>
struct Vec16<float> {
  using type = float4;
  static constexpr int W = 4;
};

// p = dinv r + beta p, in 16-byte chunks (all three are allocations of the library), beta from the np
// partials of (r.z, r.r), which every block sums and the first one stores with the convergence test (a
// late block that already sees `done` leaves p, which is not used any more).
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_pcg_dir(T *p, const T *r, const T *dinv, int64_t n_v,
                                                         PcgScalars *sc, const double *partial, int np) {
  using V = typename Vec16<T>::type;
  constexpr int W = Vec16<T>::W;
  const int64_t nvec = n_v / W;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int dn = sc->done;
  const double rz = sc->rz;
  const PartialLoads<2> sums(partial, np);
  int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  V pv{}, rv{}, dv{};
  if (c < nvec) {
    pv = reinterpret_cast<const V *>(p)[c];
    rv = reinterpret_cast<const V *>(r)[c];
    dv = reinterpret_cast<const V *>(dinv)[c];
  }
  asm volatile("" ::: "memory");   // the first loads stay ahead of the test
  double s[2];
  if (sums.sums(s, dn != 0)) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) pcg_store(sc, s[0], s[1]);
  const T b = (T)(s[0] / rz);
  for (; c < nvec; c += stride) {
    const int64_t c2 = c + stride;
    V p2{}, r2{}, d2{};
    if (c2 < nvec) {
      p2 = reinterpret_cast<const V *>(p)[c2];
      r2 = reinterpret_cast<const V *>(r)[c2];
      d2 = reinterpret_cast<const V *>(dinv)[c2];
    }
    T *ps = reinterpret_cast<T *>(&pv);
    const T *rs = reinterpret_cast<const T *>(&rv);
    const T *ds = reinterpret_cast<const T *>(&dv);
#pragma unroll
    for (int w = 0; w < W; ++w) ps[w] = ds[w] * rs[w] + b * ps[w];
    reinterpret_cast<V *>(p)[c] = pv;
    pv = p2;
    rv = r2;
    dv = d2;
  }
  if (blockIdx.x == 0)
    for (int64_t i = nvec * W + threadIdx.x; i < n_v; i += blockDim.x) p[i] = dinv[i] * r[i] + b * p[i];
}

__global__ void k_add_f32(double *x, const float *d, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] += (double)d[i];
}

__global__ void k_lincomb(double *out, double a, const double *x, double b, const double *y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (x ? a * x[i] : 0.0) + (y ? b * y[i] : 0.0);
}

// VJP of the linear free-surface conditions (d eta/dt = w, d phi_s/dt = -g eta):
// eta_bar += -g kbar_p, w_bar += kbar_e
__global__ void k_rhs_vjp_linear(const double *kbe, const double *kbp, double *eta_bar, double *w_bar, double g,
                                 int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    eta_bar[i] -= g * kbp[i];
    w_bar[i] += kbe[i];
  }
}

__global__ void k_relax_vjp(double *v, const double *cr, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    v[i] *= (1.0 - cr[i]);
}

// phi_s bar += phi_bar(surface level) - (A lambda)(surface level)
__global__ void k_surface_adj(double *phis_bar, const double *phibar, const double *Alam, int64_t n_s,
                              int64_t top0) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_s; i += (int64_t)gridDim.x * blockDim.x)
    phis_bar[i] += phibar[top0 + i] - Alam[top0 + i];
}

}  // namespace

hipError_t launch_lincomb(double *out, double a, const double *x, double b, const double *y, int64_t n,
                          hipStream_t s) {
  k_lincomb<<<kVecBlocks, kVecThreads, 0, s>>>(out, a, x, b, y, n);
  return hipGetLastError();
}

hipError_t launch_rhs_vjp_linear(const double *kbe, const double *kbp, double *eta_bar, double *w_bar, double g,
                                 int64_t n, hipStream_t s) {
  k_rhs_vjp_linear<<<kVecBlocks, kVecThreads, 0, s>>>(kbe, kbp, eta_bar, w_bar, g, n);
  return hipGetLastError();
}

hipError_t launch_relax_vjp(double *v, const double *cr, int64_t n, hipStream_t s) {
  k_relax_vjp<<<kVecBlocks, kVecThreads, 0, s>>>(v, cr, n);
  return hipGetLastError();
}

hipError_t launch_surface_adj(double *phis_bar, const double *phibar, const double *Alam, int64_t n_v, int64_t n_s,
                              hipStream_t s) {
  k_surface_adj<<<kVecBlocks, kVecThreads, 0, s>>>(phis_bar, phibar, Alam, n_s, n_v - n_s);
  return hipGetLastError();
}

hipError_t launch_set_lift(double *v, const double *phis, int64_t n_v, int64_t n_s, hipStream_t s) {
  k_set_lift<<<kVecBlocks, kVecThreads, 0, s>>>(v, phis, n_v, n_v - n_s);
  return hipGetLastError();
}

hipError_t launch_copy_top(double *x, const double *phis, int64_t n_v, int64_t n_s, hipStream_t s) {
  k_copy_top<<<kVecBlocks, kVecThreads, 0, s>>>(x, phis, n_s, n_v - n_s);
  return hipGetLastError();
}

hipError_t launch_fill(double *v, double val, int64_t n, hipStream_t s) {
  k_fill<<<kVecBlocks, kVecThreads, 0, s>>>(v, val, n);
  return hipGetLastError();
}

hipError_t launch_zero_i32(int32_t *v, int64_t n, hipStream_t s) {
  k_zero_i32<<<1, 64, 0, s>>>(v, n);
  return hipGetLastError();
}

hipError_t launch_cast_f32(const double *a, float *b, int64_t n, hipStream_t s) {
  k_cast_f32<<<kVecBlocks, kVecThreads, 0, s>>>(a, b, n);
  return hipGetLastError();
}

hipError_t launch_bnorm(const double *f, const double *y, int64_t n_v, int64_t n_s, double *partial,
                        PcgScalars *sc, double rtol, double atol, hipStream_t s) {
  k_bnorm<<<kVecBlocks, kVecThreads, 0, s>>>(f, y, n_v, n_v - n_s, partial);
  k_fin_bnorm<<<1, kVecThreads, 0, s>>>(partial, kVecBlocks, sc, rtol, atol);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_pcg_init(const double *f, const T *Ax, T *r, T *p, const T *dinv, int64_t n_v, int64_t n_s,
                           double *partial, PcgScalars *sc, bool relative_tol, double inner_rtol, hipStream_t s) {
  k_pcg_init<T><<<kVecBlocks, kVecThreads, 0, s>>>(f, Ax, r, p, dinv, n_v, n_v - n_s, partial);
  k_fin_init<<<1, kVecThreads, 0, s>>>(partial, kVecBlocks, sc, relative_tol ? 1 : 0, inner_rtol);
  return hipGetLastError();
}
template hipError_t launch_pcg_init<double>(const double *, const double *, double *, double *, const double *,
                                            int64_t, int64_t, double *, PcgScalars *, bool, double, hipStream_t);

hipError_t launch_resid_to32(const double *f, const double *Ax, float *r, float *p, float *d, const float *dinv,
                             int64_t n_v, int64_t n_s, double *partial, PcgScalars *outer, PcgScalars *inner,
                             double inner_rtol, hipStream_t s) {
  k_resid_to32<<<kVecBlocks, kVecThreads, 0, s>>>(f, Ax, r, p, d, dinv, n_v, n_v - n_s, partial);
  k_fin_outer<<<1, kVecThreads, 0, s>>>(partial, kVecBlocks, outer, inner, inner_rtol);
  return hipGetLastError();
}

hipError_t launch_finalize_pq(const double *partial, int np, PcgScalars *sc, hipStream_t s) {
  k_fin_pq<<<1, kVecThreads, 0, s>>>(partial, np, sc);
  return hipGetLastError();
}

// One PCG iteration's updates after q = A p (deferred), npq partials of p.q at the front of partial:
// x, r, the convergence test and the next direction.
template <typename T>
hipError_t launch_pcg_iteration(const Ctx &c, T *x, T *r, T *p, const T *q, const T *dinv, double *partial, int npq,
                                PcgScalars *sc, hipStream_t s) {
  const int nlv = node_levels(c), nb = node_blocks(c, nlv, nlv > 1 ? kNodeBlocks : kVecBlocks);
  double *rz = partial + npq;   // behind the partials of p.q, which other blocks may still be reading
  const int np = npq <= kFinPartials ? npq : 0;
  if (np == 0) k_fin_pq<<<1, kVecThreads, 0, s>>>(partial, npq, sc);
  with_levels(nlv, [&](auto lv) {
    k_pcg_update<lv(), T><<<nb, kVecThreads, 0, s>>>(x, r, p, apply_result<T>(c, q), dinv, c.n_s, rz, sc, partial, np);
  });
  static_assert(kVecBlocks <= kFinPartials && kNodeBlocks <= kFinPartials, "k_pcg_dir sums the update's partials");
  const int nd = (int)std::min<int64_t>((c.n_v / Vec16<T>::W + kVecThreads) / kVecThreads, kVecBlocks);
  k_pcg_dir<T><<<nd, kVecThreads, 0, s>>>(p, r, dinv, c.n_v, sc, rz, nb);
  return hipGetLastError();
}
template hipError_t launch_pcg_iteration<double>(const Ctx &, double *, double *, double *, const double *,
                                                 const double *, double *, int, PcgScalars *, hipStream_t);
template hipError_t launch_pcg_iteration<float>(const Ctx &, float *, float *, float *, const float *,
                                                const float *, double *, int, PcgScalars *, hipStream_t);

hipError_t launch_add_f32(double *x, const float *d, int64_t n_v, hipStream_t s) {
  k_add_f32<<<kVecBlocks, kVecThreads, 0, s>>>(x, d, n_v);
  return hipGetLastError();
}

}  // namespace fnpf
