// p-multigrid preconditioner for the Laplace system on A_II.
//
// The paper solves the Laplace system with CG preconditioned by algebraic multigrid (Sec. 4
// solver settings).  Here the preconditioner is a V-cycle over polynomial degrees of the same
// extruded mesh, p -> p/2 -> ... -> 1: every level is a full context of the library at its
// degree (same columns, layers and corners; geometry from eta + h and h interpolated to its
// surface nodes), with Chebyshev smoothing of the Jacobi-scaled operator D^-1 A.  The transfer
// between a level of degree pf and the next of degree pc = pf/2 is the tensor-product Lagrange
// interpolation P of the coarse element polynomial at the fine GLL nodes, element by element;
// the restriction is its exact transpose.  With the same polynomial before and after the coarse
// correction, the V-cycle is a fixed symmetric positive definite operator, so the outer
// iteration stays plain CG.
//
// Deterministic: each fine node takes its interpolated value from the column that owns it, the
// restriction counts each fine node once (in its owner column, the shared layer level in the
// upper layer), and coarse sums are assembled with the owner-computes face slots of the coarse
// level; every reduction has a fixed order.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <exception>
#include <mutex>
#include <utility>
#include <vector>

#include "deferred.h"
#include "fnpf_internal.h"
#include "reduce.h"

namespace fnpf {

namespace {

constexpr int kMgCoarseSteps = 10;      // Chebyshev steps on the coarsest level
constexpr double kMgSafety = 1.1;       // upper end of the smoothing interval over the estimate
constexpr double kMgSmoothRatio = 24.0; // smoothing interval [lmax / 24, lmax]
constexpr double kMgCoarseRatio = 30.0;
constexpr int kLanczosSteps = 20;             // first estimate of the largest eigenvalue
constexpr int kPowNext = 1;                   // power iterations per geometry update after that
constexpr int kLzScalars = 2 * kLanczosSteps + 8;
constexpr int kMgCoef = 32;                   // coefficient-table entries per level
// Grid of the streaming vector kernels of the cycle: FP32 passes move half the bytes per element
// and need twice the blocks in flight to keep HBM busy (FP64 passes are slower with the larger
// grid).  Their reductions use the same grid, so partial counts follow it; the context's partial
// buffer is sized from the table of partials.h, which lists both grids (up to two sums per block).
template <typename T>
constexpr int kVB = sizeof(T) == 4 ? 2 * kVecBlocks : kVecBlocks;
static_assert(kVB<float> == 2 * kPartialVecBlocks && kVB<double> == kPartialVecBlocks,
              "vector grids must match the partial-sum table (partials.h)");

// Interpolation tables for a fine degree pf (2..8) and pc = pf / 2:
//   c_IP[pf][r (pc+1) + a] = l^c_a(x^f_r)   coarse Lagrange basis at the fine GLL nodes
//   c_IS[pf][a (pf+1) + i] = l^f_i(x^c_a)   fine Lagrange basis at the coarse GLL nodes
__constant__ double c_IP64[kMaxN1][kMaxN1 * kMaxN1];
__constant__ float c_IP32[kMaxN1][kMaxN1 * kMaxN1];
__constant__ double c_IS64[kMaxN1][kMaxN1 * kMaxN1];

template <typename T>
__device__ __forceinline__ T ip(int pf, int k);
template <>
__device__ __forceinline__ double ip<double>(int pf, int k) { return c_IP64[pf][k]; }
template <>
__device__ __forceinline__ float ip<float>(int pf, int k) { return c_IP32[pf][k]; }

double lagrange(const double *X, int n1, int j, double x) {
  double v = 1.0;
  for (int m = 0; m < n1; ++m)
    if (m != j) v *= (x - X[m]) / (X[j] - X[m]);
  return v;
}

hipError_t upload_tables() {
  static double IP[kMaxN1][kMaxN1 * kMaxN1];
  static float IP32[kMaxN1][kMaxN1 * kMaxN1];
  static double IS[kMaxN1][kMaxN1 * kMaxN1];
  std::memset(IP, 0, sizeof IP);
  std::memset(IP32, 0, sizeof IP32);
  std::memset(IS, 0, sizeof IS);
  for (int pf = 2; pf <= kMaxP; ++pf) {
    const int pc = pf / 2;
    double xf[kMaxN1], xc[kMaxN1];
    gll_host(pf, xf, nullptr, nullptr);
    gll_host(pc, xc, nullptr, nullptr);
    for (int r = 0; r <= pf; ++r)
      for (int a = 0; a <= pc; ++a) {
        IP[pf][r * (pc + 1) + a] = lagrange(xc, pc + 1, a, xf[r]);
        IP32[pf][r * (pc + 1) + a] = (float)IP[pf][r * (pc + 1) + a];
      }
    for (int a = 0; a <= pc; ++a)
      for (int i = 0; i <= pf; ++i) IS[pf][a * (pf + 1) + i] = lagrange(xf, pf + 1, i, xc[a]);
  }
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_IP64), IP, sizeof IP);
  if (e != hipSuccess) return e;
  e = hipMemcpyToSymbol(HIP_SYMBOL(c_IP32), IP32, sizeof IP32);
  if (e != hipSuccess) return e;
  return hipMemcpyToSymbol(HIP_SYMBOL(c_IS64), IS, sizeof IS);
}

template <int P, int DIM>
struct Lay {
  static constexpr int N1 = P + 1;
  static constexpr int NH = DIM == 3 ? N1 * N1 : N1;
  static constexpr int CPB = 256 / NH;
  static constexpr int NT = CPB * NH;
};

// ---- transfer kernels ------------------------------------------------------------------------

// Coarse surface data (eta + h and h) at the coarse nodes from the fine nodal values.
template <int PF, int DIM>
__global__ __launch_bounds__(256) void k_mg_surf(const double *__restrict__ Hf, const double *__restrict__ hf,
                                                 const int32_t *__restrict__ nodes_f,
                                                 const int32_t *__restrict__ nodes_c,
                                                 const uint8_t *__restrict__ flags_c, int ncols,
                                                 double *__restrict__ Hc, double *__restrict__ hc) {
  constexpr int PC = PF / 2, N1F = PF + 1, N1C = PC + 1;
  constexpr int NHC = Lay<PC, DIM>::NH, NHF = Lay<PF, DIM>::NH;
  const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t col = g / NHC;
  const int t = (int)(g - col * NHC);
  if (col >= ncols) return;
  if (!(flags_c[col * NHC + t] & kOwned)) return;
  const int a = t % N1C, b = DIM == 3 ? t / N1C : 0;
  double sH = 0.0, sh = 0.0;
  for (int j = 0; j < (DIM == 3 ? N1F : 1); ++j) {
    const double wj = DIM == 3 ? c_IS64[PF][b * N1F + j] : 1.0;
    for (int i = 0; i < N1F; ++i) {
      const double w = wj * c_IS64[PF][a * N1F + i];
      const int n = nodes_f[col * NHF + j * N1F + i];
      sH += w * Hf[n];
      sh += w * hf[n];
    }
  }
  const int n = nodes_c[col * NHC + t];
  Hc[n] = sH;
  hc[n] = sh;
}

// Restriction b_c = P^T (r_f - q_f) (q_f.y = NULL: P^T r_f).  One thread per (column, fine
// horizontal node) loads its fine line (owner columns only; the shared layer level counts in the
// upper layer) and contracts it vertically in registers; the horizontal contraction is split in
// two LDS stages over all threads of the column: (a, j, c) sums over i, then (a, b, c) over j.
// On slices q_f comes straight from the apply's first pass and is assembled here (in 3D the apply that
// leaves slots restricts by itself, and this kernel gets complete vectors).  blockIdx.y takes a chunk of
// lpc layers.  Coarse nodes owned by the column go to b_c, the others to the coarse face slots, and
// a chunk's top level below the next chunk behind them (deferred.h: the coarse level's first kernel
// adds them); the coarse surface level is set to zero.  The vertical carry of the
// shared layer level passes through a double-buffered LDS slot per coarse horizontal node.
template <int PF, int DIM, typename T>
__global__ __launch_bounds__(256) void k_restrict(const T *__restrict__ rf, Deferred<T> qf,
                                                  T *__restrict__ bc, T *__restrict__ Fc,
                                                  const int32_t *__restrict__ nodes_f,
                                                  const uint8_t *__restrict__ flags_f,
                                                  const int32_t *__restrict__ nodes_c,
                                                  const uint8_t *__restrict__ flags_c,
                                                  const int32_t *__restrict__ slot_c, int ncols, int nz,
                                                  int64_t ns_f, int64_t ns_c, int64_t nslots_c, int lpc,
                                                  const int32_t *__restrict__ skip) {
  using LF = Lay<PF, DIM>;
  constexpr int PC = PF / 2, N1F = PF + 1, N1C = PC + 1;
  constexpr int NHF = LF::NH, CPB = LF::CPB, NHC = Lay<PC, DIM>::NH;
  constexpr int NJ = DIM == 3 ? N1F : 1;               // fine rows left after stage A
  constexpr int NA = N1C * NJ * N1C;                   // stage A items (a, j, c)
  constexpr int NB = NHC * N1C;                        // stage B items (a, b, c)
  __shared__ T sW[CPB * N1C * NHF];
  __shared__ T sA[CPB * NA];
  __shared__ T sC[CPB * 2 * NHC];
  if (skip != nullptr && *skip) return;
  const int lc = threadIdx.x / NHF;
  const int t = threadIdx.x - lc * NHF;
  const int ci = blockIdx.x * CPB + lc;
  const bool active = ci < ncols;
  const int col = active ? ci : 0;
  const int hn = active ? nodes_f[col * NHF + t] : 0;
  const bool own = active && (flags_f[col * NHF + t] & kOwned);
  const int chunk = blockIdx.y, nchunk = gridDim.y, l0 = chunk * lpc, l1 = min(l0 + lpc, nz);
  int4 sl = make_int4(-1, -1, -1, 0);
  if constexpr (DIM == 2)
    if (own && hn < qf.n_hi) sl = qf.slots[hn];
  T *W = sW + lc * N1C * NHF;
  T *A = sA + lc * NA;
  T *Cr = sC + lc * 2 * NHC;
  const int vtop = PC * nz;
  // stage B items of this thread (it = t + m NHF, the same coarse horizontal node in every layer),
  // loaded once: the coarse node where the column owns it, else -1 - its face slot
  constexpr int MI = (NB + NHF - 1) / NHF;
  int dst[MI];
#pragma unroll
  for (int m = 0; m < MI; ++m) {
    const int it = t + m * NHF;
    const int h = it % NHC;
    dst[m] = 0;
    if (active && it < NB)
      dst[m] = (flags_c[col * NHC + h] & kOwned) ? nodes_c[col * NHC + h] : -1 - slot_c[col * NHC + h];
  }
  // the fine line of layer l + 1 is loaded while layer l is contracted (raw values of both
  // operands, so that nothing waits for them before their use)
  T nr[N1F], nq[N1F], nf[N1F];
  auto load_layer = [&](int l) {
    const int kmax = (l == nz - 1) ? N1F : PF;
#pragma unroll
    for (int k = 0; k < N1F; ++k) {
      const int64_t idx = (int64_t)(l * PF + k) * ns_f + hn;
      const bool ld = own && k < kmax;
      nr[k] = ld ? rf[idx] : T(0);
      nq[k] = (ld && qf.y) ? qf.y[idx] : T(0);
      nf[k] = (DIM == 2 && sl.x >= 0 && k < PF) ? qf.F[(int64_t)(l * PF + k) * qf.n_slots + sl.x] : T(0);
    }
  };
  load_layer(l0);
  for (int l = l0; l < l1; ++l) {
    T rv[N1F];
#pragma unroll
    for (int k = 0; k < N1F; ++k) rv[k] = nr[k] - (nq[k] + nf[k]);
    if constexpr (DIM == 2) {
      // the rest of q: further face slots, and at the bottom of a chunk of the apply the lower chunk's value
      auto more = [&](int s) {
        const T *f = qf.F + (int64_t)(l * PF) * qf.n_slots + s;
#pragma unroll
        for (int k = 0; k < PF; ++k) rv[k] -= f[k * qf.n_slots];
      };
      if (sl.y >= 0) more(sl.y);
      if (sl.z >= 0) more(sl.z);
      if (sl.w > 0)
        for (int q = 1; q <= qf.lists[sl.w]; ++q) more(qf.lists[sl.w + q]);
      if (qf.nchunk > 1 && l > 0 && (l * PF) % qf.clev == 0 && own) {
        const int c = l * PF / qf.clev - 1;
        const T *top = qf.F + (int64_t)(qf.nlev + c) * qf.n_slots;
        T z = (qf.F + (int64_t)(qf.nlev + qf.nchunk - 1) * qf.n_slots)[c * ns_f + hn];
        if (sl.x >= 0) z += top[sl.x];
        if (sl.y >= 0) z += top[sl.y];
        if (sl.z >= 0) z += top[sl.z];
        if (sl.w > 0) z = list_sum(qf, top, sl.w, z);
        rv[0] -= z;
      }
    }
    if (l + 1 < l1) load_layer(l + 1);
    T w[N1C];
#pragma unroll
    for (int c = 0; c < N1C; ++c) w[c] = T(0);
    if (own) {
#pragma unroll
      for (int k = 0; k < N1F; ++k)
#pragma unroll
        for (int c = 0; c < N1C; ++c) w[c] += ip<T>(PF, k * N1C + c) * rv[k];
    }
#pragma unroll
    for (int c = 0; c < N1C; ++c) W[c * NHF + t] = w[c];
    __syncthreads();
    if constexpr (DIM == 3) {
      // stage A: A[(c NJ + j) N1C + a] = sum_i IP[i][a] W[c][j][i]
      for (int it = t; it < NA; it += NHF) {
        const int a = it % N1C, j = (it / N1C) % NJ, c = it / (N1C * NJ);
        T acc = T(0);
#pragma unroll
        for (int i = 0; i < N1F; ++i) acc += ip<T>(PF, i * N1C + a) * W[c * NHF + j * N1F + i];
        A[it] = acc;
      }
      __syncthreads();
    }
    // stage B: coarse value (a, b, c) of this layer's element, assembled
#pragma unroll 1
    for (int m = 0; m < MI; ++m) {
      const int it = t + m * NHF;
      if (!active || it >= NB) continue;
      const int h = it % NHC, c = it / NHC;            // h = b N1C + a
      const int a = h % N1C, b = h / N1C;
      T acc = T(0);
      if constexpr (DIM == 3) {
#pragma unroll
        for (int j = 0; j < N1F; ++j) acc += ip<T>(PF, j * N1C + b) * A[(c * NJ + j) * N1C + a];
      } else {
#pragma unroll
        for (int i = 0; i < N1F; ++i) acc += ip<T>(PF, i * N1C + a) * W[c * NHF + i];
      }
      if (c == 0 && l > l0) acc += Cr[((l - 1) & 1) * NHC + h];
      if (c == PC && l < l1 - 1) {
        Cr[(l & 1) * NHC + h] = acc;                   // the shared layer level, finished above
        continue;
      }
      const int v = l * PC + c;
      const bool below = c == PC && l1 < nz;           // the next chunk's bottom level
      int d = dst[0];   // dst[m] by selects (constant indices keep dst in registers)
#pragma unroll
      for (int q = 1; q < MI; ++q)
        if (m == q) d = dst[q];
      if (below) {
        if (d >= 0)
          (Fc + (int64_t)(vtop + nchunk) * nslots_c)[chunk * ns_c + d] = acc;
        else
          Fc[(int64_t)(vtop + 1 + chunk) * nslots_c + (-1 - d)] = acc;
      } else if (d >= 0) {
        bc[(int64_t)v * ns_c + d] = (v == vtop) ? T(0) : acc;
      } else if (v != vtop) {
        Fc[(int64_t)v * nslots_c + (-1 - d)] = acc;
      }
    }
    __syncthreads();
  }
}

// Prolongation x_f += P x_c, written by the owner column of each fine node; blockIdx.y takes a chunk
// of lpc layers.
template <int PF, int DIM, typename T>
__global__ __launch_bounds__(256) void k_prolong_add(const T *__restrict__ xc, T *__restrict__ xf,
                                                     const int32_t *__restrict__ nodes_f,
                                                     const uint8_t *__restrict__ flags_f,
                                                     const int32_t *__restrict__ nodes_c, int ncols, int nz,
                                                     int64_t ns_f, int64_t ns_c, int lpc,
                                                     const int32_t *__restrict__ skip) {
  using LF = Lay<PF, DIM>;
  constexpr int PC = PF / 2, N1F = PF + 1, N1C = PC + 1;
  constexpr int NHF = LF::NH, CPB = LF::CPB, NHC = Lay<PC, DIM>::NH;
  __shared__ T sX[CPB * N1C * NHC];
  if (skip != nullptr && *skip) return;
  const int lc = threadIdx.x / NHF;
  const int t = threadIdx.x - lc * NHF;
  const int ci = blockIdx.x * CPB + lc;
  const bool active = ci < ncols;
  const int col = active ? ci : 0;
  const int hn = active ? nodes_f[col * NHF + t] : 0;
  const bool own = active && (flags_f[col * NHF + t] & kOwned);
  const bool cthr = active && t < NHC;
  const int hnc = cthr ? nodes_c[col * NHC + t] : 0;
  const int i = t % N1F, j = DIM == 3 ? t / N1F : 0;
  T *X = sX + lc * N1C * NHC;
  // the coarse values of layer l + 1 and the fine values of layer l are loaded before they are
  // needed, so the loads overlap the barrier and the contractions
  T xn[N1C];
  auto load_coarse = [&](int l) {
#pragma unroll
    for (int c = 0; c < N1C; ++c) xn[c] = cthr ? xc[(int64_t)(l * PC + c) * ns_c + hnc] : T(0);
  };
  const int l0 = blockIdx.y * lpc, l1 = min(l0 + lpc, nz);
  load_coarse(l0);
  for (int l = l0; l < l1; ++l) {
    const int kend = (l == nz - 1) ? N1F : PF;
    T old[N1F];
#pragma unroll
    for (int k = 0; k < N1F; ++k) old[k] = (own && k < kend) ? xf[(int64_t)(l * PF + k) * ns_f + hn] : T(0);
    if (cthr) {
#pragma unroll
      for (int c = 0; c < N1C; ++c) X[c * NHC + t] = xn[c];
    }
    if (l + 1 < l1) load_coarse(l + 1);
    __syncthreads();
    if (own) {
      T w[N1C];
#pragma unroll
      for (int c = 0; c < N1C; ++c) {
        T acc = T(0);
#pragma unroll
        for (int b = 0; b < (DIM == 3 ? N1C : 1); ++b) {
          T inner = T(0);
#pragma unroll
          for (int a = 0; a < N1C; ++a) inner += ip<T>(PF, i * N1C + a) * X[c * NHC + b * N1C + a];
          acc += (DIM == 3 ? ip<T>(PF, j * N1C + b) : T(1)) * inner;
        }
        w[c] = acc;
      }
#pragma unroll
      for (int k = 0; k < N1F; ++k) {
        if (k < kend) {
          T u = T(0);
#pragma unroll
          for (int c = 0; c < N1C; ++c) u += ip<T>(PF, k * N1C + c) * w[c];
          xf[(int64_t)(l * PF + k) * ns_f + hn] = old[k] + u;
        }
      }
    }
    __syncthreads();
  }
}

// ---- vector kernels (grid-stride, fixed grid, deterministic partials) -----------------------

#define GRID_STRIDE(i, n) \
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// The smoothing kernels below read operator products (and restricted right-hand sides) as the
// apply's first pass (the restriction) left them and add the face slots themselves (deferred.h).

template <typename T>
struct L1 { T a; };
template <typename T>
struct L2 { T a, b; };
template <typename T>
struct L3 { T a, b, c; };
template <typename T>
struct L4 { T a, b, c, d; };

// ---- the degree-1 level as an assembled operator ---------------------------------------------
//
// The hierarchy ends in kMgCoarseSteps Chebyshev steps on the degree-1 level, which is small (8,000
// unknowns for the wave of 40 x 40 x 4, p = 5): two launches a step, of 4.1 and 2.9 us, were a third
// of a solve there.  Assembled after every geometry update (27 entries a row on regular meshes) a
// step is one launch, and levels of at most 1,024 unknowns take all steps in one workgroup.

// Entry of row (v, n) for its w-th neighbour on levels v - 1, v, v + 1 (blockIdx.y = w, .z = v): the
// sum over the columns that have both, and the two layers at v, of the element matrix entry
// sum_q f_q (B^T grad l_row).(B^T grad l_col), collocated at the element's vertices (weights 1,
// D = [[-1/2, 1/2], [-1/2, 1/2]]); grad l_row is nonzero only at points that share all but one
// index with the row.
template <int DIM, typename T>
__global__ __launch_bounds__(256) void k_p1_matrix(const double *__restrict__ cg, const double *__restrict__ hm,
                                                   int64_t hstride, const int32_t *__restrict__ ptr,
                                                   const int32_t *__restrict__ inc,
                                                   const uint8_t *__restrict__ map, int nz, int64_t n_s,
                                                   const double *__restrict__ sigma,
                                                   const double *__restrict__ half_ds, T *__restrict__ val) {
  constexpr int NH = DIM == 3 ? 4 : 2;
  const int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int w = blockIdx.y, v = blockIdx.z, nlev = gridDim.z;
  if (n >= n_s) return;
  double acc[3] = {0.0, 0.0, 0.0};
  const int pe = ptr[n + 1];
  for (int p = ptr[n]; p < pe; ++p) {
    const int o = inc[p], a = o % NH, ai = a & 1, aj = a >> 1;   // o = column NH + a
    int match = 0;                           // the column's nodes that are this neighbour
#pragma unroll
    for (int b = 0; b < NH; ++b) match |= (map[(int64_t)o * NH + b] == w ? 1 : 0) << b;
    for (; match != 0; match &= match - 1) {
      const int b = __ffs(match) - 1, bi = b & 1, bj = b >> 1;
#pragma unroll
      for (int c = 0; c < NH; ++c) {
        const int ci = c & 1, cj = c >> 1;
        const int64_t ho = o - a + c;
        const double H = cg[ho], Hx = cg[hstride + ho], hx = cg[2 * hstride + ho];
        double Hy = 0.0, hy = 0.0, A00 = hm[ho], A01 = 0.0, A10 = 0.0, A11 = 0.0, dJ;
        if constexpr (DIM == 3) {
          Hy = cg[3 * hstride + ho];
          hy = cg[4 * hstride + ho];
          A01 = hm[hstride + ho];
          A10 = hm[2 * hstride + ho];
          A11 = hm[3 * hstride + ho];
          dJ = hm[4 * hstride + ho];
        } else {
          dJ = hm[hstride + ho];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {        // the row's place in layer l: its bottom or its top
          const int l = v - k;
          if (l < 0 || l >= nz) continue;
          const double zz = half_ds[l] * H, izz = 1.0 / zz, f = dJ * zz;
#pragma unroll
          for (int kq = 0; kq < 2; ++kq) {
            const double sg = sigma[l + kq], zx = sg * Hx - hx, zy = sg * Hy - hy;
            const double bx = -(zx * A00 + zy * A10) * izz, by = -(zx * A01 + zy * A11) * izz;
            const double ri = cj == aj && kq == k ? (ai ? 0.5 : -0.5) : 0.0;
            const double rj = DIM == 3 && ci == ai && kq == k ? (aj ? 0.5 : -0.5) : 0.0;
            const double rk = c == a ? (k ? 0.5 : -0.5) : 0.0;
            const double gx = A00 * ri + A10 * rj + bx * rk, gy = A01 * ri + A11 * rj + by * rk, gz = izz * rk;
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2) {
              const double ti = cj == bj && kq == k2 ? (bi ? 0.5 : -0.5) : 0.0;
              const double tj = DIM == 3 && ci == bi && kq == k2 ? (bj ? 0.5 : -0.5) : 0.0;
              const double tk = c == b ? (k2 ? 0.5 : -0.5) : 0.0;
              const double hx2 = A00 * ti + A10 * tj + bx * tk, hy2 = A01 * ti + A11 * tj + by * tk, hz2 = izz * tk;
              acc[k2 - k + 1] += f * (gx * hx2 + gy * hy2 + gz * hz2);
            }
          }
        }
      }
    }
  }
  const int64_t plane = (int64_t)nlev * n_s, i = (int64_t)v * n_s + n;
#pragma unroll
  for (int dv = 0; dv < 3; ++dv) val[(dv * (int64_t)gridDim.y + w) * plane + i] = (T)acc[dv];
}

// One Chebyshev step with it: q = A d, r -= q, d' = c1 d + c2 dinv r, x += d' (d' apart from d, which
// other rows still read).  W > 0: the number of neighbours as a constant.
template <int W, typename T>
__global__ __launch_bounds__(256) void k_p1_step(const T *__restrict__ val, const int32_t *__restrict__ nb, int wn,
                                                 T *__restrict__ r, const T *__restrict__ d, T *__restrict__ dn,
                                                 T *__restrict__ x, const T *__restrict__ dinv,
                                                 const double *__restrict__ cf, int k, int64_t n_s, int nlev,
                                                 const int32_t *__restrict__ skip) {
  const int done = skip != nullptr ? *skip : 0;
  const T c1 = (T)cf[3 + 2 * (k - 2)], c2 = (T)cf[4 + 2 * (k - 2)];
  const int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int v = blockIdx.y;
  if (n >= n_s) return;
  const int64_t i = v * n_s + n, plane = (int64_t)nlev * n_s;
  const int64_t vm = v > 0 ? -n_s : 0, vp = v < nlev - 1 ? n_s : 0;   // the entries there are zero
  const T ri = r[i], xi = x[i], di = d[i], iv = dinv[i];
  T q = T(0);
  auto entry = [&](int w, int wt) {
    const int64_t j = v * n_s + nb[w * n_s + n];
    q += val[w * plane + i] * d[j + vm] + val[(wt + w) * plane + i] * d[j] + val[(2 * wt + w) * plane + i] * d[j + vp];
  };
  if constexpr (W > 0) {
#pragma unroll
    for (int w = 0; w < W; ++w) entry(w, W);
  } else {
    for (int w = 0; w < wn; ++w) entry(w, wn);
  }
  asm volatile("" ::: "memory");   // the loads stay ahead of the test
  if (done) return;
  const T rn = ri - q;
  const T dd = c1 * di + c2 * iv * rn;
  r[i] = rn;
  dn[i] = dd;
  x[i] = xi + dd;
}

// All steps, from x = 0, in one workgroup for a level of at most kP1One unknowns: a thread keeps its
// row of the matrix in registers, d goes through LDS.
constexpr int kP1One = 1024;
template <int W, typename T>
__global__ __launch_bounds__(kP1One) void k_p1_all(Deferred<T> b, T *x, const T *__restrict__ val,
                                                   const int32_t *__restrict__ nb, const T *__restrict__ dinv,
                                                   const double *__restrict__ cf, int n_s, int nlev,
                                                   const int32_t *__restrict__ skip) {
  __shared__ T sd[kP1One];
  const int done = skip != nullptr ? *skip : 0;
  const int i = threadIdx.x, v = i / n_s, n = i - v * n_s;
  const bool act = v < nlev;
  const int plane = nlev * n_s;
  T a[3][W], iv = T(0), bi = T(0);
  int j[W];
  const int vm = v > 0 ? -n_s : 0, vp = v < nlev - 1 ? n_s : 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    j[w] = act ? v * n_s + nb[w * n_s + n] : 0;
#pragma unroll
    for (int dv = 0; dv < 3; ++dv) a[dv][w] = act ? val[(dv * W + w) * plane + i] : T(0);
  }
  if (act) {
    iv = dinv[i];
    bi = gather_one(b, i, n, n_s, v);
  }
  if (done) return;
  T r = bi, d = (T)cf[0] * iv * bi, xi = d;
  for (int k = 2; k <= kMgCoarseSteps; ++k) {
    sd[i] = d;
    __syncthreads();
    T q = T(0);
    if (act) {
#pragma unroll
      for (int w = 0; w < W; ++w) q += a[0][w] * sd[j[w] + vm] + a[1][w] * sd[j[w]] + a[2][w] * sd[j[w] + vp];
    }
    r -= q;
    d = (T)cf[3 + 2 * (k - 2)] * d + (T)cf[4 + 2 * (k - 2)] * iv * r;
    xi += d;
    __syncthreads();
  }
  if (act) x[i] = xi;
}

// first Chebyshev step from x = 0: r = b, d = c dinv b, x = d; a deferred b is completed in bw
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_cheb0(Deferred<T> b, T *bw, T *r, T *d, T *x, const T *dinv,
                                                       const double *cf, int64_t n_s, const int32_t *skip) {
  const T c = (T)cf[0];
  for_nodes<LV>(b, n_s, skip, [&](int64_t i) { return L1<T>{dinv[i]}; },
            [&](int64_t i, const L1<T> &l, T bi) {
              const T di = c * l.a * bi;
              if (bw != nullptr) bw[i] = bi;
              r[i] = bi;
              d[i] = di;
              x[i] = di;
            });
}

// first Chebyshev step from x: r = b - q (q = A x), d = c dinv r, x += d
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_cheb1(const T *b, Deferred<T> q, T *r, T *d, T *x, const T *dinv,
                                                       const double *cf, int64_t n_s, const int32_t *skip) {
  const T c = (T)cf[0];
  for_nodes<LV>(q, n_s, skip, [&](int64_t i) { return L3<T>{b[i], dinv[i], x[i]}; },
            [&](int64_t i, const L3<T> &l, T qi) {
              const T ri = l.a - qi;
              const T di = c * l.b * ri;
              r[i] = ri;
              d[i] = di;
              x[i] = l.c + di;
            });
}

// later steps: r -= q (q = A d), d = c1 d + c2 dinv r, x += d
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_cheb_step(T *r, Deferred<T> q, T *d, T *x, const T *dinv,
                                                           const double *cf, int k, int64_t n_s,
                                                           const int32_t *skip) {
  const T c1 = (T)cf[3 + 2 * (k - 2)], c2 = (T)cf[4 + 2 * (k - 2)];
  for_nodes<LV>(q, n_s, skip, [&](int64_t i) { return L4<T>{r[i], d[i], dinv[i], x[i]}; },
            [&](int64_t i, const L4<T> &l, T qi) {
              const T ri = l.a - qi;
              const T di = c1 * l.b + c2 * l.c * ri;
              r[i] = ri;
              d[i] = di;
              x[i] = l.d + di;
            });
}

// Two-step smoothing written out (the default degree): with d1 = c0 D^-1 r0 and
// d2 = c1 d1 + c2 D^-1 (r0 - A d1), x2 = x0 + a1 d1 + a2 D^-1 (r0 - A d1) (a1 = 1 + c1, a2 = c2)
// = x0 + D^-1 ((a1 c0 + a2) r0 - a2 A d1) = x0 + (a1 + a2 / c0) d1 - a2 D^-1 A d1: no residual or
// step vector survives it.
//   y = c dinv b; a deferred b is completed in bw
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_scale(T *y, Deferred<T> b, T *bw, const T *dinv, const double *cf,
                                                       int64_t n_s, const int32_t *skip) {
  const T c = (T)cf[0];
  for_nodes<LV>(b, n_s, skip, [&](int64_t i) { return L1<T>{dinv[i]}; },
            [&](int64_t i, const L1<T> &l, T bi) {
              if (bw != nullptr) bw[i] = bi;
              y[i] = c * l.a * bi;
            });
}

//   from zero: x = dinv ((a1 c0 + a2) b - a2 q), q = A d1
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_pre2(T *x, const T *b, Deferred<T> q, const T *dinv,
                                                      const double *cf, int64_t n_s, const int32_t *skip) {
  const T e = (T)(cf[1] * cf[0] + cf[2]), a2 = (T)cf[2];
  for_nodes<LV>(q, n_s, skip, [&](int64_t i) { return L2<T>{b[i], dinv[i]}; },
            [&](int64_t i, const L2<T> &l, T qi) { x[i] = l.b * (e * l.a - a2 * qi); });
}

//   from x: d1 = c dinv (b - q1), q1 = A x
template <int LV, typename T>
__global__ __launch_bounds__(kVecThreads) void k_post2a(T *d, const T *b, Deferred<T> q1, const T *dinv,
                                                        const double *cf, int64_t n_s, const int32_t *skip) {
  const T c = (T)cf[0];
  for_nodes<LV>(q1, n_s, skip, [&](int64_t i) { return L2<T>{b[i], dinv[i]}; },
            [&](int64_t i, const L2<T> &l, T qi) { d[i] = c * l.b * (l.a - qi); });
}

//   x += (a1 + a2 / c0) d1 - a2 dinv q2, q2 = A d1 (without b - q1, so q1 needs no assembly in memory)
// DOT: also the block partials of b.x (the CG's r.z when b is the residual and x the V-cycle's
// result)
template <int LV, typename T, bool DOT>
__global__ __launch_bounds__(kVecThreads) void k_post2b(T *x, const T *b, const T *d, Deferred<T> q2,
                                                        const T *dinv, const double *cf, int64_t n_s,
                                                        const int32_t *skip, double *partial) {
  const T e = (T)(cf[1] + cf[2] / cf[0]), a2 = (T)cf[2];
  const int dn = skip != nullptr ? *skip : 0;
  double v[1] = {0.0};
  for_nodes<LV>(q2, n_s, [&](int64_t i) { return L4<T>{x[i], d[i], dinv[i], DOT ? b[i] : T(0)}; },
            [&] { return dn == 0; },
            [&](int64_t i, const L4<T> &l, T qi) {
              const T xi = l.a + (e * l.b - a2 * l.c * qi);
              x[i] = xi;
              if constexpr (DOT) v[0] += (double)l.d * (double)xi;
            });
  if constexpr (DOT) {
    if (dn == 0) block_partials<1>(v, partial);
  }
}

// PCG with a general preconditioner: x += alpha p, r -= alpha q; partial r.r.  SCALE: also the
// first step of the degree-2 V-cycle that follows on the new residual, d = c0 dinv r.  np > 0: alpha
// from the np partials of p.q (cg_alpha), else as k_fin_pq left it.
template <int LV, typename T, bool SCALE>
__global__ __launch_bounds__(kVecThreads, LV == 1 ? 8 : 1) void k_mg_update(T *x, T *r, const T *p, Deferred<T> q, int64_t n_s,
                                                           double *partial, PcgScalars *sc, T *d, const T *dinv,
                                                           const double *cf, const double *pq, int np) {
  const T c0 = SCALE ? (T)cf[0] : T(0);
  const int dn = sc->done;
  const double rz = sc->rz2;
  double alpha = sc->alpha;
  const PartialLoads<1> pv(pq, np);
  bool live = dn == 0;
  T a = T(0);
  double v[1] = {0.0};
  for_nodes<LV>(q, n_s, [&](int64_t i) { return L4<T>{x[i], r[i], p[i], SCALE ? dinv[i] : T(0)}; },
            [&] {
              if (np > 0) live = cg_alpha(pv, dn != 0, rz, sc, alpha);
              a = (T)alpha;
              return live;
            },
            [&](int64_t i, const L4<T> &l, T qi) {
              x[i] = l.a + a * l.c;
              const T ri = l.b - a * qi;
              r[i] = ri;
              if constexpr (SCALE) d[i] = c0 * l.d * ri;
              v[0] += (double)ri * (double)ri;
            });
  if (!live) return;
  block_partials<1>(v, partial);
}

__global__ __launch_bounds__(kVecThreads) void k_mg_fin_rr(const double *partial, int np, PcgScalars *sc) {
  if (sc->done) return;
  double s[1];
  final_sums<1>(partial, np, s);
  if (threadIdx.x == 0) {
    sc->rr = s[0];
    sc->iters += 1;
    if (!(s[0] == s[0]) || !(s[0] <= 1e300)) {
      sc->breakdown = 2;
      sc->done = 1;
    } else if (s[0] <= sc->tol2) {
      sc->done = 1;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_dot(const T *a, const T *b, int64_t n, double *partial,
                                                     const PcgScalars *sc) {
  if (sc->done) return;
  double v[1] = {0.0};
  GRID_STRIDE(i, n) v[0] += (double)a[i] * (double)b[i];
  block_partials<1>(v, partial);
}

// a non-positive r.z means the preconditioner is not positive definite on this residual
__device__ __forceinline__ void cg_store_rz(PcgScalars *sc, double rz) {
  sc->rz2 = rz;
  if (!(rz > 0.0) || !(rz <= 1e300)) {
    sc->breakdown = (rz == rz) ? 1 : 2;
    sc->done = 1;
  }
}

// p = z + beta p, beta = (r.z)_new / (r.z)_old (first: 0) from the np partials of r.z (every block sums them; the first one stores what
// the next kernels read).
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_mg_dir(T *p, const T *z, int64_t n, PcgScalars *sc, int first,
                                                        const double *partial, int np) {
  const int dn = sc->done;
  const double rz = sc->rz;
  const PartialLoads<1> pv(partial, np);
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  T z0 = T(0), p0 = T(0);
  if (i < n) {
    z0 = z[i];
    if (!first) p0 = p[i];
  }
  asm volatile("" ::: "memory");   // the first loads stay ahead of the test
  double s[1];
  if (pv.sums(s, dn != 0)) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) cg_store_rz(sc, s[0]);
  const T b = first ? T(0) : (T)(s[0] / rz);
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += st) {
    const int64_t i2 = i + st;
    T z1 = T(0), p1 = T(0);
    if (i2 < n) {
      z1 = z[i2];
      if (!first) p1 = p[i2];
    }
    p[i] = first ? z0 : z0 + b * p0;
    z0 = z1;
    p0 = p1;
  }
}

// Largest eigenvalue of D^-1 A.  D^-1 A is self-adjoint in <u, v>_D = sum u_i v_i / dinv_i over
// the unknowns (dinv = 0 on the Dirichlet rows, which take no part), so Lanczos in that inner
// product gives a symmetric tridiagonal matrix whose largest eigenvalue approaches lambda_max
// from below.  The top of this spectrum is clustered (element-local modes), where Lanczos needs
// far fewer products than the power iteration's Rayleigh quotient.

// v = fixed start vector on the unknowns, vp = 0; partials of <v, v>_D
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_lz_start(T *v, T *vp, const T *dinv, int64_t n, double *partial) {
  double s[1] = {0.0};
  GRID_STRIDE(i, n) {
    const T d = dinv[i];
    const T vi = d != T(0) ? T(1.0 + 0.5 * sin(0.7 * (double)i) + 0.25 * cos(0.013 * (double)i)) : T(0);
    v[i] = vi;
    vp[i] = T(0);
    if (d != T(0)) s[0] += (double)vi * (double)vi / (double)d;
  }
  block_partials<1>(s, partial);
}

// out = sum (mode 0) or its square root (mode 1), set to 0 when it is below rel^2 * ref^2
// (an invariant subspace: the recurrence then produces zeros, which add zero Ritz values only)
__global__ __launch_bounds__(kVecThreads) void k_lz_fin(const double *partial, int np, double *out, int mode,
                                                        const double *ref, double rel) {
  double s[1];
  final_sums<1>(partial, np, s);
  if (threadIdx.x == 0) {
    double v = s[0];
    if (mode == 1) {
      const double r = ref != nullptr ? fabs(*ref) : 0.0;
      v = (v > 0.0 && v > rel * rel * r * r) ? sqrt(v) : 0.0;
    }
    *out = v;
  }
}

// w = dinv q - alpha v - beta_prev vp, stored in vp; partials of <w, w>_D
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_lz_w(T *vp, const T *v, const T *q, const T *dinv, int64_t n,
                                                      const double *alpha, const double *beta_prev,
                                                      double *partial) {
  const T a = (T)*alpha, b = beta_prev != nullptr ? (T)*beta_prev : T(0);
  double s[1] = {0.0};
  GRID_STRIDE(i, n) {
    const T d = dinv[i];
    const T w = d * q[i] - a * v[i] - b * vp[i];
    vp[i] = w;
    if (d != T(0)) s[0] += (double)w * (double)w / (double)d;
  }
  block_partials<1>(s, partial);
}

// partials of a.b
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_lz_dot(const T *a, const T *b, int64_t n, double *partial) {
  double s[1] = {0.0};
  GRID_STRIDE(i, n) s[0] += (double)a[i] * (double)b[i];
  block_partials<1>(s, partial);
}

// v /= beta (0 when beta is 0)
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_lz_scale(T *v, int64_t n, const double *beta) {
  const T f = *beta > 0.0 ? (T)(1.0 / *beta) : T(0);
  GRID_STRIDE(i, n) v[i] *= f;
}

// u = y_j v (first) or u += y_j v
template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_lz_acc(T *u, const T *v, int64_t n, double y, int first) {
  const T c = (T)y;
  GRID_STRIDE(i, n) u[i] = first ? c * v[i] : u[i] + c * v[i];
}

// power iteration on D^-1 A: pw[0] = (v.Av)/(v.Dv) (Rayleigh quotient), pw[1] = 1/sqrt(v.Dv)

template <typename T>
__global__ __launch_bounds__(kVecThreads) void k_pow_dots(const T *v, const T *q, const T *dinv, int64_t n,
                                                          double *partial) {
  double s[2] = {0.0, 0.0};
  GRID_STRIDE(i, n) {
    const double vi = (double)v[i];
    s[0] += vi * (double)q[i];
    if (dinv[i] != T(0)) s[1] += vi * vi / (double)dinv[i];
  }
  block_partials<2>(s, partial);
}

__global__ __launch_bounds__(kVecThreads) void k_pow_fin(const double *partial, int np, double *pw) {
  double s[2];
  final_sums<2>(partial, np, s);
  if (threadIdx.x == 0) {
    pw[0] = s[1] > 0.0 ? s[0] / s[1] : 0.0;
    pw[1] = s[1] > 0.0 ? 1.0 / sqrt(s[1]) : 1.0;
  }
}

template <typename T>
__global__ void k_pow_next(T *v, const T *q, const T *dinv, int64_t n, const double *pw) {
  const T sc = (T)pw[1];
  GRID_STRIDE(i, n) v[i] = dinv[i] * q[i] * sc;
}

// ---- host side --------------------------------------------------------------------------------

template <typename T>
struct Prec;
template <>
struct Prec<double> {
  static constexpr fnpf_dtype dt = FNPF_F64;
  static double *const *lv(MgLevel &L) { return L.v64; }
  static double *const *fv(Ctx &c) { return c.mg_f64; }
  static const double *dinv(Ctx &c) { return c.d_dinv; }
  static bool &stale(Ctx &c) { return c.mg_stale64; }
  static double *&ev(MgLevel &L) { return L.ev64; }
  static double *&evf(Ctx &c) { return c.mg_ev64; }
  static bool &evok(MgLevel &L) { return L.ev_ok64; }
  static bool &evokf(Ctx &c) { return c.mg_ev_ok64; }
};
template <>
struct Prec<float> {
  static constexpr fnpf_dtype dt = FNPF_F32;
  static float *const *lv(MgLevel &L) { return L.v32; }
  static float *const *fv(Ctx &c) { return c.mg_f32; }
  static const float *dinv(Ctx &c) { return c.d_dinv32; }
  static bool &stale(Ctx &c) { return c.mg_stale32; }
  static float *&ev(MgLevel &L) { return L.ev32; }
  static float *&evf(Ctx &c) { return c.mg_ev32; }
  static bool &evok(MgLevel &L) { return L.ev_ok32; }
  static bool &evokf(Ctx &c) { return c.mg_ev_ok32; }
};

// n elements in *p, unless it has them (an earlier call may have failed half way)
template <typename T>
hipError_t dalloc_t(T **p, size_t n) {
  if (*p != nullptr) return hipSuccess;
  const hipError_t e = hipMalloc((void **)p, n * sizeof(T));
  if (e != hipSuccess) *p = nullptr;
  return e;
}

#define MG_DISPATCH(DIMV, PV, CALL)                    \
  switch (PV) {                                        \
    case 2: { constexpr int PF_ = 2; CALL; } break;    \
    case 3: { constexpr int PF_ = 3; CALL; } break;    \
    case 4: { constexpr int PF_ = 4; CALL; } break;    \
    case 5: { constexpr int PF_ = 5; CALL; } break;    \
    case 6: { constexpr int PF_ = 6; CALL; } break;    \
    case 7: { constexpr int PF_ = 7; CALL; } break;    \
    case 8: { constexpr int PF_ = 8; CALL; } break;    \
    default: return hipErrorInvalidValue;              \
  }

// layers per block of the transfers: the finer level's, and at most as many chunks as the coarse
// level's face buffer has room for
int transfer_lpc(const Ctx &F, const Ctx &C) { return std::max(F.lpc, C.lpc); }

template <int PF, int DIM, typename T>
hipError_t restrict_impl(Ctx &F, Ctx &C, const T *rf, const Deferred<T> &qf, T *bc, T *Fc, const int32_t *skip,
                         hipStream_t s) {
  using LF = Lay<PF, DIM>;
  const int lpc = transfer_lpc(F, C);
  const dim3 nb((F.n_eh + LF::CPB - 1) / LF::CPB, (F.nz + lpc - 1) / lpc);
  k_restrict<PF, DIM, T><<<nb, LF::NT, 0, s>>>(rf, qf, bc, Fc, F.d_eh_nodes, F.d_flags, C.d_eh_nodes, C.d_flags,
                                               C.d_slot, F.n_eh, F.nz, F.n_s, C.n_s, C.n_slots, lpc, skip);
  return hipGetLastError();
}

template <int PF, int DIM, typename T>
hipError_t prolong_impl(Ctx &F, Ctx &C, const T *xc, T *xf, const int32_t *skip, hipStream_t s) {
  using LF = Lay<PF, DIM>;
  const int lpc = transfer_lpc(F, C);
  const dim3 nb((F.n_eh + LF::CPB - 1) / LF::CPB, (F.nz + lpc - 1) / lpc);
  k_prolong_add<PF, DIM, T><<<nb, LF::NT, 0, s>>>(xc, xf, F.d_eh_nodes, F.d_flags, C.d_eh_nodes, F.n_eh, F.nz,
                                                  F.n_s, C.n_s, lpc, skip);
  return hipGetLastError();
}

template <int PF, int DIM>
hipError_t surf_impl(Ctx &F, Ctx &C, double *Hc, double *hc, hipStream_t s) {
  constexpr int NHC = Lay<PF / 2, DIM>::NH;
  const int64_t nthr = (int64_t)F.n_eh * NHC;
  k_mg_surf<PF, DIM><<<(unsigned)((nthr + 255) / 256), 256, 0, s>>>(F.d_geoH, F.d_geoh, F.d_eh_nodes, C.d_eh_nodes,
                                                                     C.d_flags, F.n_eh, Hc, hc);
  return hipGetLastError();
}

// b_c = P^T (r_f - A x), its assembly left to the reader (q: work vector for A x)
template <typename T>
hipError_t restrict_to(Ctx &F, Ctx &C, const T *rf, const T *x, T *q, T *bc, Deferred<T> &out, const int32_t *skip,
                       hipStream_t s) {
  T *Fc = face_buffer<T>(C);
  const int lpc = transfer_lpc(F, C);
  hipError_t er;
  if (apply_restrict_active(F))
    er = launch_apply_restrict(F, C, Prec<T>::dt, x, rf, bc, Fc, lpc, skip, s);
  else
    er = launch_apply(F, Prec<T>::dt, x, q, true, nullptr, skip, s, nullptr, true);
  if (er != hipSuccess) return er;
  const Deferred<T> qf = apply_result<T>(F, q);
  if (!apply_restrict_active(F)) {
    if (F.dim == 3) {
      MG_DISPATCH(3, F.p, { hipError_t e = (restrict_impl<PF_, 3, T>(F, C, rf, qf, bc, Fc, skip, s)); if (e != hipSuccess) return e; });
    } else {
      MG_DISPATCH(2, F.p, { hipError_t e = (restrict_impl<PF_, 2, T>(F, C, rf, qf, bc, Fc, skip, s)); if (e != hipSuccess) return e; });
    }
  }
  out = complete<T>(C, bc);
  out.F = Fc;
  out.slots = C.d_p_slots;
  out.lists = C.d_p_lists;
  out.n_hi = C.p_n_hi;
  out.n_slots = C.n_slots;
  out.vend = out.nlev - 1;
  out.clev = lpc * C.p;
  out.nchunk = (F.nz + lpc - 1) / lpc;
  return hipSuccess;
}

template <typename T>
hipError_t prolong_to(Ctx &F, Ctx &C, const T *xc, T *xf, const int32_t *skip, hipStream_t s) {
  if (F.dim == 3) {
    MG_DISPATCH(3, F.p, return (prolong_impl<PF_, 3, T>(F, C, xc, xf, skip, s)));
  } else {
    MG_DISPATCH(2, F.p, return (prolong_impl<PF_, 2, T>(F, C, xc, xf, skip, s)));
  }
  return hipSuccess;
}

hipError_t surf_to(Ctx &F, Ctx &C, double *Hc, double *hc, hipStream_t s) {
  if (F.dim == 3) {
    MG_DISPATCH(3, F.p, return (surf_impl<PF_, 3>(F, C, Hc, hc, s)));
  } else {
    MG_DISPATCH(2, F.p, return (surf_impl<PF_, 2>(F, C, Hc, hc, s)));
  }
  return hipSuccess;
}

// Device table of the Chebyshev coefficients, kMgCoef doubles per (precision, level): [0] 1/theta,
// [1] 1 + c1_2 and [2] c2_2 (closed-form degree 2), then (c1_k, c2_k) for steps k = 2 .. 10 of the
// three-term recurrence on [lmax / ratio, lmax], lmax = 1.1 lam.  Kernels read it from device
// memory, so captured iteration graphs stay valid when the estimates change.
template <typename T>
const double *coef_table(Ctx &c, int l) {
  return c.d_mgc + ((sizeof(T) == 8 ? 0 : 1) * (int)(c.mg.size() + 1) + l) * kMgCoef;
}

__host__ __device__ void chebyshev_coefficients(double lam, double ratio, double *cf) {
  const double lmax = kMgSafety * lam, lmin = lmax / ratio;
  const double theta = 0.5 * (lmax + lmin), delta = 0.5 * (lmax - lmin), sigma = theta / delta;
  for (int k = 0; k < kMgCoef; ++k) cf[k] = 0.0;
  cf[0] = 1.0 / theta;
  double rho0 = 1.0 / sigma;
  for (int k = 2; k <= kMgCoarseSteps; ++k) {
    const double rho1 = 1.0 / (2.0 * sigma - rho0);
    cf[3 + 2 * (k - 2)] = rho1 * rho0;
    cf[4 + 2 * (k - 2)] = 2.0 * rho1 / delta;
    if (k == 2) {
      cf[1] = 1.0 + rho1 * rho0;
      cf[2] = 2.0 * rho1 / delta;
    }
    rho0 = rho1;
  }
}

// The table of one level from its eigenvalue estimate *lam on the device, so that a geometry update
// needs no host round trip; lam_out keeps the estimate.  A non-positive or non-finite estimate
// gives a NaN table, which the solve then reports as a non-finite residual.
__global__ void k_cheb_coef(const double *lam, double ratio, double *cf, double *lam_out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double l = *lam;
  *lam_out = l;
  if (l > 0.0 && l <= 1e300) {
    chebyshev_coefficients(l, ratio, cf);
  } else {
    for (int k = 0; k < kMgCoef; ++k) cf[k] = __builtin_nan("");
  }
}

__global__ void k_set_scalar(double *p, double v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// blocks of the (level, node) kernels that write partials
template <typename T>
int partial_blocks(const Ctx &L) {
  return node_blocks(L, node_levels(L), node_levels(L) > 1 ? kNodeBlocks : kVB<T>);
}

// Chebyshev smoothing of A x = b on level L (D^-1 A spectrum estimate lam), m steps.  From zero:
// x = p(D^-1 A) D^-1 b; otherwise x += p(D^-1 A) D^-1 (b - A x).  On return r = b - A x_{m-1}
// and d = x_m - x_{m-1}.  A deferred b (from zero only) is completed in place.
// line: B^-1 (the level's vertical line blocks, line_smoother.hip) in place of D^-1.
template <typename T>
hipError_t smooth(Ctx &L, const Deferred<T> &b, T *x, T *r, T *d, T *q, const double *cf, int m, bool from_zero,
                  const int32_t *skip, hipStream_t s, bool line = false) {
  const int64_t ns = L.n_s;
  const int nlv = node_levels(L), nb = node_blocks(L, nlv);
  T *bw = b.F != nullptr ? const_cast<T *>(b.y) : nullptr;
  if (line) {
    hipError_t e = hipSuccess;
    if (from_zero) {
      // the line solves read complete vectors: complete b first (r = b, the rest is overwritten)
      if (b.F != nullptr) with_levels(nlv, [&](auto lv) { k_cheb0<lv(), T><<<nb, kVecThreads, 0, s>>>(b, bw, r, d, x, Prec<T>::dinv(L), cf, ns, skip); });
      e = line_cheb0<T>(L, b.y, r, d, x, cf, skip, s);
    } else {
      if ((e = launch_apply(L, Prec<T>::dt, x, q, true, nullptr, skip, s)) != hipSuccess) return e;
      e = line_cheb1<T>(L, b.y, q, r, d, x, cf, skip, s);
    }
    for (int k = 2; k <= m && e == hipSuccess; ++k) {
      if ((e = launch_apply(L, Prec<T>::dt, d, q, true, nullptr, skip, s)) != hipSuccess) return e;
      e = line_chebk<T>(L, q, r, d, x, cf, k, skip, s);
    }
    return e;
  }
  const T *dinv = Prec<T>::dinv(L);
  if (from_zero) {
    with_levels(nlv, [&](auto lv) { k_cheb0<lv(), T><<<nb, kVecThreads, 0, s>>>(b, bw, r, d, x, dinv, cf, ns, skip); });
  } else {
    hipError_t e = launch_apply(L, Prec<T>::dt, x, q, true, nullptr, skip, s, nullptr, true);
    if (e != hipSuccess) return e;
    with_levels(nlv, [&](auto lv) { k_cheb1<lv(), T><<<nb, kVecThreads, 0, s>>>(b.y, apply_result<T>(L, q), r, d, x, dinv, cf, ns, skip); });
  }
  for (int k = 2; k <= m; ++k) {
    hipError_t e = launch_apply(L, Prec<T>::dt, d, q, true, nullptr, skip, s, nullptr, true);
    if (e != hipSuccess) return e;
    with_levels(nlv, [&](auto lv) { k_cheb_step<lv(), T><<<nb, kVecThreads, 0, s>>>(r, apply_result<T>(L, q), d, x, dinv, cf, k, ns, skip); });
  }
  return hipGetLastError();
}

template <typename T>
T *&p1_values(Ctx &c);
template <>
double *&p1_values<double>(Ctx &c) { return c.d_p1_val64; }
template <>
float *&p1_values<float>(Ctx &c) { return c.d_p1_val32; }

// Levels whose assembled operator stays within the 256 MB cache with room to spare: a row is read
// whole at every step (216 bytes in FP64), so beyond it the matrix-free apply moves less.
constexpr size_t kP1MaxBytes = size_t(96) << 20;

// Rows are padded with zero entries to a width that the kernels know at compile time, so that all
// loads of a row are in flight together: slices, quadrilaterals four to a node, five and six to a
// node.  On the tank around a cylinder (2,922 x 5 rows, at most 11 neighbours) a step takes 4.4 us,
// with the width as an argument 6.2 us.
constexpr int kP1Widths[] = {3, 9, 11, 13};
static size_t p1_width(size_t w) {
  for (const int k : kP1Widths)
    if (w <= (size_t)k) return k;
  return w;
}
template <typename F>
void with_p1_width(int w, F f) {
  switch (w) {
    case 3: f(std::integral_constant<int, 3>()); break;
    case 9: f(std::integral_constant<int, 9>()); break;
    case 11: f(std::integral_constant<int, 11>()); break;
    case 13: f(std::integral_constant<int, 13>()); break;
    default: f(std::integral_constant<int, 0>()); break;
  }
}

// Neighbour lists of a degree-1 level (host, once).
fnpf_status p1_build(Ctx &c) {
  const int nh = c.nh;
  std::vector<std::vector<int32_t>> nb(c.n_s);
  std::vector<int32_t> ptr(c.n_s + 1, 0), inc;
  for (int32_t id : c.h_eh_nodes) ptr[id + 1]++;
  for (int64_t n = 0; n < c.n_s; ++n) {
    ptr[n + 1] += ptr[n];
    nb[n].push_back((int32_t)n);
  }
  inc.resize(c.h_eh_nodes.size());
  std::vector<int32_t> fill(ptr.begin(), ptr.end() - 1);
  std::vector<uint8_t> map(c.h_eh_nodes.size() * nh);
  size_t w = 1;
  for (size_t o = 0; o < c.h_eh_nodes.size(); ++o) {
    const int32_t n = c.h_eh_nodes[o];
    inc[fill[n]++] = (int32_t)o;
    for (int b = 0; b < nh; ++b) {
      const int32_t m = c.h_eh_nodes[o / nh * nh + b];
      const auto at = std::find(nb[n].begin(), nb[n].end(), m);
      const size_t k = at - nb[n].begin();
      if (at == nb[n].end()) nb[n].push_back(m);
      w = std::max(w, nb[n].size());
      if (k > 255) return FNPF_ERR_ARG;
      map[o * nh + b] = (uint8_t)k;
    }
  }
  w = p1_width(w);
  std::vector<int32_t> list(w * c.n_s);
  for (size_t k = 0; k < w; ++k)
    for (int64_t n = 0; n < c.n_s; ++n) list[k * c.n_s + n] = k < nb[n].size() ? nb[n][k] : (int32_t)n;
  auto up = [](auto **d, const auto &h) {
    if (dalloc_t(d, h.size()) != hipSuccess) return false;
    return hipMemcpy(*d, h.data(), h.size() * sizeof(h[0]), hipMemcpyHostToDevice) == hipSuccess;
  };
  if (!up(&c.d_p1_nb, list) || !up(&c.d_p1_ptr, ptr) || !up(&c.d_p1_inc, inc) || !up(&c.d_p1_map, map))
    return FNPF_ERR_ALLOC;
  c.p1_w = (int)w;
  return FNPF_OK;
}

// the assembled operator of the level's current geometry
template <typename T>
hipError_t p1_assemble(Ctx &c, hipStream_t s) {
  if (p1_values<T>(c) == nullptr) return hipSuccess;
  const int64_t hs = (int64_t)c.n_eh * c.nh;
  const dim3 nb((unsigned)((c.n_s + 255) / 256), c.p1_w, c.nz + 1);
  auto kern = c.dim == 3 ? k_p1_matrix<3, T> : k_p1_matrix<2, T>;
  kern<<<nb, 256, 0, s>>>(c.d_cg64, c.d_hm, hs, c.d_p1_ptr, c.d_p1_inc, c.d_p1_map, c.nz, c.n_s, c.d_sigma,
                          c.d_half_ds, p1_values<T>(c));
  return hipGetLastError();
}

// kMgCoarseSteps Chebyshev steps from zero with it (r, d, d2: work vectors)
template <typename T>
hipError_t p1_smooth(Ctx &L, const Deferred<T> &b, T *x, T *r, T *d, T *d2, const double *cf, const int32_t *skip,
                     hipStream_t s) {
  const T *dinv = Prec<T>::dinv(L), *val = p1_values<T>(L);
  const int nlev = L.nz + 1;
  if (L.n_v <= kP1One && L.p1_w <= kP1Widths[2]) {   // (13 entries in FP64 do not fit its registers)
    with_p1_width(L.p1_w, [&](auto w) {
      if constexpr (w() > 0 && w() <= kP1Widths[2])
        k_p1_all<w(), T><<<1, (unsigned)((L.n_v + 63) / 64 * 64), 0, s>>>(b, x, val, L.d_p1_nb, dinv, cf, (int)L.n_s,
                                                                          nlev, skip);
    });
    return hipGetLastError();
  }
  const int nlv = node_levels(L);
  with_levels(nlv, [&](auto lv) {
    k_cheb0<lv(), T><<<node_blocks(L, nlv), kVecThreads, 0, s>>>(b, nullptr, r, d, x, dinv, cf, L.n_s, skip);
  });
  const dim3 nb((unsigned)((L.n_s + 255) / 256), nlev);
  for (int k = 2; k <= kMgCoarseSteps; ++k) {
    with_p1_width(L.p1_w, [&](auto w) {
      k_p1_step<w(), T><<<nb, 256, 0, s>>>(val, L.d_p1_nb, L.p1_w, r, d, d2, x, dinv, cf, k, L.n_s, nlev, skip);
    });
    std::swap(d, d2);
  }
  return hipGetLastError();
}

// V-cycle on level l (0 = this context) for the right-hand side b (completed in place where it is
// deferred), result in x.
// pre_scaled (level 0, degree 2): d = c0 dinv b is already in place (k_mg_update<T, true>).
template <typename T>
hipError_t vcycle(Ctx &c, int l, const Deferred<T> &b, T *x, const int32_t *skip, int m, hipStream_t s,
                  double *dot_partial = nullptr, bool *dot_done = nullptr, bool pre_scaled = false) {
  Ctx &L = l == 0 ? c : *c.mg[l - 1].c;
  T *r, *d, *q;
  if (l == 0) {
    r = Prec<T>::fv(c)[1];
    d = Prec<T>::fv(c)[2];
    q = Prec<T>::fv(c)[3];
  } else {
    r = Prec<T>::lv(c.mg[l - 1])[2];
    d = Prec<T>::lv(c.mg[l - 1])[3];
    q = Prec<T>::lv(c.mg[l - 1])[4];
  }
  const double *cf = coef_table<T>(c, l);
  const int last = (int)c.mg.size();
  const bool line = c.mg_line;
  if (l == last && !line && p1_values<T>(L) != nullptr) return p1_smooth<T>(L, b, x, r, d, q, cf, skip, s);
  if (l == last) return smooth<T>(L, b, x, r, d, q, cf, kMgCoarseSteps, true, skip, s, line);
  MgLevel &C = c.mg[l];
  T *bc = Prec<T>::lv(C)[0], *xc = Prec<T>::lv(C)[1];
  const int64_t ns = L.n_s;
  const int nlv = node_levels(L), nb = node_blocks(L, nlv);
  const T *dinv = Prec<T>::dinv(L);
  Deferred<T> bd;
  hipError_t e = hipSuccess;
  // y = A v with the assembly left to the reader
  auto product = [&](const T *v, T *y) {
    return launch_apply(L, Prec<T>::dt, v, y, true, nullptr, skip, s, nullptr, true);
  };
  if (m == 2 && !line) {
    if (!(l == 0 && pre_scaled))
      with_levels(nlv, [&](auto lv) { k_scale<lv(), T><<<nb, kVecThreads, 0, s>>>(d, b, b.F != nullptr ? const_cast<T *>(b.y) : nullptr, dinv, cf, ns, skip); });
    if ((e = product(d, q)) != hipSuccess) return e;
    with_levels(nlv, [&](auto lv) { k_pre2<lv(), T><<<nb, kVecThreads, 0, s>>>(x, b.y, apply_result<T>(L, q), dinv, cf, ns, skip); });
    if ((e = restrict_to<T>(L, *C.c, b.y, x, q, bc, bd, skip, s)) != hipSuccess) return e;
    if ((e = vcycle<T>(c, l + 1, bd, xc, skip, m, s)) != hipSuccess) return e;
    if ((e = prolong_to<T>(L, *C.c, xc, x, skip, s)) != hipSuccess) return e;
    if ((e = product(x, q)) != hipSuccess) return e;
    with_levels(nlv, [&](auto lv) { k_post2a<lv(), T><<<nb, kVecThreads, 0, s>>>(d, b.y, apply_result<T>(L, q), dinv, cf, ns, skip); });
    if ((e = product(d, q)) != hipSuccess) return e;
    if (dot_partial != nullptr) {
      with_levels(nlv, [&](auto lv) { k_post2b<lv(), T, true><<<partial_blocks<T>(L), kVecThreads, 0, s>>>(x, b.y, d, apply_result<T>(L, q), dinv, cf, ns, skip, dot_partial); });
      if (dot_done) *dot_done = true;
    } else {
      with_levels(nlv, [&](auto lv) { k_post2b<lv(), T, false><<<nb, kVecThreads, 0, s>>>(x, b.y, d, apply_result<T>(L, q), dinv, cf, ns, skip, nullptr); });
    }
    return hipGetLastError();
  }
  e = smooth<T>(L, b, x, r, d, q, cf, m, true, skip, s, line);
  if (e != hipSuccess) return e;
  // residual of the smoothed x, r - A d, restricted directly
  e = restrict_to<T>(L, *C.c, r, d, q, bc, bd, skip, s);
  if (e != hipSuccess) return e;
  e = vcycle<T>(c, l + 1, bd, xc, skip, m, s);
  if (e != hipSuccess) return e;
  e = prolong_to<T>(L, *C.c, xc, x, skip, s);
  if (e != hipSuccess) return e;
  return smooth<T>(L, complete<T>(L, b.y), x, r, d, q, cf, m, false, skip, s, line);
}

// Eigenvalues and eigenvectors of a small symmetric matrix a[n][n] (row-major, destroyed) by
// cyclic Jacobi rotations: w[k] and column k of z[n][n].
void symmetric_eigen(int n, std::vector<double> &a, std::vector<double> &w, std::vector<double> &z) {
  z.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) z[(size_t)i * n + i] = 1.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) {
        const double x = a[(size_t)i * n + j] * a[(size_t)i * n + j];
        tot += x;
        if (i != j) off += x;
      }
    if (off <= 1e-30 * tot) break;
    for (int p = 0; p < n - 1; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = a[(size_t)p * n + q];
        if (apq == 0.0) continue;
        const double theta = (a[(size_t)q * n + q] - a[(size_t)p * n + p]) / (2.0 * apq);
        const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
        for (int k = 0; k < n; ++k) {   // columns p, q
          const double akp = a[(size_t)k * n + p], akq = a[(size_t)k * n + q];
          a[(size_t)k * n + p] = c * akp - sn * akq;
          a[(size_t)k * n + q] = sn * akp + c * akq;
        }
        for (int k = 0; k < n; ++k) {   // rows p, q
          const double apk = a[(size_t)p * n + k], aqk = a[(size_t)q * n + k];
          a[(size_t)p * n + k] = c * apk - sn * aqk;
          a[(size_t)q * n + k] = sn * apk + c * aqk;
        }
        for (int k = 0; k < n; ++k) {
          const double zkp = z[(size_t)k * n + p], zkq = z[(size_t)k * n + q];
          z[(size_t)k * n + p] = c * zkp - sn * zkq;
          z[(size_t)k * n + q] = sn * zkp + c * zkq;
        }
      }
  }
  w.resize(n);
  for (int i = 0; i < n; ++i) w[i] = a[(size_t)i * n + i];
}

// kLanczosSteps Lanczos steps on D^-1 A of level L from the fixed start vector (vectors v, vp, q);
// the largest Ritz value is the estimate, and a second pass over the same recurrence (its
// coefficients kept from the first) forms the Ritz vector in u for the later warm updates.
template <typename T>
hipError_t lanczos_lambda(Ctx &c, Ctx &L, T *u, T *v, T *vp, T *q, double &lam, hipStream_t s) {
  const T *dinv = Prec<T>::dinv(L);
  const int64_t n = L.n_v;
  constexpr int K = kLanczosSteps;
  double *al = c.d_mg_lz, *be = c.d_mg_lz + K, *nrm = c.d_mg_lz + 2 * K;
  const double rel = 1e-12;
  std::vector<double> y(K, 0.0);
  for (int pass = 0; pass < 2; ++pass) {
    T *a = v, *b = vp;
    k_lz_start<T><<<kVB<T>, kVecThreads, 0, s>>>(a, b, dinv, n, c.d_partial);
    k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, nrm, 1, nullptr, 0.0);
    k_lz_scale<T><<<kVB<T>, kVecThreads, 0, s>>>(a, n, nrm);
    for (int j = 0; j < K; ++j) {
      if (pass == 1) k_lz_acc<T><<<kVB<T>, kVecThreads, 0, s>>>(u, a, n, y[j], j == 0);
      if (pass == 1 && j == K - 1) break;
      hipError_t e = launch_apply(L, Prec<T>::dt, a, q, true, nullptr, nullptr, s);
      if (e != hipSuccess) return e;
      if (pass == 0) {
        k_lz_dot<T><<<kVB<T>, kVecThreads, 0, s>>>(a, q, n, c.d_partial);
        k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, al + j, 0, nullptr, 0.0);
      }
      k_lz_w<T><<<kVB<T>, kVecThreads, 0, s>>>(b, a, q, dinv, n, al + j, j > 0 ? be + j - 1 : nullptr,
                                                   c.d_partial);
      if (pass == 0) k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, be + j, 1, al + j, rel);
      k_lz_scale<T><<<kVB<T>, kVecThreads, 0, s>>>(b, n, be + j);
      std::swap(a, b);
    }
    if (pass == 0) {
      std::vector<double> h(2 * K);
      hipError_t e = hipMemcpyAsync(h.data(), c.d_mg_lz, sizeof(double) * 2 * K, hipMemcpyDeviceToHost, s);
      if (e != hipSuccess) return e;
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
      std::vector<double> t((size_t)K * K, 0.0), w, z;
      for (int j = 0; j < K; ++j) {
        t[(size_t)j * K + j] = h[j];
        if (j + 1 < K) t[(size_t)j * K + j + 1] = t[(size_t)(j + 1) * K + j] = h[K + j];
      }
      symmetric_eigen(K, t, w, z);
      int top = 0;
      for (int k = 1; k < K; ++k)
        if (w[k] > w[top]) top = k;
      lam = w[top];
      for (int j = 0; j < K; ++j) y[j] = z[(size_t)j * K + top];
    }
  }
  return hipGetLastError();
}

// The same Lanczos recurrence for B^-1 A (B: the level's vertical line blocks), self-adjoint in
// <u, v>_B = u^T B v = (L^T u).(L^T v): w = B^-1 q - alpha v - beta vp (one line solve), its B-norm
// from the factor, alpha = v.A v as before.
template <typename T>
hipError_t lanczos_lambda_line(Ctx &c, Ctx &L, T *u, T *v, T *vp, T *q, double &lam, hipStream_t s) {
  const T *dinv = Prec<T>::dinv(L);   // only places the start vector on the unknowns
  const int64_t n = L.n_v;
  constexpr int K = kLanczosSteps;
  double *al = c.d_mg_lz, *be = c.d_mg_lz + K, *nrm = c.d_mg_lz + 2 * K;
  const double rel = 1e-12;
  std::vector<double> y(K, 0.0);
  hipError_t e = hipSuccess;
  for (int pass = 0; pass < 2; ++pass) {
    T *a = v, *b = vp;
    k_lz_start<T><<<kVB<T>, kVecThreads, 0, s>>>(a, b, dinv, n, c.d_partial);
    if ((e = line_bnorm_partials<T>(L, a, c.d_partial, kVB<T>, s)) != hipSuccess) return e;
    k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, nrm, 1, nullptr, 0.0);
    k_lz_scale<T><<<kVB<T>, kVecThreads, 0, s>>>(a, n, nrm);
    for (int j = 0; j < K; ++j) {
      if (pass == 1) k_lz_acc<T><<<kVB<T>, kVecThreads, 0, s>>>(u, a, n, y[j], j == 0);
      if (pass == 1 && j == K - 1) break;
      if ((e = launch_apply(L, Prec<T>::dt, a, q, true, nullptr, nullptr, s)) != hipSuccess) return e;
      if (pass == 0) {
        k_lz_dot<T><<<kVB<T>, kVecThreads, 0, s>>>(a, q, n, c.d_partial);
        k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, al + j, 0, nullptr, 0.0);
      }
      if ((e = line_lanczos_w<T>(L, q, a, b, al + j, j > 0 ? be + j - 1 : nullptr, s)) != hipSuccess) return e;
      if (pass == 0) {
        if ((e = line_bnorm_partials<T>(L, b, c.d_partial, kVB<T>, s)) != hipSuccess) return e;
        k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, be + j, 1, al + j, rel);
      }
      k_lz_scale<T><<<kVB<T>, kVecThreads, 0, s>>>(b, n, be + j);
      std::swap(a, b);
    }
    if (pass == 0) {
      std::vector<double> h(2 * K);
      if ((e = hipMemcpyAsync(h.data(), c.d_mg_lz, sizeof(double) * 2 * K, hipMemcpyDeviceToHost, s)) != hipSuccess)
        return e;
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
      std::vector<double> t((size_t)K * K, 0.0), w, z;
      for (int j = 0; j < K; ++j) {
        t[(size_t)j * K + j] = h[j];
        if (j + 1 < K) t[(size_t)j * K + j + 1] = t[(size_t)(j + 1) * K + j] = h[K + j];
      }
      symmetric_eigen(K, t, w, z);
      int top = 0;
      for (int k = 1; k < K; ++k)
        if (w[k] > w[top]) top = k;
      lam = w[top];
      for (int j = 0; j < K; ++j) y[j] = z[(size_t)j * K + top];
    }
  }
  return hipGetLastError();
}

// power-iteration scalars of B^-1 A: pw[0] = (v.Av)/(v.Bv), pw[1] = sqrt(v.Bv) (pw[2], pw[3]: the sums)
__global__ void k_line_pow_fin(double *pw) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double vbv = pw[3];
  pw[0] = vbv > 0.0 ? pw[2] / vbv : 0.0;
  pw[1] = vbv > 0.0 ? sqrt(vbv) : 1.0;
}

// Largest eigenvalue of D^-1 A on level L, left in *pw on the device: Lanczos the first time
// (Ritz vector into v), then Rayleigh-quotient power iterations from the previous eigenvector
// estimate v after each geometry update (no host synchronisation).  w1, w2, q are work vectors.
// With the line smoother (c.mg_line) the same for B^-1 A.
template <typename T>
hipError_t estimate_lambda(Ctx &c, Ctx &L, T *v, T *q, T *w1, T *w2, bool warm, double *pw, hipStream_t s) {
  if (!warm) {
    double lam = 0.0;
    hipError_t e = c.mg_line ? lanczos_lambda_line<T>(c, L, v, w1, w2, q, lam, s)
                             : lanczos_lambda<T>(c, L, v, w1, w2, q, lam, s);
    if (e != hipSuccess) return e;
    k_set_scalar<<<1, 1, 0, s>>>(pw, lam);
    return hipGetLastError();
  }
  const T *dinv = Prec<T>::dinv(L);
  const int64_t n = L.n_v;
  if (c.mg_line) {
    for (int it = 0; it < kPowNext; ++it) {
      hipError_t e = launch_apply(L, Prec<T>::dt, v, q, true, nullptr, nullptr, s);
      if (e != hipSuccess) return e;
      k_lz_dot<T><<<kVB<T>, kVecThreads, 0, s>>>(v, q, n, c.d_partial);
      k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, pw + 2, 0, nullptr, 0.0);
      if ((e = line_bnorm_partials<T>(L, v, c.d_partial, kVB<T>, s)) != hipSuccess) return e;
      k_lz_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, pw + 3, 0, nullptr, 0.0);
      k_line_pow_fin<<<1, 1, 0, s>>>(pw);
      if ((e = line_apply<T>(L, q, v, s)) != hipSuccess) return e;
      k_lz_scale<T><<<kVB<T>, kVecThreads, 0, s>>>(v, n, pw + 1);
    }
    return hipGetLastError();
  }
  for (int it = 0; it < kPowNext; ++it) {
    hipError_t e = launch_apply(L, Prec<T>::dt, v, q, true, nullptr, nullptr, s);
    if (e != hipSuccess) return e;
    k_pow_dots<T><<<kVB<T>, kVecThreads, 0, s>>>(v, q, dinv, n, c.d_partial);
    k_pow_fin<<<1, kVecThreads, 0, s>>>(c.d_partial, kVB<T>, pw);
    k_pow_next<T><<<kVB<T>, kVecThreads, 0, s>>>(v, q, dinv, n, pw);
  }
  return hipGetLastError();
}

}  // namespace

// Builds the coarse levels (contexts at degrees p/2, p/4, ..., 1) and their work vectors.
static fnpf_status build_levels(Ctx &c) {
  {
    // contexts of several threads may come here at once: the tables are built in static memory
    static std::mutex first_use;
    static bool uploaded[64] = {false};
    const std::lock_guard<std::mutex> lock(first_use);
    if (c.device >= 0 && c.device < 64 && !uploaded[c.device]) {
      if (upload_tables() != hipSuccess) return FNPF_ERR_HIP;
      uploaded[c.device] = true;
    }
  }
  Ctx *F = &c;
  while (F->p > 1) {
    const int pc = F->p / 2;
    std::vector<int32_t> nodes;
    int64_t ns = 0;
    std::string err = coarse_numbering(*F, pc, nodes, ns);
    if (!err.empty()) {
      c.err = "p-multigrid: " + err;
      return FNPF_ERR_ARG;
    }
    fnpf_mesh_desc d{};
    d.dim = F->dim;
    d.p = pc;
    d.nz = F->nz;
    d.n_eh = F->n_eh;
    d.n_s = ns;
    d.eh_nodes = nodes.data();
    d.eh_corner = F->h_corner.data();
    d.eh_arc = F->h_arc.empty() ? nullptr : F->h_arc.data();
    d.eh_face_tag = F->h_tags.data();
    d.layer_s = F->h_layer_s.data();
    d.g = F->g;
    MgLevel L;
    fnpf_status st = fnpf_create(&d, &L.child);
    if (st != FNPF_OK) {
      c.err = std::string("p-multigrid: coarse level: ") + fnpf_last_error(nullptr);
      return st;
    }
    L.c = &ctx_of(L.child);
    if (dalloc_t(&L.Hc, L.c->n_s) != hipSuccess || dalloc_t(&L.hc, L.c->n_s) != hipSuccess) {
      c.mg.push_back(L);
      return FNPF_ERR_ALLOC;
    }
    c.mg.push_back(L);
    F = c.mg.back().c;
  }
  // (its kernels have a level a block in the grid's y and z, which HIP limits to 65,536)
  if (!c.mg.empty() && (size_t)27 * c.mg.back().c->n_v * sizeof(float) <= kP1MaxBytes && c.nz + 1 <= 65535) {
    const fnpf_status st = p1_build(*c.mg.back().c);
    if (st != FNPF_OK && st != FNPF_ERR_ARG) return st;   // ARG: a node with too many neighbours stays matrix-free
  }
  if (dalloc_t(&c.d_mgc, (size_t)2 * (c.mg.size() + 1) * kMgCoef) != hipSuccess) return FNPF_ERR_ALLOC;
  if (dalloc_t(&c.d_mg_lz, (size_t)kLzScalars) != hipSuccess) return FNPF_ERR_ALLOC;
  if (dalloc_t(&c.d_mg_lam, (size_t)2 * (c.mg.size() + 1)) != hipSuccess) return FNPF_ERR_ALLOC;
  if (hipMemset(c.d_mg_lam, 0, sizeof(double) * 2 * (c.mg.size() + 1)) != hipSuccess) return FNPF_ERR_HIP;
  void *ip64 = nullptr, *ip32 = nullptr;
  if (hipGetSymbolAddress(&ip64, HIP_SYMBOL(c_IP64)) != hipSuccess ||
      hipGetSymbolAddress(&ip32, HIP_SYMBOL(c_IP32)) != hipSuccess)
    return FNPF_ERR_HIP;
  auto tables = [&](Ctx &L) {
    L.d_ip64 = (const double *)ip64 + L.p * kMaxN1 * kMaxN1;
    L.d_ip32 = (const float *)ip32 + L.p * kMaxN1 * kMaxN1;
  };
  tables(c);
  for (auto &L : c.mg) tables(*L.c);
  c.mg_built = true;
  c.mg_stale64 = c.mg_stale32 = true;
  return FNPF_OK;
}

// A failure leaves no level behind: a later call starts afresh.
fnpf_status mg_build(Ctx &c) {
  if (c.mg_built) return FNPF_OK;
  try {
    const fnpf_status st = build_levels(c);
    if (st != FNPF_OK) mg_free(c);
    return st;
  } catch (const std::exception &) {
    mg_free(c);
    throw;
  }
}

void mg_free(Ctx &c) {
  for (auto &L : c.mg) {
    if (L.Hc) (void)hipFree(L.Hc);
    if (L.hc) (void)hipFree(L.hc);
    for (int k = 0; k < 5; ++k) {
      if (L.v64[k]) (void)hipFree(L.v64[k]);
      if (L.v32[k]) (void)hipFree(L.v32[k]);
    }
    if (L.ev64) (void)hipFree(L.ev64);
    if (L.ev32) (void)hipFree(L.ev32);
    if (L.child) fnpf_destroy(L.child);
  }
  c.mg.clear();
  for (int k = 0; k < 4; ++k) {
    if (c.mg_f64[k]) (void)hipFree(c.mg_f64[k]);
    if (c.mg_f32[k]) (void)hipFree(c.mg_f32[k]);
    c.mg_f64[k] = nullptr;
    c.mg_f32[k] = nullptr;
  }
  if (c.mg_ev64) (void)hipFree(c.mg_ev64);
  if (c.mg_ev32) (void)hipFree(c.mg_ev32);
  c.mg_ev64 = nullptr;
  c.mg_ev32 = nullptr;
  c.mg_ev_ok64 = c.mg_ev_ok32 = false;
  if (c.d_mgc) (void)hipFree(c.d_mgc);
  c.d_mgc = nullptr;
  if (c.d_mg_lz) (void)hipFree(c.d_mg_lz);
  c.d_mg_lz = nullptr;
  if (c.d_mg_lam) (void)hipFree(c.d_mg_lam);
  c.d_mg_lam = nullptr;
  c.mg_built = false;
}

// Brings the coarse levels up to the current geometry (and FP32 data when T is float) and
// re-estimates the smoothing intervals.  The work vectors of precision T are allocated here.
template <typename T>
fnpf_status mg_refresh(Ctx &c, hipStream_t s) {
  fnpf_status st = mg_build(c);
  if (st != FNPF_OK) return st;
  {
    T **fv = const_cast<T **>(Prec<T>::fv(c));
    for (int k = 0; k < 4; ++k)
      if (dalloc_t(&fv[k], c.n_v) != hipSuccess) return FNPF_ERR_ALLOC;
    if (dalloc_t(&Prec<T>::evf(c), c.n_v) != hipSuccess) return FNPF_ERR_ALLOC;
    for (auto &L : c.mg) {
      T **lv = const_cast<T **>(Prec<T>::lv(L));
      for (int k = 0; k < 5; ++k)
        if (dalloc_t(&lv[k], L.c->n_v) != hipSuccess) return FNPF_ERR_ALLOC;
      if (dalloc_t(&Prec<T>::ev(L), L.c->n_v) != hipSuccess) return FNPF_ERR_ALLOC;
      if (sizeof(T) == 4 && ctx_ensure32(*L.c) != FNPF_OK) return FNPF_ERR_ALLOC;
    }
    if (!c.mg.empty()) {
      Ctx &L = *c.mg.back().c;
      const size_t n = (size_t)3 * L.p1_w * L.n_v;
      if (n > 0 && n * sizeof(T) <= kP1MaxBytes && dalloc_t(&p1_values<T>(L), n) != hipSuccess) return FNPF_ERR_ALLOC;
    }
  }
  if (!Prec<T>::stale(c)) return FNPF_OK;
  Ctx *F = &c;
  for (auto &L : c.mg) {
    L.c->keep_diag = c.mg_line;
    if (surf_to(*F, *L.c, L.Hc, L.hc, s) != hipSuccess) return FNPF_ERR_HIP;
    st = geom_impl_total(*L.c, L.Hc, L.hc, s);
    if (st != FNPF_OK) return st;
    F = L.c;
  }
  if (!c.mg.empty() && !c.mg_line && p1_assemble<T>(*c.mg.back().c, s) != hipSuccess) return FNPF_ERR_HIP;
  if (c.mg_line) {
    // the vertical line blocks of every level from its current geometry, factored
    if (line_setup(c, s) != hipSuccess) return FNPF_ERR_HIP;
    for (auto &L : c.mg)
      if (line_setup(*L.c, s) != hipSuccess) return FNPF_ERR_HIP;
  }
  // eigenvalue estimates, warm-started from the previous geometry's eigenvector estimates, and the
  // coefficient table of this precision, all stream-ordered before any later use
  {
    const int nl = (int)c.mg.size() + 1;
    const int base = (sizeof(T) == 8 ? 0 : 1) * nl;
    double *pw = c.d_mg_scal;   // two scalars of the power iteration, apart from the partials
    for (int l = 0; l < nl; ++l) {
      hipError_t e;
      if (l == 0) {
        e = estimate_lambda<T>(c, c, Prec<T>::evf(c), Prec<T>::fv(c)[3], Prec<T>::fv(c)[1], Prec<T>::fv(c)[2],
                               Prec<T>::evokf(c), pw, s);
        Prec<T>::evokf(c) = true;
      } else {
        MgLevel &L = c.mg[l - 1];
        e = estimate_lambda<T>(c, *L.c, Prec<T>::ev(L), Prec<T>::lv(L)[4], Prec<T>::lv(L)[2], Prec<T>::lv(L)[3],
                               Prec<T>::evok(L), pw, s);
        Prec<T>::evok(L) = true;
      }
      if (e != hipSuccess) return FNPF_ERR_HIP;
      k_cheb_coef<<<1, 1, 0, s>>>(pw, l == nl - 1 ? kMgCoarseRatio : kMgSmoothRatio,
                                  c.d_mgc + (base + l) * kMgCoef, c.d_mg_lam + base + l);
      if (hipGetLastError() != hipSuccess) return FNPF_ERR_HIP;
    }
  }
  Prec<T>::stale(c) = false;
  return FNPF_OK;
}
template fnpf_status mg_refresh<double>(Ctx &, hipStream_t);
template fnpf_status mg_refresh<float>(Ctx &, hipStream_t);

template <typename T>
hipError_t mg_vcycle(Ctx &c, const T *r, T *z, const int32_t *skip, int smooth_deg, hipStream_t s,
                     double *dot_partial, bool *dot_done, bool pre_scaled) {
  if (dot_done) *dot_done = false;
  return vcycle<T>(c, 0, complete<T>(c, r), z, skip, smooth_deg, s, dot_partial, dot_done,
                   pre_scaled && smooth_deg == 2 && !c.mg.empty() && !c.mg_line);
}
template hipError_t mg_vcycle<double>(Ctx &, const double *, double *, const int32_t *, int, hipStream_t, double *,
                                      bool *, bool);
template hipError_t mg_vcycle<float>(Ctx &, const float *, float *, const int32_t *, int, hipStream_t, double *,
                                     bool *, bool);

static bool mg_prescale(const Ctx &c, int smooth_deg) { return smooth_deg == 2 && !c.mg.empty() && !c.mg_line; }

// Selects point (Jacobi) or vertical line smoothing; a change re-estimates every level's
// smoothing interval and rebuilds the line factors at the next refresh.
void mg_set_line(Ctx &c, bool line) {
  c.keep_diag = line;   // the line factors read every level's whole diagonal
  for (auto &L : c.mg) L.c->keep_diag = line;
  if (c.mg_line == line) return;
  c.mg_line = line;
  c.mg_stale64 = c.mg_stale32 = true;
  c.mg_ev_ok64 = c.mg_ev_ok32 = false;
  for (auto &L : c.mg) L.ev_ok64 = L.ev_ok32 = false;
}

template <typename T>
static hipError_t mg_update_impl(Ctx &c, T *x, T *r, const T *p, const T *q, double *partial, int npq, PcgScalars *sc,
                                 hipStream_t s, bool pre) {
  const int nb = partial_blocks<T>(c);
  const Deferred<T> qd = apply_result<T>(c, q);
  // the partials of r.r go behind those of p.q, which other blocks may still be reading
  double *rr = partial + npq;
  const int np = npq <= kFinPartials ? npq : 0;
  if (np == 0) {
    hipError_t e = launch_finalize_pq(partial, npq, sc, s);
    if (e != hipSuccess) return e;
  }
  with_levels(node_levels(c), [&](auto lv) {
    if (pre)
      k_mg_update<lv(), T, true><<<nb, kVecThreads, 0, s>>>(x, r, p, qd, c.n_s, rr, sc, Prec<T>::fv(c)[2],
                                                            Prec<T>::dinv(c), coef_table<T>(c, 0), partial, np);
    else
      k_mg_update<lv(), T, false><<<nb, kVecThreads, 0, s>>>(x, r, p, qd, c.n_s, rr, sc, nullptr, nullptr, nullptr,
                                                             partial, np);
  });
  k_mg_fin_rr<<<1, kVecThreads, 0, s>>>(rr, nb, sc);
  return hipGetLastError();
}

hipError_t launch_mg_update(Ctx &c, fnpf_dtype dt, void *x, void *r, const void *p, const void *q, double *partial,
                            int npq, PcgScalars *sc, hipStream_t s, int smooth_deg) {
  const bool pre = mg_prescale(c, smooth_deg);
  if (dt == FNPF_F64)
    return mg_update_impl<double>(c, (double *)x, (double *)r, (const double *)p, (const double *)q, partial, npq, sc,
                                  s, pre);
  return mg_update_impl<float>(c, (float *)x, (float *)r, (const float *)p, (const float *)q, partial, npq, sc, s,
                               pre);
}

template <typename T>
static hipError_t mg_dot_dir_impl(Ctx &c, const T *r, const T *z, T *p, double *partial, PcgScalars *sc, int first,
                                  hipStream_t s, bool have_partials) {
  // the V-cycle's last kernel took the partials on its own grid
  const int nf = (int)std::min<int64_t>((c.n_v + kVecThreads - 1) / kVecThreads, kVB<T>);
  const int np = have_partials ? partial_blocks<T>(c) : nf;
  if (!have_partials) k_dot<T><<<nf, kVecThreads, 0, s>>>(r, z, c.n_v, partial, sc);
  static_assert(kVB<T> <= kFinPartials && kNodeBlocks <= kFinPartials, "k_mg_dir sums the partials");
  k_mg_dir<T><<<nf, kVecThreads, 0, s>>>(p, z, c.n_v, sc, first, partial, np);
  return hipGetLastError();
}

hipError_t launch_mg_dot_dir(Ctx &c, fnpf_dtype dt, const void *r, const void *z, void *p, double *partial,
                             PcgScalars *sc, int first, hipStream_t s, bool have_partials) {
  if (dt == FNPF_F64)
    return mg_dot_dir_impl<double>(c, (const double *)r, (const double *)z, (double *)p, partial, sc, first, s,
                                   have_partials);
  return mg_dot_dir_impl<float>(c, (const float *)r, (const float *)z, (float *)p, partial, sc, first, s,
                                have_partials);
}

}  // namespace fnpf
