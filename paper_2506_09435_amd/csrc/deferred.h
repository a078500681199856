// deferred.h - vectors whose last assembly step is left to the kernel that reads them.
//
// Pass 1 of the owner-computes apply (and the restriction) leaves at a node the owner's value in y
// and the other tiles' (columns') values in face slots F, and, with the layers split into chunks,
// the lower chunk's value at a chunk interface in Z (behind F's level rows).  The next kernel of a
// solve reads every node of the vector anyway, so it adds them itself: that saves a launch and a
// read and write of y at the shared nodes per operator product (the face pass: 4.4 us of 17.9 for
// the periodic wave of 40 x 40 x 4, p = 5; 62 us of 334 for the sea of 256 x 128 x 6, p = 6).
#pragma once

#include <type_traits>

#include "fnpf_internal.h"

namespace fnpf {

template <typename T>
struct Deferred {
  const T *y = nullptr;
  const T *F = nullptr;             // nullptr: y is complete
  // a node's slots (nodes from n_hi on have none) in increasing order: up to three (-1: no more) and,
  // for a node with others, the place in `lists` of their number and of them (0: none).  Up to three
  // in one load, since each further dependent load costs these kernels about 1 us on small meshes.
  const int4 *slots = nullptr;
  const int32_t *lists = nullptr;
  int64_t n_hi = 0, n_slots = 0;
  int vend = 0;                     // levels from here on are complete (the masked top level)
  int nlev = 0, clev = 0, nchunk = 1;
};

template <typename T>
T *face_buffer(const Ctx &c);
template <>
inline double *face_buffer<double>(const Ctx &c) { return c.d_F64; }
template <>
inline float *face_buffer<float>(const Ctx &c) { return c.d_F32; }

// y as launch_apply(..., defer) left it (masked)
template <typename T>
Deferred<T> apply_result(const Ctx &c, const T *y) {
  Deferred<T> d;
  d.y = y;
  d.nlev = c.p * c.nz + 1;
  if (!owner_apply_active(c)) return d;
  d.F = face_buffer<T>(c);
  d.slots = c.d_t_slots;
  d.lists = c.d_t_lists;
  d.n_hi = c.t_n_hi;
  d.n_slots = c.n_tslots;
  d.vend = d.nlev - 1;
  d.clev = c.lpc * c.p;
  d.nchunk = (c.nz + c.lpc - 1) / c.lpc;
  return d;
}

template <typename T>
Deferred<T> complete(const Ctx &c, const T *y) {
  Deferred<T> d;
  d.y = y;
  d.nlev = c.p * c.nz + 1;
  return d;
}

// two surface fields y [2][n_s]: the owned columns' values, the others in the slots c.d_sF [2][n_slots]
inline Deferred<double> surface_result(const Ctx &c, const double *y) {
  Deferred<double> d;
  d.y = y;
  d.F = c.d_sF;
  d.slots = c.d_p_slots;
  d.lists = c.d_p_lists;
  d.n_hi = c.p_n_hi;
  d.n_slots = c.n_slots;
  return d;
}

// Grid-stride vector kernels over (levels, node): a task is 256 nodes at LV levels, a thread's LV
// values being in flight together.
inline int64_t node_tasks(const Ctx &c, int lv) { return (c.n_s + 255) / 256 * ((c.p * c.nz + lv) / lv); }
// Levels a thread: on small meshes as many as let all blocks be resident at once (eight per CU), so
// that the kernel is one chain of loads; large meshes are bound by HBM and take one level at a time
// (four rows of every operand at once were a third slower on the sea of 256 x 128 x 6, p = 6).
constexpr int kNodeBlocks = 8 * 256;
// (Kernels of one level a thread run at most 2,048 blocks.  Some need more than the 80 scalar registers
// with which eight blocks fit a CU, and the blocks left over make a second round: launch bounds keep them
// there.  The multigrid's FP32 update on that sea: 229 us with 80, 296 with 96.)
inline int node_levels(const Ctx &c) {
  return node_tasks(c, 1) <= kNodeBlocks ? 1 : node_tasks(c, 2) <= kNodeBlocks ? 2 : node_tasks(c, 4) <= kNodeBlocks ? 4 : 1;
}
inline int node_blocks(const Ctx &c, int lv, int most = 2 * kNodeBlocks) {
  return (int)(node_tasks(c, lv) < most ? node_tasks(c, lv) : most);
}

#ifdef __HIPCC__
// q + the slots of one level (row f of F) beyond a node's first three
template <typename T>
__device__ __forceinline__ T list_sum(const Deferred<T> &a, const T *f, int at, T q) {
  for (int k = 1; k <= a.lists[at]; ++k) q += f[a.lists[at + k]];
  return q;
}

// both fields of a surface_result at node n (nodes from n_hi on are complete)
__device__ __forceinline__ void gather_pair(const Deferred<double> &v, int64_t n, int64_t n_s, double &a, double &b) {
  a = v.y[n];
  b = v.y[n_s + n];
  if (n >= v.n_hi) return;
  const int4 s = v.slots[n];
  const double *f = v.F, *g = v.F + v.n_slots;
  if (s.x >= 0) a += f[s.x], b += g[s.x];
  if (s.y >= 0) a += f[s.y], b += g[s.y];
  if (s.z >= 0) a += f[s.z], b += g[s.z];
  if (s.w > 0) a = list_sum(v, f, s.w, a), b = list_sum(v, g, s.w, b);
}

// the assembled value at one node and level
template <typename T>
__device__ __forceinline__ T gather_one(const Deferred<T> &a, int64_t i, int64_t n, int64_t n_s, int v) {
  T q = a.y[i];
  if (n >= a.n_hi && a.nchunk <= 1) return q;
  int4 s = make_int4(-1, -1, -1, 0);
  if (n < a.n_hi) s = a.slots[n];
  auto add = [&](const T *row) {
    if (s.x >= 0) q += row[s.x];
    if (s.y >= 0) q += row[s.y];
    if (s.z >= 0) q += row[s.z];
    if (s.w > 0) q = list_sum(a, row, s.w, q);
  };
  if (v < a.vend) add(a.F + (int64_t)v * a.n_slots);
  if (a.nchunk > 1 && v > 0 && v < a.vend && v % a.clev == 0) {
    const int c = v / a.clev - 1;
    q += (a.F + (int64_t)(a.nlev + a.nchunk - 1) * a.n_slots)[c * n_s + n];
    add(a.F + (int64_t)(a.nlev + c) * a.n_slots);
  }
  return q;
}

// For every node n and level v, i = v n_s + n: use(i, load(i), q), q the assembled value of a (the
// slots in increasing order, then the chunk interface's).  The loads of the next task are issued
// before the current one is used, and those of the first before the skip flag is tested: on small
// meshes the time of these kernels is the chain of their loads, not their number.  start(): what
// else to do between the first loads and their use; false ends the block.
template <int LV, typename T, typename Load, typename Start, typename Use>
__device__ __forceinline__ void for_nodes(const Deferred<T> &a, int64_t n_s, Load load, Start start, Use use) {
  using V = decltype(load((int64_t)0));
  const int nbx = (int)((n_s + 255) >> 8), ntask = nbx * ((a.nlev + LV - 1) / LV);
  int task = blockIdx.x, v, n;
  int4 s = make_int4(-1, -1, -1, 0);
  bool ok;
  T q[LV];
  V L[LV];
  // the loads of a task that depend on no other load (levels and nodes past the end repeat the last)
  auto fetch = [&](int t, int &fv, int &fn, int4 &fs, bool &fok, T(&fq)[LV], V(&fL)[LV]) {
    const int ch = t / nbx;
    fv = ch * LV;
    fn = (t - ch * nbx) * 256 + threadIdx.x;
    fok = fn < n_s;
    fs = make_int4(-1, -1, -1, 0);
    if (fok && fn < a.n_hi) fs = a.slots[fn];
    const int64_t nn = fok ? fn : n_s - 1;
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      const int64_t i = (int64_t)min(fv + u, a.nlev - 1) * n_s + nn;
      fq[u] = a.y[i];
      fL[u] = load(i);
    }
  };
  if (task < ntask) fetch(task, v, n, s, ok, q, L);
  asm volatile("" ::: "memory");   // keeps the loads above start()'s tests
  if (!start()) return;
  while (task < ntask) {
    // the slots' values, all in flight together; at the level between two chunks also the lower
    // chunk's value z and its slots g
    T f[LV][3], g[LV][3], z[LV];
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      const int w = v + u, c = a.nchunk > 1 ? w / a.clev - 1 : -1;
      const bool in = w < a.vend, face = c >= 0 && in && w == (c + 1) * a.clev;
      const T *row = a.F + (int64_t)w * a.n_slots, *top = a.F + (int64_t)(a.nlev + c) * a.n_slots;
      f[u][0] = in && s.x >= 0 ? row[s.x] : T(0);
      f[u][1] = in && s.y >= 0 ? row[s.y] : T(0);
      f[u][2] = in && s.z >= 0 ? row[s.z] : T(0);
      z[u] = g[u][0] = g[u][1] = g[u][2] = T(0);
      if (face) {
        z[u] = ok ? (a.F + (int64_t)(a.nlev + a.nchunk - 1) * a.n_slots)[c * n_s + n] : T(0);
        if (s.x >= 0) g[u][0] = top[s.x];
        if (s.y >= 0) g[u][1] = top[s.y];
        if (s.z >= 0) g[u][2] = top[s.z];
      }
    }
    const int task2 = task + gridDim.x;
    int v2 = 0, n2 = 0;
    int4 s2 = make_int4(-1, -1, -1, 0);
    bool ok2 = false;
    T q2[LV];
    V L2[LV];
    if (task2 < ntask) fetch(task2, v2, n2, s2, ok2, q2, L2);
    if (ok) {
#pragma unroll
      for (int u = 0; u < LV; ++u) {
        const int w = v + u;
        if (w < a.nlev) {
          T qi = q[u] + f[u][0] + f[u][1] + f[u][2];
          if (s.w > 0 && w < a.vend) qi = list_sum(a, a.F + (int64_t)w * a.n_slots, s.w, qi);
          qi = qi + z[u] + g[u][0] + g[u][1] + g[u][2];
          if (s.w > 0 && a.nchunk > 1 && w > 0 && w < a.vend && w % a.clev == 0)
            qi = list_sum(a, a.F + (int64_t)(a.nlev + w / a.clev - 1) * a.n_slots, s.w, qi);
          use((int64_t)w * n_s + n, L[u], qi);
        }
      }
    }
    task = task2;
    v = v2;
    n = n2;
    s = s2;
    ok = ok2;
#pragma unroll
    for (int u = 0; u < LV; ++u) {
      q[u] = q2[u];
      L[u] = L2[u];
    }
  }
}

template <int LV, typename T, typename Load, typename Use>
__device__ __forceinline__ void for_nodes(const Deferred<T> &a, int64_t n_s, const int32_t *skip, Load load, Use use) {
  const int dn = skip != nullptr ? *skip : 0;
  for_nodes<LV>(a, n_s, load, [&] { return dn == 0; }, use);
}
#endif

// calls f with LV = lv as a constant
template <typename F>
inline void with_levels(int lv, F f) {
  if (lv == 1)
    f(std::integral_constant<int, 1>());
  else if (lv == 2)
    f(std::integral_constant<int, 2>());
  else
    f(std::integral_constant<int, 4>());
}

}  // namespace fnpf
