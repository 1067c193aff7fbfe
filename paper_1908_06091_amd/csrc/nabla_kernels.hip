// nabla_kernels.hip -- gfx950 kernels of the edge-based median-dual
// finite-volume nabla operators (Section 4.7, Figure 33: gradient,
// divergence, curl; the Laplacian is the divergence of the gradient).
//
// Field layout follows the NodeColumns function space (Section 4.5,
// Figure 31): a node's vertical column is contiguous, [node][level];
// vectors are [node][level][2].  Wavefront lanes run over levels, so every
// load and store of a column is coalesced.
//
// Per node i and level k the operators are signed sums over the node's own
// edges in a fixed order (ascending edge id, pole edge last):
//   gradient   G_i = sum_r sS_r (x_i + x_n)/2        (pole edge: lat only)
//   divergence D_i = sum_r sS_lon (u_i+u_n)/2 + sS_lat (W_i+W_n)/2, W = v cos
//   curl       C_i = sum_r sS_lon (v_i+v_n)/2 - sS_lat (Z_i+Z_n)/2, Z = u cos
// scaled by alpha_i = R/V_i (beta_i = R cos/V_i for the meridional gradient).
// Pole edges enter the gradient only (W and Z vanish on the pole line).
// No atomics: every output element has exactly one writer, so results are
// bitwise reproducible and independent of the launch shape.
//
// FP32 fields: the same sums over the promoted values, formed in FP64 with
// explicit fused multiply-adds and rounded to FP32 once at the end (the
// vector ALU runs FP64 at the FP32 rate, so this costs a conversion per
// value and a third of the operations of compensated FP32 sums).
//
// Compiled with -ffp-contract=off: no operation is fused unless written so,
// and every launch form of an operator produces the same bits.  (The
// separate edge-flux form, flux buffer then gather, exists for FP64 fields:
// a buffer of FP32 fluxes could not carry the FP64 terms.)
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

#include "internal.h"

namespace atlasx {

enum { OP_GRAD = 0, OP_DIV = 1, OP_CURL = 2 };

// native 2-vectors (kept in registers; also the [node][level][2] element)
typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// Tiles are numbered so that each XCD (workgroups are dealt round-robin to
// the 8 XCDs) receives a contiguous run of the processing order and keeps
// neighbouring columns in its own L2.
__device__ __forceinline__ int xcd_tile(int b, int per_xcd) {
  return (b & 7) * per_xcd + (b >> 3);
}

// Chunked tiles: either the mesh's tiles or fixed blocks of positions.
__device__ __forceinline__ bool tile_range(const DevMesh &m, int tile, int npb,
                                           int &p0, int &p1) {
  if (npb > 0) {
    p0 = tile * npb;
    if (p0 >= m.V) return false;
    p1 = min(m.V, p0 + npb);
    return true;
  }
  if (tile >= m.ntiles) return false;
  p0 = m.tile_ptr[tile];
  p1 = m.tile_ptr[tile + 1];
  return true;
}

// ---------------------------------------------------------------------------
// Per-element arithmetic.  A policy holds the running state of one output
// element (one node, one level) and is fed the node's incidences in CSR
// order; every launch form drives the same policy, so all forms produce the
// same bits.
// ---------------------------------------------------------------------------
// Output stores are non-temporal (streamed past the caches, so they do not
// evict input columns that neighbours still need); ATLASX_CACHED_STORE
// selects ordinary stores.
__device__ __forceinline__ void st_out(double *p, double v) {
#ifndef ATLASX_CACHED_STORE
  __builtin_nontemporal_store(v, p);
#else
  *p = v;
#endif
}
__device__ __forceinline__ void st_out(float *p, float v) {
#ifndef ATLASX_CACHED_STORE
  __builtin_nontemporal_store(v, p);
#else
  *p = v;
#endif
}
__device__ __forceinline__ void st_out2(double *p, double x, double y) {
  v2d v = {x, y};
#ifndef ATLASX_CACHED_STORE
  __builtin_nontemporal_store(v, reinterpret_cast<v2d *>(p));
#else
  *reinterpret_cast<v2d *>(p) = v;
#endif
}
__device__ __forceinline__ void st_out2(float *p, float x, float y) {
  v2f v = {x, y};
#ifndef ATLASX_CACHED_STORE
  __builtin_nontemporal_store(v, reinterpret_cast<v2f *>(p));
#else
  *reinterpret_cast<v2f *>(p) = v;
#endif
}

template <class T, int OP> struct Pol;

// FP64 gradient: G += sS (x_i + x_n)/2; the pole edge feeds the lat part.
template <> struct Pol<double, OP_GRAD> {
  static constexpr int kOp = OP_GRAD;
  using V = double;
  static constexpr bool kVecIn = false, kVecOut = true;
  struct St { double xi, gl, gt; };
  static __device__ __forceinline__ void init(St &s, V xi, double) { s.xi = xi; s.gl = 0.0; s.gt = 0.0; }
  static __device__ __forceinline__ void add(St &s, V xn, const double2 &S, bool pole, double) {
    const double xe = 0.5 * (s.xi + xn);
    if (!pole) s.gl = s.gl + S.x * xe;
    s.gt = s.gt + S.y * xe;
  }
  using Out = v2d;
  static __device__ __forceinline__ Out result(const St &s, double al, double be) {
    return Out{al * s.gl, be * s.gt};
  }
  // the same from halved normals Sh = S/2 (exact; same bits, one
  // multiplication less)
  static __device__ __forceinline__ void add_half(St &s, V xn, const double2 &Sh, bool pole, double) {
    const double xe = s.xi + xn;
    if (!pole) s.gl = s.gl + Sh.x * xe;
    s.gt = s.gt + Sh.y * xe;
  }
  static __device__ __forceinline__ Out result_half(const St &s, double al, double be) {
    return result(s, al, be);
  }
  static __device__ __forceinline__ void store(double *out, size_t idx, const St &s, double al,
                                               double be) {
    const Out r = result(s, al, be);
    st_out2(out + 2 * idx, r.x, r.y);
  }
  static __device__ __forceinline__ void keep(St &s, const St &t, bool use) {
    s.gl = use ? t.gl : s.gl;
    s.gt = use ? t.gt : s.gt;
  }
  static __device__ __forceinline__ void settle(St &s) { asm volatile("" : "+v"(s.gl), "+v"(s.gt)); }
};

// FP64 divergence / curl: sum of sS_lon a_e +- sS_lat b_e with edge
// averages of a = u (v) and b = v cos (u cos); pole edges do not enter.
template <int OP> struct PolDC64 {
  static constexpr int kOp = OP;
  using V = v2d;
  static constexpr bool kVecIn = true, kVecOut = false;
  struct St { double ai, bi, acc; };
  static __device__ __forceinline__ void init(St &s, V ui, double ci) {
    s.ai = (OP == OP_DIV) ? ui.x : ui.y;
    s.bi = ((OP == OP_DIV) ? ui.y : ui.x) * ci;
    s.acc = 0.0;
  }
  static __device__ __forceinline__ void add(St &s, V un, const double2 &S, bool, double cn) {
    const double an = (OP == OP_DIV) ? un.x : un.y;
    const double bn = ((OP == OP_DIV) ? un.y : un.x) * cn;
    const double ae = 0.5 * (s.ai + an), be = 0.5 * (s.bi + bn);
    const double f = (OP == OP_DIV) ? S.x * ae + S.y * be : S.x * ae - S.y * be;
    s.acc = s.acc + f;
  }
  using Out = double;
  static __device__ __forceinline__ Out result(const St &s, double al, double) {
    return al * s.acc;
  }
  static __device__ __forceinline__ void add_half(St &s, V un, const double2 &Sh, bool, double cn) {
    const double an = (OP == OP_DIV) ? un.x : un.y;
    const double bn = ((OP == OP_DIV) ? un.y : un.x) * cn;
    const double ae = s.ai + an, be = s.bi + bn;
    const double f = (OP == OP_DIV) ? Sh.x * ae + Sh.y * be : Sh.x * ae - Sh.y * be;
    s.acc = s.acc + f;
  }
  static __device__ __forceinline__ Out result_half(const St &s, double al, double be) {
    return result(s, al, be);
  }
  static __device__ __forceinline__ void store(double *out, size_t idx, const St &s, double al,
                                               double be) {
    st_out(out + idx, result(s, al, be));
  }
  static __device__ __forceinline__ void keep(St &s, const St &t, bool use) {
    s.acc = use ? t.acc : s.acc;
  }
  static __device__ __forceinline__ void settle(St &s) { asm volatile("" : "+v"(s.acc)); }
};
template <> struct Pol<double, OP_DIV> : PolDC64<OP_DIV> {};
template <> struct Pol<double, OP_CURL> : PolDC64<OP_CURL> {};

// FP32 fields: the FP64 sums with fused multiply-adds, of the normals
// themselves (the edge averages' factor 1/2 is applied to the sum: exact).
// O1280, 137 levels, against compensated FP32 sums of the differences, which
// took four operations per term and kept the SIMDs busy all the time:
// gradient 3.78 -> 3.15 ms, divergence 4.52 -> 4.31, Laplacian 7.98 -> 6.22;
// O640, 91 levels, divergence and curl in one pass 1.13 -> 0.97.
template <> struct Pol<float, OP_GRAD> {
  static constexpr int kOp = OP_GRAD;
  using V = float;
  static constexpr bool kVecIn = false, kVecOut = true;
  struct St { double xi, gl, gt; };
  static __device__ __forceinline__ void init(St &s, V xi, double) { s.xi = xi; s.gl = 0.0; s.gt = 0.0; }
  static __device__ __forceinline__ void add(St &s, V xn, const double2 &S, bool pole, double) {
    const double xe = s.xi + (double)xn;
    if (!pole) s.gl = __builtin_fma(S.x, xe, s.gl);
    s.gt = __builtin_fma(S.y, xe, s.gt);
  }
  using Out = v2f;
  static __device__ __forceinline__ Out result(const St &s, double al, double be) {
    return Out{(float)(al * (0.5 * s.gl)), (float)(be * (0.5 * s.gt))};
  }
  static __device__ __forceinline__ void add_half(St &s, V xn, const double2 &Sh, bool pole,
                                                  double cn) {
    add(s, xn, Sh, pole, cn);
  }
  static __device__ __forceinline__ Out result_half(const St &s, double al, double be) {
    return Out{(float)(al * s.gl), (float)(be * s.gt)};
  }
  static __device__ __forceinline__ void store(float *out, size_t idx, const St &s, double al,
                                               double be) {
    const Out r = result(s, al, be);
    st_out2(out + 2 * idx, r.x, r.y);
  }
  static __device__ __forceinline__ void keep(St &s, const St &t, bool use) {
    s.gl = use ? t.gl : s.gl;
    s.gt = use ? t.gt : s.gt;
  }
  static __device__ __forceinline__ void settle(St &s) { asm volatile("" : "+v"(s.gl), "+v"(s.gt)); }
  // (not volatile: a volatile statement counts as a write to memory, and the
  // uniform loads after it would become vector loads)
  static __device__ __forceinline__ void hold(St &s) { asm("" : "+v"(s.gl), "+v"(s.gt)); }
};

template <int OP> struct PolDC32 {
  static constexpr int kOp = OP;
  using V = v2f;
  static constexpr bool kVecIn = true, kVecOut = false;
  struct St { double ai, bi, acc; };
  static __device__ __forceinline__ void init(St &s, V ui, double ci) {
    s.ai = (OP == OP_DIV) ? ui.x : ui.y;
    s.bi = (double)((OP == OP_DIV) ? ui.y : ui.x) * ci;
    s.acc = 0.0;
  }
  static __device__ __forceinline__ void add(St &s, V un, const double2 &S, bool, double cn) {
    const double an = (OP == OP_DIV) ? un.x : un.y, qn = (OP == OP_DIV) ? un.y : un.x;
    const double ae = s.ai + an, be = __builtin_fma(qn, cn, s.bi);
    s.acc = __builtin_fma(S.x, ae, s.acc);
    s.acc = __builtin_fma((OP == OP_DIV) ? S.y : -S.y, be, s.acc);
  }
  using Out = float;
  static __device__ __forceinline__ Out result(const St &s, double al, double) {
    return (float)(al * (0.5 * s.acc));
  }
  static __device__ __forceinline__ void add_half(St &s, V un, const double2 &Sh, bool pole,
                                                  double cn) {
    add(s, un, Sh, pole, cn);
  }
  static __device__ __forceinline__ Out result_half(const St &s, double al, double) {
    return (float)(al * s.acc);
  }
  static __device__ __forceinline__ void store(float *out, size_t idx, const St &s, double al,
                                               double be) {
    st_out(out + idx, result(s, al, be));
  }
  static __device__ __forceinline__ void keep(St &s, const St &t, bool use) {
    s.acc = use ? t.acc : s.acc;
  }
  static __device__ __forceinline__ void settle(St &s) { asm volatile("" : "+v"(s.acc)); }
  static __device__ __forceinline__ void hold(St &s) { asm("" : "+v"(s.acc)); }
};
template <> struct Pol<float, OP_DIV> : PolDC32<OP_DIV> {};
template <> struct Pol<float, OP_CURL> : PolDC32<OP_CURL> {};

// One element at level k (any nlev); used by the generic column loop and
// by the flat form.
template <class T, int OP>
__device__ __forceinline__ void element(const DevMesh &m, const T *__restrict__ in,
                                        T *__restrict__ out, int nlev, int p, int node, int r0,
                                        int r1, int k) {
  using P = Pol<T, OP>;
  using V = typename P::V;
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const double ci = P::kVecIn ? m.coslat[node] : 0.0;
  typename P::St st;
  P::init(st, vin[(size_t)node * L + k], ci);
  for (int r = r0; r < r1; ++r) {
    const uint32_t nb = (uint32_t)m.nbr[r];
    const bool pole = (nb & kPoleBit) != 0;
    if (P::kVecIn && pole) continue;
    const double2 S = m.S[r];
    const size_t n = nb & ~kPoleBit;
    const double cn = P::kVecIn ? m.coslat[n] : 0.0;
    P::add(st, vin[n * L + k], S, pole, cn);
  }
  const double al = m.alpha[p], be = P::kVecOut ? m.beta[p] : 0.0;
  P::store(out, (size_t)node * L + k, st, al, be);
}

// Chunked column form: work units are (level chunk, tile), chunk-major, so
// the whole mesh is swept once per chunk and consecutive parallels of one
// chunk meet in the XCD's L2.  One wavefront per position; lanes over the
// chunk's levels.
template <class T, int OP>
__global__ void __launch_bounds__(1024) k_column_chunked(DevMesh m, const T *__restrict__ in,
                                                         T *__restrict__ out, int nlev, int npb,
                                                         int kc, int ntiles, int per_xcd) {
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int c = u / ntiles;
  int p0, p1;
  if (!tile_range(m, u - c * ntiles, npb, p0, p1)) return;
  const int k0 = c * kc;
  if (k0 >= nlev) return;
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int k = k0 + lane;
  const bool active = lane < kc && k < nlev;
  for (int p = p0 + wave; p < p1; p += nw) {
    const int node = __builtin_amdgcn_readfirstlane(m.perm[p]);
    const int r0 = __builtin_amdgcn_readfirstlane(m.rowp[p]);
    const int r1 = __builtin_amdgcn_readfirstlane(m.rowp[p + 1]);
    if (active) element<T, OP>(m, in, out, nlev, p, node, r0, r1, k);
  }
}

// ---------------------------------------------------------------------------
// Column form: one wavefront per position, lanes over levels.  NCH chunks
// of 64 levels are processed together and all of a node's incidences (up to
// G) are fetched in one round trip, so up to G*NCH column loads are in
// flight per wavefront.  The position record and the incidence rows are
// wavefront-uniform (scalar loads); the next position's record is fetched
// while the current one is computed.
// ---------------------------------------------------------------------------
// One group of up to G incidences starting at rb: every load first (the
// incidence arrays are padded, so entries past the row name valid nodes and
// need no branch), then the accumulation in row order.
template <class P, int NCH, int G>
__device__ __forceinline__ void column_group(const DevMesh &m, const typename P::V *__restrict__ vin,
                                             size_t L, const int (&kk)[NCH], int rb, int n,
                                             typename P::St (&st)[NCH]) {
  using V = typename P::V;
  uint32_t nb[G];
  double2 S[G];
  double cn[G];
  V xn[G][NCH];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    nb[j] = (uint32_t)m.nbr[rb + j];
    S[j] = m.S[rb + j];
    cn[j] = P::kVecIn ? m.ncos[rb + j] : 0.0;
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const size_t q = nb[j] & ~kPoleBit;
#pragma unroll
    for (int c = 0; c < NCH; ++c) xn[j][c] = vin[q * L + kk[c]];
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    if (j < n) {
      const bool pole = (nb[j] & kPoleBit) != 0;
      if (!(P::kVecIn && pole)) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) P::add(st[c], xn[j][c], S[j], pole, cn[j]);
      }
    }
  }
}

// ONE_GROUP: every row has at most G incidences and is handled by a single
// group without a loop (a loop back-edge makes the compiler wait for every
// outstanding memory operation, stores included, before the next loads).
template <class T, int OP, int NCH, int G, bool ONE_GROUP>
__device__ __forceinline__ void column_node(const DevMesh &m, const T *__restrict__ in,
                                            T *__restrict__ out, int nlev, const PosRec &pr,
                                            int k0) {
  using P = Pol<T, OP>;
  using V = typename P::V;
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const int node = pr.node, r0 = pr.r0, r1 = pr.r1;
  int kk[NCH];  // the lane's levels k0, k0 + 64, ..., clamped to the column
#pragma unroll
  for (int c = 0; c < NCH; ++c) kk[c] = min(k0 + 64 * c, nlev - 1);
  const double ci = P::kVecIn ? m.coslat[node] : 0.0;
  typename P::St st[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) P::init(st[c], vin[(size_t)node * L + kk[c]], ci);
  if (ONE_GROUP) {
    column_group<P, NCH, G>(m, vin, L, kk, r0, r1 - r0, st);
  } else {
    for (int rb = r0; rb < r1; rb += G) column_group<P, NCH, G>(m, vin, L, kk, rb, min(G, r1 - rb), st);
  }
  const double al = pr.alpha, be = P::kVecOut ? pr.beta : 0.0;
  // (FP32: the sums are held here.  Else they move into the branch around the
  // store, and the normals' loads with them, behind the wait for the columns:
  // 720x360 quadrilaterals, gradient, 37 levels 61.7 against 55.2 us)
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) P::hold(st[c]);
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c)
    if (k0 + 64 * c < nlev) P::store(out, (size_t)node * L + k0 + 64 * c, st[c], al, be);
}

template <class T, int OP, int NCH, int G>
__device__ __forceinline__ void column_pos(const DevMesh &m, const T *__restrict__ in,
                                           T *__restrict__ out, int nlev, int p,
                                           const PosRec &pr, int lane) {
  // G = 6: one load group covers every row of a mesh of degree <= 6 (the
  // octahedral mesh, pole edge included); G = 8: rows in groups
  if constexpr (NCH > 0) {
    column_node<T, OP, NCH, G, G == 6>(m, in, out, nlev, pr, lane);
  } else if constexpr (sizeof(T) == 4) {
    // any nlev: 256 levels at a time (vector columns 192; 64 at a time, each
    // incidence's loads waited for on their own, 720x360 quadrilaterals, 300
    // levels, took 451 us for the gradient and 476 for the divergence, 271 and
    // 434 this way)
    constexpr int N = Pol<T, OP>::kVecIn ? 3 : 4;
    for (int k0 = lane; k0 - lane < nlev; k0 += 64 * N)
      column_node<T, OP, N, G, G == 6>(m, in, out, nlev, pr, k0);
  } else {
    // any nlev: 64 levels after another (256 at a time: 721 against 590 us)
    for (int k = lane; k < nlev; k += 64) element<T, OP>(m, in, out, nlev, p, pr.node, pr.r0, pr.r1, k);
  }
}

// Tiled schedule (cyc == 0): one workgroup per tile / block of positions.
// Persistent schedule (cyc > 0 workgroups per XCD): the wavefronts of XCD x
// take positions of its share [V x/8, V (x+1)/8) cyclically, wavefront g at
// step t computing position lo + g + t * (cyc * waves per block).
template <class T, int OP, int NCH, int G>
__global__ void __launch_bounds__(512) k_column(DevMesh m, const T *__restrict__ in,
                                                 T *__restrict__ out, int nlev, int npb,
                                                 int per_xcd, int cyc) {
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int p, p1, stride;
  if (cyc > 0) {
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
    const int lo = (int)((int64_t)m.V * x / 8);
    p1 = (int)((int64_t)m.V * (x + 1) / 8);
    p = lo + i * nw + wave;
    stride = cyc * nw;
  } else {
    int p0;
    if (!tile_range(m, xcd_tile(blockIdx.x, per_xcd), npb, p0, p1)) return;
    p = p0 + wave;
    stride = nw;
  }
  if (p >= p1) return;
  PosRec cur = m.pos[p];
  for (; p < p1; p += stride) {
    const PosRec nxt = m.pos[min(p + stride, p1 - 1)];  // prefetch
    column_pos<T, OP, NCH, G>(m, in, out, nlev, p, cur, lane);
    cur = nxt;
  }
}

// ---------------------------------------------------------------------------
// Level-vector column form: as the column form, but every lane owns NV
// consecutive levels of the column and moves them with one 16-byte access
// (FP64 scalar columns: 2 levels per lane; FP32 scalar: 4; FP32 vector: 2).
// A wavefront load instruction then carries 1 KiB instead of 256-512 B, so a
// node needs 2-3x fewer vector memory instructions -- the address path, not
// the bytes, is what limits the one-level-per-lane form.  Column starts are
// only element-aligned (a column of 137 FP64 levels is 1096 B), so these are
// unaligned 16-byte accesses.  A lane's first level is clamped to
// nlev - NV: every access stays inside the column, and the lanes at the end
// recompute and store levels that a neighbouring lane also owns -- the same
// operation sequence, so the same bits are written twice.
// ---------------------------------------------------------------------------
// Buffer accesses.  A column (or a node's output run) is described by a
// buffer resource whose range is exactly that column; a lane whose offset is
// out of range makes no memory access at all (loads return 0, stores are
// dropped).  Lanes past the last lane vector therefore cost no cache
// traffic, unlike clamped duplicate accesses.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
__device__ i32x4 buf_load16(i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v4i32");
__device__ i32x2 buf_load8(i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v2i32");
__device__ void buf_store16(i32x4 v, i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v4i32");
__device__ void buf_store8(i32x2 v, i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v2i32");
__device__ void buf_store4(int v, i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.i32");

constexpr int kBufOff = 0x7fffff00;  // an offset outside every range used here
#ifndef ATLASX_CACHED_STORE
constexpr int kStoreAux = 2;         // non-temporal (streamed past the caches)
#else
constexpr int kStoreAux = 0;
#endif

// Raw buffer resource (stride 0) over [base, base + bytes); wavefront-uniform.
__device__ __forceinline__ i32x4 make_rsrc(const void *base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  i32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;
  return r;
}

// Read-only mesh data seen through the constant address space: the compiler
// may then serve wavefront-uniform reads with scalar loads even where the
// kernel also writes through buffer stores (which it cannot prove disjoint
// from a generic pointer).
#define ATLASX_CST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ const ATLASX_CST T *cst(const T *p) {
  return (const ATLASX_CST T *)p;
}

// Structures read field by field through the constant address space.
__device__ __forceinline__ double2 cst_double2(const double2 *p, size_t i) {
  const ATLASX_CST double *d = cst(reinterpret_cast<const double *>(p));
  double2 r;
  r.x = d[2 * i];
  r.y = d[2 * i + 1];
  return r;
}
__device__ __forceinline__ PosRec cst_pos(const PosRec *p, size_t i) {
  const ATLASX_CST PosRec *q = cst(p) + i;
  PosRec r;
  r.node = q->node;
  r.r0 = q->r0;
  r.r1 = q->r1;
  r.selfslot = q->selfslot;
  r.alpha = q->alpha;
  r.beta = q->beta;
  return r;
}

typedef int i32x3 __attribute__((ext_vector_type(3)));
__device__ int buf_load4(i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.i32");
__device__ i32x3 buf_load12(i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v3i32");
__device__ void buf_store12(i32x3 v, i32x4 rsrc, int voff, int soff, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v3i32");

// A lane vector of 4..32 bytes, in 16-, 8- and 4-byte pieces.
template <class R>
__device__ __forceinline__ R buf_load(const i32x4 &rsrc, int voff) {
  constexpr int B = (int)sizeof(R);
  static_assert(B % 4 == 0 && B <= 32, "lane vectors are 4..32 bytes");
  int w[B / 4];
  int at = 0;
#pragma unroll
  for (; at + 16 <= B; at += 16) {
    const i32x4 v = buf_load16(rsrc, voff + at, 0, 0);
    w[at / 4] = v.x; w[at / 4 + 1] = v.y; w[at / 4 + 2] = v.z; w[at / 4 + 3] = v.w;
  }
  if constexpr (B % 16 == 12) {
    const i32x3 v = buf_load12(rsrc, voff + (B / 16) * 16, 0, 0);
    w[(B / 16) * 4] = v.x;
    w[(B / 16) * 4 + 1] = v.y;
    w[(B / 16) * 4 + 2] = v.z;
  } else {
    if constexpr (B % 16 >= 8) {
      const i32x2 v = buf_load8(rsrc, voff + (B / 16) * 16, 0, 0);
      w[(B / 16) * 4] = v.x;
      w[(B / 16) * 4 + 1] = v.y;
    }
    if constexpr (B % 8 == 4) w[B / 4 - 1] = buf_load4(rsrc, voff + B - 4, 0, 0);
  }
  R r;
  __builtin_memcpy(&r, w, B);
  return r;
}

// Stores `W` 32-bit words of one lane at byte offset `ob`, in 16-, 8- and
// 4-byte pieces (non-temporal).
template <int W>
__device__ __forceinline__ void buf_store_words(const int (&w)[W], const i32x4 &rsrc, int ob) {
#pragma unroll
  for (int k = 0; k + 4 <= W; k += 4)
    buf_store16(i32x4{w[k], w[k + 1], w[k + 2], w[k + 3]}, rsrc, ob + 4 * k, 0, kStoreAux);
  if constexpr (W % 4 == 3) {
    buf_store12(i32x3{w[W - 3], w[W - 2], w[W - 1]}, rsrc, ob + 4 * (W - 3), 0, kStoreAux);
  } else {
    if constexpr (W % 4 >= 2)
      buf_store8(i32x2{w[(W / 4) * 4], w[(W / 4) * 4 + 1]}, rsrc, ob + 16 * (W / 4), 0, kStoreAux);
    if constexpr (W % 2 == 1) buf_store4(w[W - 1], rsrc, ob + 4 * (W - 1), 0, kStoreAux);
  }
}

// A lane vector: NV consecutive levels of one column, NV * sizeof(V) bytes.
template <class V> struct ElemOf { using E = V; static constexpr int C = 1; };
template <> struct ElemOf<v2d> { using E = double; static constexpr int C = 2; };
template <> struct ElemOf<v2f> { using E = float; static constexpr int C = 2; };

template <class V, int NV> struct LaneVec {
  using E = typename ElemOf<V>::E;
  static constexpr int C = ElemOf<V>::C;
  struct raw {
    E e[NV * C];
  };
  static __device__ __forceinline__ V get(const raw &r, int v) {
    if constexpr (C == 1) {
      return r.e[v];
    } else {
      return V{r.e[2 * v], r.e[2 * v + 1]};
    }
  }
};

// The level-vector form exists for this element type and width: NV levels
// of at most 32 bytes per lane.
template <class T, int OP, int NV>
constexpr bool lane_vec_ok() {
  return NV >= 1 && NV <= 4 && NV * sizeof(typename Pol<T, OP>::V) <= 32;
}

// Incidences every row of a mesh has besides its pole edge (the octahedral
// meshes: at least 4); below it the level-vector kernels need no select.
constexpr int kMinRow = 4;

// One node (rows of at most 6 incidences, one load group), NCH chunks of
// 64 lanes x NV levels.
template <class T, int OP, int NV, int NCH>
__device__ __forceinline__ void colv_node(const DevMesh &m, const T *__restrict__ in,
                                          T *__restrict__ out, int nlev, const PosRec &pr,
                                          int lane) {
  using P = Pol<T, OP>;
  using V = typename P::V;
  using LV = LaneVec<V, NV>;
  using R = typename LV::raw;
  using Out = typename P::Out;
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(V));
  const int node = pr.node, r0 = pr.r0, n = pr.r1 - pr.r0;
  // lane vector c of this lane starts at level s[c]; the last vector is
  // clamped inside the column, lanes past it get an out-of-range offset
  const int nvec = (nlev + NV - 1) / NV;
  int s[NCH], off[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = lane + 64 * c;
    s[c] = min(NV * idx, nlev - NV);
    off[c] = idx < nvec ? s[c] * (int)sizeof(V) : kBufOff;
  }
  const double ci = P::kVecIn ? cst(m.coslat)[node] : 0.0;
  typename P::St st[NCH][NV];
  {
    const i32x4 rs = make_rsrc(vin + (size_t)node * L, col_bytes);
    R xi[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) xi[c] = buf_load<R>(rs, off[c]);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int v = 0; v < NV; ++v) P::init(st[c][v], LV::get(xi[c], v), ci);
  }
  constexpr int G = 6;
  uint32_t nb[G];
  double2 S[G];
  double cn[G];
  R xn[G][NCH];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    nb[j] = (uint32_t)cst(m.nbr)[r0 + j];
    S[j] = cst_double2(m.S, r0 + j);
    cn[j] = P::kVecIn ? cst(m.ncos)[r0 + j] : 0.0;
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const size_t q = nb[j] & ~kPoleBit;
    const i32x4 rs = make_rsrc(vin + q * L, col_bytes);
#pragma unroll
    for (int c = 0; c < NCH; ++c) xn[j][c] = buf_load<R>(rs, off[c]);
  }
  // Every incidence of the group is accumulated into a candidate state and
  // kept by a select (not a branch): the loads above then have unconditional
  // uses and stay one burst, instead of being moved into a branch per
  // incidence and waited for one at a time.  Padding entries (j >= n) and
  // pole edges of div/curl leave the state as it was.
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const bool pole = (nb[j] & kPoleBit) != 0;
    if (j < kMinRow) {  // present in every row, never the pole edge
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int v = 0; v < NV; ++v) P::add(st[c][v], LV::get(xn[j][c], v), S[j], false, cn[j]);
      continue;
    }
    const bool use = j < n && !(P::kVecIn && pole);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        typename P::St t = st[c][v];
        P::add(t, LV::get(xn[j][c], v), S[j], pole, cn[j]);
        P::keep(st[c][v], t, use);
      }
  }
  // A lane's NV results are contiguous in the output run of the node:
  // written in 16-byte pieces (8 / 4 bytes for a shorter run).
  const double al = pr.alpha, be = P::kVecOut ? pr.beta : 0.0;
  const i32x4 ro = make_rsrc(out + (size_t)node * L * (sizeof(Out) / sizeof(T)),
                             (uint32_t)(L * sizeof(Out)));
  constexpr int W = NV * (int)sizeof(Out) / 4;  // 32-bit words per lane vector
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    int w[W];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const Out r = P::result(st[c][v], al, be);
      __builtin_memcpy(&w[v * (int)sizeof(Out) / 4], &r, sizeof(Out));
    }
    const int ob = off[c] == kBufOff ? kBufOff : s[c] * (int)sizeof(Out);
    buf_store_words<W>(w, ro, ob);
  }
}

// Same schedules as k_column (tiled, or persistent wave-cyclic).  The
// occupancy hint lets the register allocator keep a node's whole load burst
// in flight (at the default target it delays part of the burst to save
// registers, and each delayed load is then waited for on its own).  The
// most waves per SIMD at which the burst fits without spilling: five for
// FP32 in one chunk; four up to two chunks (FP32 lanes above 8 bytes: two),
// and for FP64 lanes of at most 16 bytes (the FP64 divergence: 97 registers and
// 7.31 ms, against 169 and 7.73 ms at two); otherwise two.
template <class T, int LB, int NCH> constexpr int colv_waves() {
  return sizeof(T) == 4 ? (NCH == 1 ? 5 : NCH == 2 && LB <= 8 ? 4 : 2)
         : NCH <= 2 || LB <= 16 ? 4 : 2;
}
// The same for the one-pass divergence + curl (two states per level).
template <class T, int NV, int NCH> constexpr int colv_dc_waves() {
  return sizeof(T) == 4 ? (NCH == 1 ? (NV <= 3 ? 5 : 4) : NCH == 2 && NV <= 1 ? 4 : 2)
         : NCH <= 2 || (NV == 1 && NCH == 3) ? 4 : 2;
}

template <class T, int OP, int NV, int NCH>
__global__ void __launch_bounds__(512)
    __attribute__((amdgpu_waves_per_eu(
        colv_waves<T, NV * (int)sizeof(typename Pol<T, OP>::V), NCH>(),
        colv_waves<T, NV * (int)sizeof(typename Pol<T, OP>::V), NCH>())))
    k_colv(DevMesh m, const T *__restrict__ in,
                                               T *__restrict__ out, int nlev, int npb,
                                               int per_xcd, int cyc) {
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int p, p1, stride;
  if (cyc > 0) {
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
    const int lo = (int)((int64_t)m.V * x / 8);
    p1 = (int)((int64_t)m.V * (x + 1) / 8);
    p = lo + i * nw + wave;
    stride = cyc * nw;
  } else {
    int p0;
    if (!tile_range(m, xcd_tile(blockIdx.x, per_xcd), npb, p0, p1)) return;
    p = p0 + wave;
    stride = nw;
  }
  if (p >= p1) return;
  PosRec cur = cst_pos(m.pos, p);
  for (; p < p1; p += stride) {
    const PosRec nxt = cst_pos(m.pos, min(p + stride, p1 - 1));  // prefetch
    colv_node<T, OP, NV, NCH>(m, in, out, nlev, cur, lane);
    cur = nxt;
  }
}

// Divergence and curl of one vector field in one pass: the column form of
// colv_node with both operators' states fed from the same loads, so (u, v)
// is read once and each output gets exactly the operation sequence of its
// own operator (bitwise equal to the two separate calls).
template <class T, int NV, int NCH>
__device__ __forceinline__ void colv_node_dc(const DevMesh &m, const T *__restrict__ in,
                                             T *__restrict__ out_d, T *__restrict__ out_c,
                                             int nlev, const PosRec &pr, int lane) {
  using PD = Pol<T, OP_DIV>;
  using PC = Pol<T, OP_CURL>;
  using V = typename PD::V;
  using LV = LaneVec<V, NV>;
  using R = typename LV::raw;
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(V));
  const int node = pr.node, r0 = pr.r0, n = pr.r1 - pr.r0;
  const int nvec = (nlev + NV - 1) / NV;
  int s[NCH], off[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = lane + 64 * c;
    s[c] = min(NV * idx, nlev - NV);
    off[c] = idx < nvec ? s[c] * (int)sizeof(V) : kBufOff;
  }
  const double ci = cst(m.coslat)[node];
  typename PD::St sd[NCH][NV];
  typename PC::St sc[NCH][NV];
  {
    const i32x4 rs = make_rsrc(vin + (size_t)node * L, col_bytes);
    R xi[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) xi[c] = buf_load<R>(rs, off[c]);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        PD::init(sd[c][v], LV::get(xi[c], v), ci);
        PC::init(sc[c][v], LV::get(xi[c], v), ci);
      }
  }
  constexpr int G = 6;
  uint32_t nb[G];
  double2 S[G];
  double cn[G];
  R xn[G][NCH];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    nb[j] = (uint32_t)cst(m.nbr)[r0 + j];
    S[j] = cst_double2(m.S, r0 + j);
    cn[j] = cst(m.ncos)[r0 + j];
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const size_t q = nb[j] & ~kPoleBit;
    const i32x4 rs = make_rsrc(vin + q * L, col_bytes);
#pragma unroll
    for (int c = 0; c < NCH; ++c) xn[j][c] = buf_load<R>(rs, off[c]);
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const bool pole = (nb[j] & kPoleBit) != 0;
    if (j < kMinRow) {
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          PD::add(sd[c][v], LV::get(xn[j][c], v), S[j], false, cn[j]);
          PC::add(sc[c][v], LV::get(xn[j][c], v), S[j], false, cn[j]);
        }
      continue;
    }
    const bool use = j < n && !pole;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        typename PD::St td = sd[c][v];
        PD::add(td, LV::get(xn[j][c], v), S[j], pole, cn[j]);
        PD::keep(sd[c][v], td, use);
        typename PC::St tc = sc[c][v];
        PC::add(tc, LV::get(xn[j][c], v), S[j], pole, cn[j]);
        PC::keep(sc[c][v], tc, use);
      }
  }
  const double al = pr.alpha;
  const i32x4 rd = make_rsrc(out_d + (size_t)node * L, (uint32_t)(L * sizeof(T)));
  const i32x4 rc = make_rsrc(out_c + (size_t)node * L, (uint32_t)(L * sizeof(T)));
  constexpr int W = NV * (int)sizeof(T) / 4;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    int wd[W], wc[W];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const T a = PD::result(sd[c][v], al, 0.0);
      const T b = PC::result(sc[c][v], al, 0.0);
      __builtin_memcpy(&wd[v * (int)sizeof(T) / 4], &a, sizeof(T));
      __builtin_memcpy(&wc[v * (int)sizeof(T) / 4], &b, sizeof(T));
    }
    const int ob = off[c] == kBufOff ? kBufOff : s[c] * (int)sizeof(T);
    buf_store_words<W>(wd, rd, ob);
    buf_store_words<W>(wc, rc, ob);
  }
}

template <class T, int NV, int NCH>
__global__ void __launch_bounds__(512)
    __attribute__((amdgpu_waves_per_eu(colv_dc_waves<T, NV, NCH>(), colv_dc_waves<T, NV, NCH>())))
    k_colv_dc(DevMesh m, const T *__restrict__ in, T *__restrict__ out_d,
              T *__restrict__ out_c, int nlev, int npb, int per_xcd) {
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int p0, p1;
  if (!tile_range(m, xcd_tile(blockIdx.x, per_xcd), npb, p0, p1)) return;
  for (int p = p0 + wave; p < p1; p += nw) {
    const PosRec pr = cst_pos(m.pos, p);
    colv_node_dc<T, NV, NCH>(m, in, out_d, out_c, nlev, pr, lane);
  }
}

// Levels per lane of the level-vector form for (T, OP, nlev).  FP64 (bound
// by memory traffic): 16-byte lanes.  FP32 (its FP64 sums and conversions
// weigh more against half the bytes): the width (1..4 levels, at most 32 bytes per
// lane) that needs the fewest level slots per lane (NV x chunks of 64
// lanes; the arithmetic runs once per slot), then the fewest load
// instructions per column, then one chunk (193 to 256 levels of a vector
// column on four levels per lane or two chunks of two: F640, 200 levels,
// divergence 2713 against 3373 us).  `want` > 0 forces a width.  0 when the form
// does not apply (mesh degree above 6 or a row shorter than kMinRow, no
// width fitting the column, more than 4 chunks) and the one-level-per-lane
// column kernel runs instead.
template <class T, int OP>
__host__ __device__ inline int auto_level_vec(int nlev, int maxdeg, int mindeg, int want = 0) {
  if (maxdeg > 6 || mindeg < kMinRow) return 0;
  const int vb = (int)sizeof(typename Pol<T, OP>::V);
  if (want == 0 && sizeof(T) == 8) want = 16 / vb;
  int best = 0, best_slots = 1 << 30, best_loads = 1 << 30;
  for (int nv = 1; nv <= 4; ++nv) {
    if (nv * vb > 32 || nlev < nv || (want > 0 && nv != want)) continue;
    const int nch = ((nlev + nv - 1) / nv + 63) / 64;
    if (nch > 4) continue;
    const int bytes = nv * vb;
    const int pieces = bytes / 16 + ((bytes % 16) ? 1 : 0);  // 16/12/8/4-byte accesses
    const int slots = nv * nch, loads = nch * pieces;
    if (slots < best_slots ||
        (slots == best_slots && (loads < best_loads || (loads == best_loads && nch == 1)))) {
      best = nv;
      best_slots = slots;
      best_loads = loads;
    }
  }
  return best;
}

// ---------------------------------------------------------------------------
// Parallel-sweep form.  A workgroup owns one tile (a longitude sector of a
// band of parallels) and one chunk of levels.  It walks down the band one
// parallel at a time, keeping the runs of the parallels above, at and below
// the current one in a 4-slot LDS ring buffer; while it computes parallel q
// it has the loads of parallel q+2 in flight (staged through registers).
// Every column is read from memory once per chunk plus a thin halo; every
// neighbour comes from LDS.  One wavefront per position, lanes over levels.
// ---------------------------------------------------------------------------
template <class T, int OP, int EPT>
__global__ void __launch_bounds__(1024) k_sweep(DevMesh m, const T *__restrict__ in,
                                               T *__restrict__ out, int nlev, int kcmax,
                                               int ntiles, int per_xcd) {
  using P = Pol<T, OP>;
  using V = typename P::V;
  constexpr int G = 8;  // incidences fetched together
  extern __shared__ __align__(16) unsigned char smem_raw[];
  V *buf = reinterpret_cast<V *>(smem_raw);
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int c = u / ntiles;
  const int tile = u - c * ntiles;
  const int k0 = c * kcmax;
  if (k0 >= nlev) return;
  const int kc = min(kcmax, nlev - k0);
  const int s0 = m.tile_seg[tile];
  const int nseg = m.tile_seg[tile + 1] - s0;
  const int slot_stride = m.segmax * kc;  // elements per LDS slot
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool lane_on = lane < kc;

  // staging: wavefront w moves nodes w, w+nw, ... of a run; lanes = levels
  V regs[EPT];
  const int lane_c = min(lane, kc - 1);
  auto fetch = [&](int q) {
    const int4 sg = m.seg[s0 + q];  // ring offset, ring size, first index, length
    // no branches around the loads: slots past the run re-read its last node
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int t = max(0, min(wave + i * nw, sg.w - 1));
      int ii = sg.z + t;
      if (ii >= sg.y) ii -= sg.y;
      regs[i] = vin[(size_t)(sg.x + ii) * L + k0 + lane_c];
    }
  };
  auto deposit = [&](int q) {
    const int len = m.seg[s0 + q].w;
    V *b = buf + (q & 3) * slot_stride;
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int t = wave + i * nw;
      if (t < len && lane_on) b[t * kc + lane] = regs[i];
    }
  };

  // first and last parallel with positions of this tile
  int qa = nseg, qb = -1;
  for (int q = 0; q < nseg; ++q) {
    const int2 pr = m.seg_pos[s0 + q];
    if (pr.y > pr.x) {
      qa = min(qa, q);
      qb = q;
    }
  }
  if (qb < 0) return;
  for (int q = 0; q <= min(nseg - 1, qa + 1); ++q) {
    fetch(q);
    deposit(q);
  }
  __syncthreads();
  for (int q = qa; q <= qb; ++q) {
    const bool pf = q + 2 < nseg;
    if (pf) fetch(q + 2);
    const int2 pr = m.seg_pos[s0 + q];
    if (lane_on) {
      const V *bq = buf + (q & 3) * slot_stride;
      for (int p = pr.x + wave; p < pr.y; p += nw) {
        const PosRec rec = m.pos[p];
        const int node = rec.node, r0 = rec.r0, r1 = rec.r1, ts = rec.selfslot;
        const double ci = P::kVecIn ? m.coslat[node] : 0.0;
        typename P::St st;
        P::init(st, bq[ts * kc + lane], ci);
        for (int rb = r0; rb < r1; rb += G) {
          // all loads of the group first (indices clamped into the row),
          // then the accumulation in row order
          int lr[G];
          double2 S[G];
          V xn[G];
          double cn[G];
#pragma unroll
          for (int j = 0; j < G; ++j) {  // whole group, contiguous (arrays padded)
            lr[j] = m.lref[rb + j];
            S[j] = m.S[rb + j];
            cn[j] = P::kVecIn ? m.ncos[rb + j] : 0.0;
          }
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const int l = lr[j] & ~kLrefPole;
            xn[j] = buf[((q + (l >> 16) - 1) & 3) * slot_stride + (l & 0xffff) * kc + lane];
          }
#pragma unroll
          for (int j = 0; j < G; ++j) {
            if (rb + j >= r1) break;
            const bool pole = (lr[j] & kLrefPole) != 0;
            if (P::kVecIn && pole) continue;
            P::add(st, xn[j], S[j], pole, cn[j]);
          }
        }
        const double al = rec.alpha, be = P::kVecOut ? rec.beta : 0.0;
        P::store(out, (size_t)node * L + k0 + lane, st, al, be);
      }
    }
    if (pf) deposit(q + 2);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Flat form: lanes over flattened (position, level) pairs of the tile --
// full lanes for short columns (nlev = 1 .. 40).
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// Level-vector sweep form.  As the parallel sweep above, but every LDS entry
// and every lane holds a lane vector of NV levels (16 bytes), a workgroup
// covers `vpc` lane vectors of every column (a level chunk), columns are
// staged into LDS with range-checked buffer loads (one pass over each
// column per chunk, coalesced over the run), and each position's result is
// written with buffer stores (lanes past the chunk make no access).  The
// geometry of the positions is staged into LDS as well, one step ahead (the
// position records of run q+2 and the incidence rows of run q+1 while run
// q is computed), so a position needs no dependent scalar loads: per step
// the chain is one LDS read of its record and rows, one of its neighbours.
// ---------------------------------------------------------------------------
constexpr int kSweepEpt = 4;   // staged lane vectors per thread and run
constexpr int kGeoWords = 11;  // 16-byte words of staged rows per position:
                               // S[6] (6), lref[8] (2), ncos[6] (3)

template <class T, int OP, int NV, int EPT>
__global__ void __launch_bounds__(1024) k_sweepv(DevMesh m, const T *__restrict__ in,
                                                 T *__restrict__ out, int nlev, int vpc,
                                                 int ntiles, int per_xcd) {
  using P = Pol<T, OP>;
  using V = typename P::V;
  using LV = LaneVec<V, NV>;
  using R = typename LV::raw;
  using Out = typename P::Out;
  constexpr int WPP = P::kVecIn ? kGeoWords : 8;  // rows words staged per position
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int segmax = m.segmax;
  R *buf = reinterpret_cast<R *>(smem_raw);                        // [4][segmax][vpc]
  i32x4 *gpos = reinterpret_cast<i32x4 *>(buf + 4 * segmax * vpc);  // [4][segmax][2]
  i32x4 *grow = gpos + 4 * segmax * 2;                              // [4][segmax][kGeoWords]
  // chunk-minor order: the chunks of a tile run next to each other on one
  // XCD, so the geometry and the cache lines a chunk boundary splits are
  // fetched once into its L2
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int nvec = (nlev + NV - 1) / NV;
  const int nchunk = (nvec + vpc - 1) / vpc;
  const int tile = u / nchunk;
  const int c = u - tile * nchunk;
  if (tile >= ntiles) return;
  const int v0 = c * vpc;
  if (v0 >= nvec) return;
  const int nvc = min(vpc, nvec - v0);  // lane vectors in this chunk
  const int s0 = cst(m.tile_seg)[tile];
  const int nseg = cst(m.tile_seg)[tile + 1] - s0;
  const int slot_stride = segmax * vpc;  // lane vectors per LDS slot
  const V *vin = reinterpret_cast<const V *>(in);
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(V));
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int *segi = reinterpret_cast<const int *>(m.seg);
  const int *segp = reinterpret_cast<const int *>(m.seg_pos);
  auto first = [&](int k) { return min(NV * (v0 + k), nlev - NV); };
  auto run_lo = [&](int q) { return cst(segp)[2 * (s0 + q)]; };
  auto run_hi = [&](int q) { return cst(segp)[2 * (s0 + q) + 1]; };

  // ---- columns: item = (node t of the segment, lane vector k); a thread's
  // items are the same every step (computed once)
  R regs[EPT];
  int it_t[EPT], it_off[EPT], it_lds[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int i = threadIdx.x + e * (int)blockDim.x;
    const int t = i / nvc, k = i - t * nvc;
    it_t[e] = t;
    it_off[e] = first(k) * (int)sizeof(V);
    it_lds[e] = t * vpc + k;
  }
  int seg_len = 0;
  auto fetch = [&](int q) {
    const int rb = cst(segi)[4 * (s0 + q)], nx = cst(segi)[4 * (s0 + q) + 1];
    const int lo = cst(segi)[4 * (s0 + q) + 2];
    seg_len = cst(segi)[4 * (s0 + q) + 3];
    const i32x4 rs = make_rsrc(vin + (size_t)rb * L, (uint32_t)nx * col_bytes);
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      int ii = lo + it_t[e];
      if (ii >= nx) ii -= nx;
      const int off = it_t[e] < seg_len ? ii * (int)col_bytes + it_off[e] : kBufOff;
      regs[e] = buf_load<R>(rs, off);
    }
  };
  auto deposit = [&](int q) {
    R *b = buf + (q & 3) * slot_stride;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (it_t[e] < seg_len) b[it_lds[e]] = regs[e];
  };
  // ---- position records of run q (2 words each) and rows of run q (WPP
  // words each, at the record's first incidence); a thread moves at most one
  // word of each kind per step (the dispatch guarantees the block is large
  // enough)
  i32x4 preg = {0, 0, 0, 0}, rreg = {0, 0, 0, 0};
  int pitem = -1, ritem = -1;
  auto fetch_pos = [&](int q) {
    const int plo = run_lo(q), n = run_hi(q) - plo;
    pitem = (int)threadIdx.x < 2 * n ? (int)threadIdx.x : -1;
    if (pitem >= 0) {
      const i32x4 *src = reinterpret_cast<const i32x4 *>(m.pos + plo + (pitem >> 1)) + (pitem & 1);
      preg = *src;
    }
  };
  auto deposit_pos = [&](int q) {
    if (pitem >= 0) gpos[((q & 3) * segmax) * 2 + pitem] = preg;
  };
  auto fetch_rows = [&](int q) {
    const int n = run_hi(q) - run_lo(q);
    ritem = (int)threadIdx.x < WPP * n ? (int)threadIdx.x : -1;
    if (ritem >= 0) {
      const int t = ritem / WPP, w = ritem - t * WPP;
      const int r0 = gpos[((q & 3) * segmax + t) * 2].y;  // staged record: node, r0, r1, slot
      const unsigned char *src;
      if (w < 6) src = reinterpret_cast<const unsigned char *>(m.S + r0 + w);
      else if (w < 8) src = reinterpret_cast<const unsigned char *>(m.lref + r0) + 16 * (w - 6);
      else src = reinterpret_cast<const unsigned char *>(m.ncos + r0) + 16 * (w - 8);
      i32x4 v;
      __builtin_memcpy(&v, src, 16);
      rreg = v;
    }
  };
  auto deposit_rows = [&](int q) {
    if (ritem >= 0) {
      const int t = ritem / WPP, w = ritem - t * WPP;
      grow[((q & 3) * segmax + t) * kGeoWords + w] = rreg;
    }
  };

  // first and last parallel with positions of this tile
  int qa = nseg, qb = -1;
  for (int q = 0; q < nseg; ++q) {
    if (run_hi(q) > run_lo(q)) {
      qa = min(qa, q);
      qb = q;
    }
  }
  if (qb < 0) return;
  for (int q = 0; q <= min(nseg - 1, qa + 1); ++q) {
    fetch(q);
    deposit(q);
  }
  fetch_pos(qa);
  deposit_pos(qa);
  if (qa + 1 < nseg) {
    fetch_pos(qa + 1);
    deposit_pos(qa + 1);
  }
  __syncthreads();
  fetch_rows(qa);
  deposit_rows(qa);
  __syncthreads();

  const int kc = min(lane, nvc - 1);  // lanes past the chunk read a valid entry
  const int s_l = first(kc);
  const bool lane_on = lane < nvc;
  for (int q = qa; q <= qb; ++q) {
    const bool pf = q + 2 < nseg;
    if (pf) {
      fetch(q + 2);
      fetch_pos(q + 2);
    }
    const bool rf = q + 1 < nseg;
    if (rf) fetch_rows(q + 1);
    const int plo = run_lo(q), phi = run_hi(q);
    const R *bq = buf + (q & 3) * slot_stride;
    const i32x4 *gp = gpos + (q & 3) * segmax * 2;
    const i32x4 *gr = grow + (q & 3) * segmax * kGeoWords;
    for (int p = plo + wave; p < phi; p += nw) {
      const int t = p - plo;
      const i32x4 w0 = gp[2 * t], w1 = gp[2 * t + 1];
      const int node = w0.x, n = w0.z - w0.y, selfslot = w0.w;
      double al, be;
      {
        const int a2[2] = {w1.x, w1.y}, b2[2] = {w1.z, w1.w};
        __builtin_memcpy(&al, a2, 8);
        __builtin_memcpy(&be, b2, 8);
      }
      if (!P::kVecOut) be = 0.0;
      const double ci = P::kVecIn ? cst(m.coslat)[node] : 0.0;
      constexpr int G = 6;
      double2 S[G];
      int lr[8];
      double cn[G];
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const i32x4 v = gr[t * kGeoWords + j];
        __builtin_memcpy(&S[j], &v, 16);
      }
      {
        const i32x4 a = gr[t * kGeoWords + 6], b = gr[t * kGeoWords + 7];
        lr[0] = a.x; lr[1] = a.y; lr[2] = a.z; lr[3] = a.w;
        lr[4] = b.x; lr[5] = b.y; lr[6] = b.z; lr[7] = b.w;
      }
      if (P::kVecIn) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const i32x4 v = gr[t * kGeoWords + 8 + k];
          __builtin_memcpy(&cn[2 * k], &v, 16);
        }
      } else {
#pragma unroll
        for (int j = 0; j < G; ++j) cn[j] = 0.0;
      }
      typename P::St st[NV];
      {
        const R xi = bq[selfslot * vpc + kc];
#pragma unroll
        for (int v = 0; v < NV; ++v) P::init(st[v], LV::get(xi, v), ci);
      }
      R xn[G];
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int l = lr[j] & ~kLrefPole;
        xn[j] = buf[((q + ((l >> 16) & 3) - 1) & 3) * slot_stride + (l & 0xffff) * vpc + kc];
      }
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const bool pole = (lr[j] & kLrefPole) != 0;
        if (j < kMinRow) {  // present in every row, never the pole edge
#pragma unroll
          for (int v = 0; v < NV; ++v) P::add(st[v], LV::get(xn[j], v), S[j], false, cn[j]);
          continue;
        }
        const bool use = j < n && !(P::kVecIn && pole);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          typename P::St tt = st[v];
          P::add(tt, LV::get(xn[j], v), S[j], pole, cn[j]);
          P::keep(st[v], tt, use);
        }
      }
      const i32x4 ro = make_rsrc(out + (size_t)node * L * (sizeof(Out) / sizeof(T)),
                                 (uint32_t)(L * sizeof(Out)));
      constexpr int W = NV * (int)sizeof(Out) / 4;
      int w[W];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const Out r = P::result(st[v], al, be);
        __builtin_memcpy(&w[v * (int)sizeof(Out) / 4], &r, sizeof(Out));
      }
      const int ob = lane_on ? s_l * (int)sizeof(Out) : kBufOff;
      buf_store_words<W>(w, ro, ob);
    }
    if (pf) {
      deposit(q + 2);
      deposit_pos(q + 2);
    }
    if (rf) deposit_rows(q + 1);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Wave-specialised sweep.  The same walk down a tile's band as k_sweepv, but
// the waves of a workgroup split the work: producer waves only move data
// into LDS, with buffer loads that write LDS directly (no registers, no
// deposit pass), and consumer waves only compute from LDS and store
// results.  One vector-memory counter per wave counts loads and stores
// alike and retires them in order; so a wave that both stored results and
// later waited for its next loads would wait for those stores too.  Here the
// consumers never wait on memory (their stores drain while the next
// parallels are computed) and the producers wait only for their own loads.
// The producers form two groups that take alternate runs: at step q the
// group of run q+3 loads its columns and packed records into its ring
// slots, and at the end of step q the other group waits for run q+2, which
// it issued one step earlier -- so every load has two steps to land.  The
// consumers compute the own positions of run q from runs q-1, q, q+1.  The
// roles run separate loops that meet at one workgroup barrier per step.
//
// A run's columns lie in its ring slot row by row, vpc 16-byte vectors each.
// A position's neighbours are named by their row in the whole ring (run r of
// a tile always takes slot r mod 5, so the rows are known when the mesh is
// built): one multiply-add turns a reference into an LDS address.
//
// Lanes.  An element is the least a lane computes: 8 bytes of a scalar
// column (one FP64 level, two FP32 ones), 16 of a vector column (the one-pass
// FP32 divergence and curl: 8, for its registers).  A position
// takes LPN lanes, lane h of them the elements h, h + LPN, ... (NE of them),
// so one decoding of a record serves NE elements, and every store
// instruction writes one contiguous run of the row.  Results go through
// plain stores: rows start at any multiple of the element size, and the L2
// merges the lines that two rows or two instructions share (streaming
// stores of such rows write them twice: 4.0 against 5.1 TB/s, whole rows).
// ---------------------------------------------------------------------------
// Per position: one 16-byte word of references ({own row | n << 16 | flags,
// rows 0 and 1, rows 2 and 3, rows 4 and 5}, one set for each cut of the
// tiles) and a packed record of 16-byte words: for scalar inputs {node, 0,
// alpha}, {beta, cos(lat)}, S[6] / 2; for vector inputs cos(lat) in beta's
// place and the neighbours' cos(lat) at the end.
constexpr int kSgeoWordsS = 8, kSgeoWordsV = 11;
// Elements per lane: at most what 128 registers hold (one workgroup of up to
// 1024 threads per compute unit).  FP32 vector inputs stop at three, since
// four spill 3 to 9 registers: O731, FP32 divergence, 110 levels, 1230 us
// with four of them and 870 with three, 64 levels 662 and 470; divergence and
// curl, 32 levels, 486 and 390.  (Five spill 2 to 4 of the FP64 divergence's
// and the FP32 gradient's and still win: 947 against 992 us, 80 levels, and
// 776 against 788, 130 levels.)
template <class T, int OP, bool DC>
constexpr int sweepw_max_ne() {
  return sizeof(T) == 8 ? (DC ? 3 : 5) : OP == OP_GRAD ? 5 : 3;
}
// Levels of an element.
template <class T, bool DC>
constexpr int sweepw_elem_levels() {
  return sizeof(T) == 8 || DC ? 1 : 2;
}
constexpr int kSweepwGroups = 2;     // producer groups (runs taken in turn)
constexpr int kSweepwGroupWaves = 2; // waves of a group
constexpr int kSweepwLead = kSweepwSlots - 2;     // run q + lead issued at step q; field
                                                  // ring: runs q-1 .. q+lead
constexpr int kSweepwGeoSlots = kSweepwLead + 1;  // record ring: runs q .. q+lead
// Lanes without an element read past their row: LPN * NE elements from its
// start, less than LPN (32) more than the plan's chunk has.  Rows of a shorter
// last chunk start earlier by more than they are shorter, so no read ends
// further than this past the space of its ring.
constexpr int kSweepwLdsTail = 32 * 16;

__device__ __forceinline__ void lds_dma16(const i32x4 &rsrc, void *lds_wave_base, int voff) {
  __amdgpu_buffer_rsrc_t r;
  __builtin_memcpy(&r, &rsrc, 16);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      r, (__attribute__((address_space(3))) void *)lds_wave_base, 16, voff, 0, 0, 0);
}

// A piece's table of runs, entry q in lane q of every wavefront: read once,
// then a step's entry comes by v_readlane.  (Read by scalar loads when a step
// needs them, the entries of most steps came from beyond the L2, a round trip
// on the path of every load and every step.)  Entries from 64 on, of bands
// taller than the library's, are read when needed.
__device__ __forceinline__ int4 cst_int4(const int4 *p, size_t i) {
  const ATLASX_CST int *d = cst(reinterpret_cast<const int *>(p));
  return make_int4(d[4 * i], d[4 * i + 1], d[4 * i + 2], d[4 * i + 3]);
}
__device__ __forceinline__ int2 cst_int2(const int2 *p, size_t i) {
  const ATLASX_CST int *d = cst(reinterpret_cast<const int *>(p));
  return make_int2(d[2 * i], d[2 * i + 1]);
}
struct RunTable {
  const int4 *src;
  int4 v;
  __device__ __forceinline__ RunTable(const int4 *p, int n, int lane)
      : src(p), v(p[min(lane, n - 1)]) {}
  __device__ __forceinline__ int4 operator()(int q) const {
    if (q >= 64) return cst_int4(src, q);
    return make_int4(__builtin_amdgcn_readlane(v.x, q), __builtin_amdgcn_readlane(v.y, q),
                     __builtin_amdgcn_readlane(v.z, q), __builtin_amdgcn_readlane(v.w, q));
  }
};
struct PosTable {
  const int2 *src;
  int2 v;
  __device__ __forceinline__ PosTable(const int2 *p, int n, int lane)
      : src(p), v(p[min(lane, n - 1)]) {}
  __device__ __forceinline__ int2 operator()(int q) const {
    if (q >= 64) return cst_int2(src, q);
    return make_int2(__builtin_amdgcn_readlane(v.x, q), __builtin_amdgcn_readlane(v.y, q));
  }
};

// The loads of a run's columns by one wavefront of a producer group of `nwv`:
// its i-th load instruction moves 64 items (node t of the run, vector k of
// the chunk) whose offsets from the run's first column are the same for
// every run, so they are computed once; a load then costs a few scalar
// instructions.  (With the offsets recomputed per load, issuing a step's
// loads took as long as their latency: O1280, 137 levels, FP64 divergence
// 5.12 -> 4.87 ms, gradient 4.59 -> 4.47, FP32 gradient 2.47 -> 2.36; the
// fused Laplacian's loads alone 4.87 -> 3.95.)  The sweep's ring slots are at
// most 32 KB, 16 load instructions for each of two wavefronts; the fused
// Laplacian's plan keeps to one wavefront's.
constexpr int kRunLoads = 16;
static_assert(kSweepwSlots * kRunLoads * 64 * 16 * kSweepwGroupWaves >= 160 * 1024,
              "the loads of a run fill the largest ring slot");
struct RunLoader {
  int rel[kRunLoads];
  int w, nwv, lane, nvc;
  uint32_t col_bytes;
  // (the last vector of a column ends with the column)
  __device__ __forceinline__ RunLoader(int w, int nwv, int lane, int nvc, int v0,
                                       uint32_t col_bytes)
      : w(w), nwv(nwv), lane(lane), nvc(nvc), col_bytes(col_bytes) {
    const int i0 = w * 64 + lane, di = nwv * 64;
    int t = i0 / nvc, k = i0 - t * nvc;
    const int dt = di / nvc, dk = di - dt * nvc;
#pragma unroll
    for (int i = 0; i < kRunLoads; ++i) {
      rel[i] = t * (int)col_bytes + min(16 * (v0 + k), (int)col_bytes - 16);
      t += dt;
      k += dk;
      if (k >= nvc) {
        k -= nvc;
        ++t;
      }
    }
  }
  // run f = {ring offset, ring size, first, length} of the field at `base`
  __device__ __forceinline__ void load(const unsigned char *base, const int4 &f,
                                       i32x4 *slot) const {
    const int nitems = f.w * nvc;
    const bool wraps = f.z + f.w > f.y;
    const unsigned char *ring = base + (size_t)f.x * col_bytes;
    const uint32_t start = (uint32_t)f.z * col_bytes, size = (uint32_t)f.y * col_bytes;
    const i32x4 rs = make_rsrc(wraps ? ring : ring + start, wraps ? size : (uint32_t)f.w * col_bytes);
#pragma unroll
    for (int i = 0; i < kRunLoads; ++i) {
      const int b = w + i * nwv;
      if (b * 64 >= nitems) break;
      int off = rel[i];
      if (wraps) {  // past the parallel's end: on from its first column
        const uint32_t o = (uint32_t)off + start;
        off = (int)min(o, o - size);
      }
      // lanes past the run's last item stay off: the words behind it belong
      // to the next slot
      if ((b + 1) * 64 <= nitems || b * 64 + lane < nitems) lds_dma16(rs, slot + b * 64, off);
    }
  }
  // `words` contiguous 16-byte words
  __device__ __forceinline__ void copy(const int4 *src, i32x4 *dst, int words) const {
    const i32x4 rs = make_rsrc(src, (uint32_t)words * 16u);
    for (int b = w; b * 64 < words; b += nwv)
      if ((b + 1) * 64 <= words || b * 64 + lane < words)
        lds_dma16(rs, dst + b * 64, (b * 64 + lane) * 16);
  }
};

// DC (OP = OP_DIV only): the curl of the same field as well, into out2,
// from the same loads; each output bitwise that of its own operator.
template <class T, int OP, int LPN, int NE, bool DC>
__global__ void __launch_bounds__(1024) k_sweepw(SweepView m, const int4 *__restrict__ geo,
                                                 const T *__restrict__ in, T *__restrict__ out,
                                                 T *__restrict__ out2, int nlev, int vpc,
                                                 int per_xcd) {
  static_assert(!DC || OP == OP_DIV, "the one-pass curl rides on the divergence");
  using P = Pol<T, OP>;
  using PC = Pol<T, OP_CURL>;
  using V = typename P::V;
  using Out = typename P::Out;
  constexpr int NV = 16 / (int)sizeof(V);          // levels per vector
  constexpr int EL = sweepw_elem_levels<T, DC>();
  constexpr int EB = EL * (int)sizeof(V);          // bytes of an element
  constexpr int EPV = 16 / EB;                     // elements per vector
  constexpr int GW = P::kVecIn ? kSgeoWordsV : kSgeoWordsS;
  constexpr int NPW = kSweepwGroups * kSweepwGroupWaves;
  constexpr int NPN = 64 / LPN;                    // positions per wavefront
  struct __align__(EB) Elem { V v[EL]; };
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int segmax = m.segmax, gcap = m.pmax * GW;
  i32x4 *fbuf = reinterpret_cast<i32x4 *>(smem_raw);  // [field slots][segmax][nvc]
  i32x4 *rbuf = fbuf + kSweepwSlots * segmax * vpc;    // [record slots][pmax] references
  i32x4 *gbuf = rbuf + kSweepwGeoSlots * m.pmax;       // [record slots][gcap] records
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int nvec = (nlev + NV - 1) / NV;
  const int nchunk = (nvec + vpc - 1) / vpc;
  const int tile = u / nchunk;
  const int c = u - tile * nchunk;
  if (tile >= m.ntiles) return;
  const int v0 = c * vpc;
  if (v0 >= nvec) return;
  const int nvc = min(vpc, nvec - v0);  // vectors in this chunk
  const int s0 = cst(m.tile_seg)[tile];
  const int nseg = cst(m.tile_seg)[tile + 1] - s0;
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(V));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const PosTable own(m.seg_pos + s0, nseg, lane);
  // first and last parallel with positions of this tile
  int qa = nseg, qb = -1;
  for (int q = 0; q < nseg; ++q) {
    const int2 sp = own(q);
    if (sp.y > sp.x) {
      qa = min(qa, q);
      qb = q;
    }
  }
  if (qb < 0) return;

  if (wave < NPW) {
    // ---- producers: group grp loads the runs r with r mod groups = grp ----
    const int grp = wave / kSweepwGroupWaves, gwave = wave - grp * kSweepwGroupWaves;
    const unsigned char *field = reinterpret_cast<const unsigned char *>(in);
    const RunTable runs(m.seg + s0, nseg, lane);
    const RunLoader ld(gwave, kSweepwGroupWaves, lane, nvc, v0, col_bytes);
    // columns, references and records of run q into the ring slots of q
    auto load = [&](int q) {
      ld.load(field, runs(q), fbuf + (q % kSweepwSlots) * segmax * nvc);
      const int2 sp = own(q);
      const int slot = q % kSweepwGeoSlots, n = sp.y - sp.x;
      ld.copy(m.refs + sp.x, rbuf + slot * m.pmax, n);
      ld.copy(geo + (size_t)sp.x * GW, gbuf + slot * gcap, n * GW);
    };
    // prologue: runs qa-1 .. qa+1 (waited), then qa+2 .. qa+lead-1, by their
    // groups (run r is waited for at the end of step r-2)
    for (int q = max(0, qa - 1); q <= min(nseg - 1, qa + 1); ++q)
      if (q % kSweepwGroups == grp) load(q);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (int r = qa + 2; r < min(nseg, qa + kSweepwLead); ++r)
      if (r % kSweepwGroups == grp) load(r);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    for (int q = qa; q <= qb; ++q) {
      if (q + kSweepwLead < nseg && (q + kSweepwLead) % kSweepwGroups == grp)
        load(q + kSweepwLead);
      // run q+2 (issued lead-2 steps ago by its group, which has issued
      // nothing since) is in LDS before step q+1 reads it
      if ((q + 2) % kSweepwGroups == grp) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    // loads of runs past qb + 2 are never read; let them land before exit
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }

  // ---- consumers ----------------------------------------------------------
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  const int cw = wave - NPW, ncw = nw - NPW;
  const int sub = lane / LPN, hl = lane - sub * LPN;
  const int nel = nvc * EPV;  // elements in this chunk
  const uint32_t rowb = (uint32_t)nvc * 16u;
  const unsigned char *lane_base = smem_raw + hl * EB;
  // byte offset in the output row of the lane's element g: its vector is
  // clamped inside the column, so the last one may repeat levels
  int off_g[NE];
#pragma unroll
  for (int g = 0; g < NE; ++g) {
    const int e = hl + g * LPN;
    off_g[g] = (min(NV * (v0 + e / EPV), nlev - NV) + EL * (e % EPV)) * (int)sizeof(Out);
  }
  const size_t row_out = L * sizeof(Out);

  // the sums and results of one position; FULL: six incidences, none a pole
  // edge (nearly every position), so nothing is selected
  auto position = [&](const i32x4 *rec, const i32x4 &ref, auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    // (keeps the compiler from hoisting the two instances' common reads, all
    // six neighbours', above the branch between them)
    if constexpr (!FULL) asm volatile("" ::: "memory");
    const i32x4 w0 = rec[0], w1 = rec[1];
    double al, sc;  // alpha; beta or cos(lat)
    {
      const int a2[2] = {w0.z, w0.w}, b2[2] = {w1.x, w1.y};
      __builtin_memcpy(&al, a2, 8);
      __builtin_memcpy(&sc, b2, 8);
    }
    const int flags = ref.x;
    const uint32_t rw[6] = {(uint32_t)ref.y & 0xffffu, (uint32_t)ref.y >> 16,
                            (uint32_t)ref.z & 0xffffu, (uint32_t)ref.z >> 16,
                            (uint32_t)ref.w & 0xffffu, (uint32_t)ref.w >> 16};
    typename P::St st[NE][EL];
    typename PC::St stc[DC ? NE : 1][EL];
    const unsigned char *self = lane_base + __umul24((uint32_t)flags & 0xffffu, rowb);
#pragma unroll
    for (int g = 0; g < NE; ++g) {
      const Elem x = *reinterpret_cast<const Elem *>(self + g * LPN * EB);
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        P::init(st[g][e], x.v[e], sc);
        if constexpr (DC) PC::init(stc[g][e], x.v[e], sc);
      }
    }
    // Neighbour j + 1 is read while neighbour j is added.  With many
    // elements the reads must not move further up (all six neighbours at
    // once would spill).
    Elem x[2][NE];
    auto read = [&](int j) {
      const unsigned char *col = lane_base + __umul24(rw[j], rowb);
#pragma unroll
      for (int g = 0; g < NE; ++g)
        x[j & 1][g] = *reinterpret_cast<const Elem *>(col + g * LPN * EB);
    };
    read(0);
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (j < 5) read(j + 1);
      double2 Sh;
      {
        const i32x4 v = rec[2 + j];
        __builtin_memcpy(&Sh, &v, 16);
      }
      double cn = 0.0;
      if constexpr (P::kVecIn) __builtin_memcpy(&cn, reinterpret_cast<const double *>(rec + 8) + j, 8);
      const bool pole = !FULL && j >= kMinRow && (flags & (kSgeoPole << j)) != 0;
      const bool use = FULL || j < kMinRow || (j < ((flags >> 16) & 7) && !(P::kVecIn && pole));
#pragma unroll
      for (int g = 0; g < NE; ++g) {
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          const V xn = x[j & 1][g].v[e];
          if (FULL || j < kMinRow) {
            P::add_half(st[g][e], xn, Sh, false, cn);
            if constexpr (DC) PC::add_half(stc[g][e], xn, Sh, false, cn);
          } else {
            typename P::St tt = st[g][e];
            P::add_half(tt, xn, Sh, pole, cn);
            P::keep(st[g][e], tt, use);
            if constexpr (DC) {
              typename PC::St tc = stc[g][e];
              PC::add_half(tc, xn, Sh, pole, cn);
              PC::keep(stc[g][e], tc, use);
            }
          }
        }
      }
      if constexpr (NE * EL * (DC ? 2 : 1) >= 3) __builtin_amdgcn_sched_barrier(0);
    }
    // (the sums are formed here, not in the branch around each store)
#pragma unroll
    for (int g = 0; g < NE; ++g)
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        P::settle(st[g][e]);
        if constexpr (DC) PC::settle(stc[g][e]);
      }
    struct OutElem { Out v[EL]; };
    const size_t base = (size_t)(uint32_t)w0.x * row_out;
#pragma unroll
    for (int g = 0; g < NE; ++g) {
      if (hl + g * LPN < nel) {
        OutElem o;
#pragma unroll
        for (int e = 0; e < EL; ++e) o.v[e] = P::result_half(st[g][e], al, sc);
        __builtin_memcpy(reinterpret_cast<unsigned char *>(out) + base + off_g[g], &o, sizeof(o));
        if constexpr (DC) {
#pragma unroll
          for (int e = 0; e < EL; ++e) o.v[e] = PC::result_half(stc[g][e], al, sc);
          __builtin_memcpy(reinterpret_cast<unsigned char *>(out2) + base + off_g[g], &o, sizeof(o));
        }
      }
    }
  };
  for (int q = qa; q <= qb; ++q) {
    const int2 sp = own(q);
    const int n = sp.y - sp.x;
    const i32x4 *rq = rbuf + (q % kSweepwGeoSlots) * m.pmax;
    const i32x4 *gq = gbuf + (q % kSweepwGeoSlots) * gcap;
    for (int t = NPN * cw + sub; t < n; t += NPN * ncw) {
      const i32x4 ref = rq[t];
      if (__builtin_amdgcn_ballot_w64((ref.x & kSgeoFull) == 0) == 0)
        position(gq + t * GW, ref, std::true_type{});
      else
        position(gq + t * GW, ref, std::false_type{});
    }
    // this step's LDS reads are done before the producers refill a slot
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// The instance for LPN lanes per position (8, 16 or 32) and NE elements per
// lane (1 .. sweepw_max_ne).
template <class T, int OP, bool DC, int LPN, int NE = 1>
void (*sweepw_kernel_ne(int ne))(SweepView, const int4 *, const T *, T *, T *, int, int, int) {
  if constexpr (NE < sweepw_max_ne<T, OP, DC>()) {
    if (ne > NE) return sweepw_kernel_ne<T, OP, DC, LPN, NE + 1>(ne);
  }
  return &k_sweepw<T, OP, LPN, NE, DC>;
}
template <class T, int OP, bool DC>
auto sweepw_kernel(int lpn, int ne) {
  return lpn == 8    ? sweepw_kernel_ne<T, OP, DC, 8>(ne)
         : lpn == 16 ? sweepw_kernel_ne<T, OP, DC, 16>(ne)
                     : sweepw_kernel_ne<T, OP, DC, 32>(ne);
}

// ---------------------------------------------------------------------------
// Fused Laplacian: one pass over the two-ring plan.  A workgroup owns one
// tile and one chunk of lane vectors and walks the tile's window of
// parallels.  At step q it forms the gradient at every node of the g-run of
// parallel q from the field runs q-1, q, q+1 (LDS) into a 4-slot LDS ring,
// and the divergence of those gradients at the tile's own positions of
// parallel q-2 from the g-runs q-3, q-2, q-1 (the ring slot written at step
// q held the g-run of q-4, last read at step q-1).  Meanwhile it loads the
// field run of parallel q+2 and the packed geometry of step q+1 (records of
// the g-run q+1 and of the own positions of parallel q-1) into registers
// and deposits them in LDS after the compute, so the compute reads nothing
// but LDS.  Every gradient goes through the gradient policy and is rounded
// to its output type exactly as the two-pass form stores it, and every
// divergence through the divergence policy: the result is bitwise that of
// the two passes.
// ---------------------------------------------------------------------------
constexpr int kGGeoWords = 10;  // packed gradient-node record (16-byte words):
                                // S[6] / 2, refs[8], (alpha, beta),
                                // (f self, n, cos lat)
constexpr int kLGeoWords = 13;  // packed own-position record: S[6] / 2,
                                // refs[8], (alpha, cos lat), (node, n, g self),
                                // ncos[6] (FP32 only: the FP64 kernel stages
                                // the first kLGeoWords64 words)
constexpr int kLGeoWords64 = 10;
constexpr int kGeoEpt = 2;      // geometry words a thread stages per step
constexpr int kLsweepEpt = 2;   // field lane vectors a thread stages per step

// FP64 steps of the fused Laplacian with halved normals Sh = S / 2 (exact):
// (xi + xn) Sh rounds like S (0.5 (xi + xn)), so these give the bits of
// Pol<double, OP_GRAD>::add and PolDC64<OP_DIV>::add (operands not
// subnormal).  For the divergence the second component arrives as
// w = v cos(lat), the product PolDC64 forms from v and the node's cos(lat).
__device__ __forceinline__ void grad_add_half(Pol<double, OP_GRAD>::St &s, double xn,
                                              const double2 &Sh, bool pole) {
  const double xe = s.xi + xn;
  if (!pole) s.gl = s.gl + Sh.x * xe;
  s.gt = s.gt + Sh.y * xe;
}
__device__ __forceinline__ void div_init_w(PolDC64<OP_DIV>::St &s, const v2d &uw) {
  s.ai = uw.x;
  s.bi = uw.y;
  s.acc = 0.0;
}
__device__ __forceinline__ void div_add_half_w(PolDC64<OP_DIV>::St &s, const v2d &uw,
                                               const double2 &Sh) {
  const double ae = s.ai + uw.x, be = s.bi + uw.y;
  s.acc = s.acc + (Sh.x * ae + Sh.y * be);
}
// (overloads for the FP32 instantiation, never called)
__device__ __forceinline__ void grad_add_half(Pol<float, OP_GRAD>::St &, float, const double2 &,
                                              bool) {}
__device__ __forceinline__ void div_init_w(PolDC32<OP_DIV>::St &, const v2f &) {}
__device__ __forceinline__ void div_add_half_w(PolDC32<OP_DIV>::St &, const v2f &,
                                               const double2 &) {}

template <class T, int NV, int EPT, int NL>
__global__ void __launch_bounds__(1024) k_lsweep(DevMesh m, const T *__restrict__ in,
                                                 T *__restrict__ out, int nlev, int vpc,
                                                 int ntiles, int per_xcd, int lpn) {
  using PG = Pol<T, OP_GRAD>;
  using PD = Pol<T, OP_DIV>;
  using LF = LaneVec<T, NV>;
  using RF = typename LF::raw;         // NV levels of the field
  using GV = typename PD::V;           // gradient (zonal, meridional) of one level
  using LG = LaneVec<GV, NV>;
  using RG = typename LG::raw;         // NV levels of the gradient
  static_assert(sizeof(typename PG::Out) == sizeof(GV), "gradient output type");
  constexpr int G = 6;
  // FP64 keeps the second gradient component multiplied by cos(lat) in the
  // ring (the divergence's b = v cos(lat), formed once per node instead of
  // once per incidence) and uses the halved normals as they are
  constexpr bool F64 = sizeof(T) == 8;
  constexpr int LGW = F64 ? kLGeoWords64 : kLGeoWords;  // own-position words staged
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int fmax = m.l2_fmax, gmax = m.l2_gmax;
  const int gw = gmax * kGGeoWords;                          // g part of a geometry slot
  const int geo_stride = gw + m.l2_pmax * LGW;               // words per geometry slot
  // the gradient ring holds each lane vector as two planes of its first
  // and second half (consecutive lanes then read consecutive 16-byte words)
  static_assert(sizeof(RG) == 2 * sizeof(RF), "gradient lane vector = two field lane vectors");
  RF *fbuf = reinterpret_cast<RF *>(smem_raw);               // [4][fmax][vpc]
  RF *gbuf = fbuf + 4 * fmax * vpc;                          // [4][gmax][2][vpc]
  i32x4 *geo = reinterpret_cast<i32x4 *>(gbuf + 8 * gmax * vpc);  // [2][geo_stride]
  const int fstride = fmax * vpc, gstride = 2 * gmax * vpc;
  auto gload = [&](int at) {  // at: ring slot offset + node * 2 * vpc + lane vector
    RG r;
    __builtin_memcpy(&r, &gbuf[at], sizeof(RF));
    __builtin_memcpy(reinterpret_cast<char *>(&r) + sizeof(RF), &gbuf[at + vpc], sizeof(RF));
    return r;
  };
  // chunk-minor order (as in k_sweepv): a tile's chunks share its geometry
  // and boundary lines through one XCD's L2
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int nvec = (nlev + NV - 1) / NV;
  const int nchunk = (nvec + vpc - 1) / vpc;
  const int tile = u / nchunk;
  const int c = u - tile * nchunk;
  if (tile >= ntiles) return;
  const int v0 = c * vpc;
  if (v0 >= nvec) return;
  const int nvc = min(vpc, nvec - v0);
  const int k0 = cst(m.l2_tile_seg)[tile];
  const int W = cst(m.l2_tile_seg)[tile + 1] - k0;
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(T));
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  auto first = [&](int k) { return min(NV * (v0 + k), nlev - NV); };

  // ---- field runs: item = (node t of the run, lane vector k); a thread's
  // items are the same every step
  RF regs[EPT];
  int it_t[EPT], it_off[EPT], it_lds[EPT];  // it_off: byte offset of (t, k) from the run start
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int i = threadIdx.x + e * (int)blockDim.x;
    const int t = i / nvc, k = i - t * nvc;
    it_t[e] = t;
    it_off[e] = t * (int)col_bytes + first(k) * (int)sizeof(T);
    it_lds[e] = t * vpc + k;
  }
  int run_len = 0;
  auto fetch = [&](int q) {
    const int4 f = cst_int4(m.l2_fseg, k0 + q);  // {ring offset, ring size, first, length}
    run_len = f.w;
    const i32x4 rs = make_rsrc(in + (size_t)f.x * L, (uint32_t)f.y * col_bytes);
    const int start = f.z * (int)col_bytes, wrap = f.y * (int)col_bytes;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      int off = start + it_off[e];
      if (off >= wrap) off -= wrap;  // the run wraps round the parallel
      regs[e] = buf_load<RF>(rs, it_t[e] < run_len ? off : kBufOff);
    }
  };
  auto deposit = [&](int q) {
    RF *b = fbuf + (q & 3) * fstride;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (it_t[e] < run_len) b[it_lds[e]] = regs[e];
  };
  // ---- packed geometry of step q: the g-run records of parallel q (words
  // [0, glen * kGGeoWords)) and the own-position records of parallel q - 2
  // (from word gw on), into slot q & 1
  // On deposit, the references of a record become LDS element offsets for
  // the step it serves (ring slot and run slot resolved, the pole flag
  // kept), and the self slots likewise, so the compute adds only the lane.
  // A thread's geometry items are fixed: item i < gw is word i % kGGeoWords
  // of g record i / kGGeoWords; item gw + j is word j % kLGeoWords of own
  // position record j / kLGeoWords.
  i32x4 greg[kGeoEpt];
  int gdst[kGeoEpt], gkind[kGeoEpt];  // kind: 0 plain, 1 f-refs, 2 f-self, 3 g-refs, 4 g-self
  int grec[kGeoEpt], gword[kGeoEpt];  // record index (-1: none) and word
  bool gisg[kGeoEpt], gon[kGeoEpt];
#pragma unroll
  for (int e = 0; e < kGeoEpt; ++e) {
    const int i = threadIdx.x + e * (int)blockDim.x;
    gdst[e] = i;
    gisg[e] = i < gw;
    if (i < gw) {
      grec[e] = i / kGGeoWords;
      gword[e] = i - grec[e] * kGGeoWords;
      gkind[e] = (gword[e] == 6 || gword[e] == 7) ? 1 : (gword[e] == 9) ? 2 : 0;
    } else if (i < geo_stride) {
      grec[e] = (i - gw) / LGW;
      gword[e] = (i - gw) - grec[e] * LGW;
      gkind[e] = (gword[e] == 6 || gword[e] == 7) ? 3 : (gword[e] == 9) ? 4 : 0;
    } else {
      grec[e] = -1;
      gword[e] = 0;
      gkind[e] = 0;
    }
    gon[e] = false;
  }
  auto fref = [&](int r, int qq) {
    const int l = r & ~kLrefPole;
    return (r & kLrefPole) | (((qq + ((l >> 16) & 3) - 1) & 3) * fstride + (l & 0xffff) * vpc);
  };
  auto gref = [&](int r, int qq) {
    const int l = r & ~kLrefPole;
    return (r & kLrefPole) | (((qq + ((l >> 16) & 3) - 1) & 3) * gstride + (l & 0xffff) * 2 * vpc);
  };
  auto fetch_geo = [&](int q) {
    int ng = 0, gb = 0, p0 = 0, np = 0;  // records of each kind this step
    if (q < W) {
      const int4 gs = cst_int4(m.l2_gseg, k0 + q);
      ng = gs.y;
      gb = gs.z;
    }
    if (q >= 2 && q - 2 < W) {
      const int2 sp = cst_int2(m.l2_seg_pos, k0 + q - 2);
      p0 = sp.x;
      np = sp.y - sp.x;
    }
#pragma unroll
    for (int e = 0; e < kGeoEpt; ++e) {
      gon[e] = grec[e] >= 0 && grec[e] < (gisg[e] ? ng : np);
      if (gon[e]) {
        const int4 *src = gisg[e] ? m.l2_ggeo + (size_t)(gb + grec[e]) * kGGeoWords
                                  : m.l2_lgeo + (size_t)(p0 + grec[e]) * kLGeoWords;
        greg[e] = *reinterpret_cast<const i32x4 *>(src + gword[e]);
      }
    }
  };
  auto deposit_geo = [&](int q) {  // records of step q: g-run q, own positions of q - 2
    i32x4 *g = geo + (q & 1) * geo_stride;
#pragma unroll
    for (int e = 0; e < kGeoEpt; ++e) {
      if (!gon[e]) continue;
      i32x4 v = greg[e];
      if (gkind[e] == 1) {
        v.x = fref(v.x, q); v.y = fref(v.y, q); v.z = fref(v.z, q); v.w = fref(v.w, q);
      } else if (gkind[e] == 2) {
        v.x = (q & 3) * fstride + v.x * vpc;
      } else if (gkind[e] == 3) {
        v.x = gref(v.x, q - 2); v.y = gref(v.y, q - 2); v.z = gref(v.z, q - 2); v.w = gref(v.w, q - 2);
      } else if (gkind[e] == 4) {
        v.z = ((q - 2) & 3) * gstride + v.z * 2 * vpc;
      }
      g[gdst[e]] = v;
    }
  };

  for (int q = 0; q < min(W, 2); ++q) {
    fetch(q);
    deposit(q);
  }
  fetch_geo(0);
  deposit_geo(0);
  __syncthreads();

  // lpn lanes per node, 64 / lpn nodes per wavefront (lanes past the last
  // whole group idle); lane hl of a group walks the chunk's lane vectors
  // hl, hl + lpn, ... (NL of them, lpn * NL >= nvc) with the node's
  // geometry in registers, so one broadcast read of a record serves
  // 64 / lpn nodes and NL lane vectors
  const int npw = 64 / lpn;
  const int sub = lane / lpn;
  const int hl = lane - sub * lpn;
  const bool sub_on = sub < npw;
  for (int q = 0; q < W + 2; ++q) {
    const bool pf = q + 2 < W;
    if (pf) fetch(q + 2);
    const bool gf = q + 1 < W + 2;
    if (gf) fetch_geo(q + 1);
    const i32x4 *gq = geo + (q & 1) * geo_stride;
    // ---- gradients at the g-run of parallel q
    if (q < W) {
      const int glen = sub_on ? cst_int4(m.l2_gseg, k0 + q).y : 0;
      for (int s = npw * wave + sub; s < glen; s += npw * nw) {
        const i32x4 *r = gq + s * kGGeoWords;
        double2 S[G];  // halved normals (FP64), the normals (FP32)
        int lr[8];
#pragma unroll
        for (int j = 0; j < G; ++j) {
          __builtin_memcpy(&S[j], &r[j], 16);
          if constexpr (!F64) S[j] = make_double2(S[j].x + S[j].x, S[j].y + S[j].y);
        }
        {
          const i32x4 a = r[6], b = r[7];
          lr[0] = a.x; lr[1] = a.y; lr[2] = a.z; lr[3] = a.w;
          lr[4] = b.x; lr[5] = b.y; lr[6] = b.z; lr[7] = b.w;
        }
        double al, be;
        {
          const i32x4 w8 = r[8];
          const int a2[2] = {w8.x, w8.y}, b2[2] = {w8.z, w8.w};
          __builtin_memcpy(&al, a2, 8);
          __builtin_memcpy(&be, b2, 8);
        }
        const i32x4 w9 = r[9];
        const int fself = w9.x, n = w9.y;  // fself: LDS offset
        double cosg;
        {
          const int c2[2] = {w9.z, w9.w};
          __builtin_memcpy(&cosg, c2, 8);
        }
#pragma unroll 1
        for (int i = 0; i < NL; ++i) {
          const int k = hl + lpn * i;
          const int kc = min(k, nvc - 1);  // lanes past the chunk read a valid entry
          typename PG::St st[NV];
          {
            const RF xi = fbuf[fself + kc];
#pragma unroll
            for (int v = 0; v < NV; ++v) PG::init(st[v], LF::get(xi, v), 0.0);
          }
          RF xn[G];
#pragma unroll
          for (int j = 0; j < G; ++j) xn[j] = fbuf[(lr[j] & ~kLrefPole) + kc];
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const bool pole = (lr[j] & kLrefPole) != 0;
            if (j < kMinRow) {  // present in every row, never the pole edge
#pragma unroll
              for (int v = 0; v < NV; ++v) {
                if constexpr (F64) grad_add_half(st[v], LF::get(xn[j], v), S[j], false);
                else PG::add(st[v], LF::get(xn[j], v), S[j], false, 0.0);
              }
              continue;
            }
            const bool use = j < n;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              typename PG::St tt = st[v];
              if constexpr (F64) grad_add_half(tt, LF::get(xn[j], v), S[j], pole);
              else PG::add(tt, LF::get(xn[j], v), S[j], pole, 0.0);
              PG::keep(st[v], tt, use);
            }
          }
          RG g;
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const typename PG::Out o = PG::result(st[v], al, be);
            g.e[2 * v] = o.x;
            if constexpr (F64) g.e[2 * v + 1] = o.y * cosg;  // v cos(lat), as the divergence forms it
            else g.e[2 * v + 1] = o.y;
          }
          if (k < nvc) {
            RF *d = gbuf + (q & 3) * gstride + s * 2 * vpc + kc;
            __builtin_memcpy(d, &g, sizeof(RF));
            __builtin_memcpy(d + vpc, reinterpret_cast<const char *>(&g) + sizeof(RF), sizeof(RF));
          }
        }
      }
    }
    // The staged loads go to LDS here, between the two phases: the slots
    // they fill (field ring (q + 2) mod 4, geometry slot (q + 1) mod 2) are
    // read by neither phase of this step, the gradient phase has hidden
    // their latency, and the wait for them comes before this step's output
    // stores (vector memory operations retire in issue order).
    if (pf) deposit(q + 2);
    if (gf) deposit_geo(q + 1);
    // ---- Laplacian at the own positions of parallel q - 2
    if (q >= 2) {
      const int q2 = q - 2;
      const int2 sp = cst_int2(m.l2_seg_pos, k0 + q2);
      const int nown = sub_on ? sp.y - sp.x : 0;
      for (int t = npw * wave + sub; t < nown; t += npw * nw) {
        const i32x4 *r = gq + gw + t * LGW;
        double2 S[G];  // halved normals (FP64), the normals (FP32)
        int lr[8];
        double cn[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
          __builtin_memcpy(&S[j], &r[j], 16);
          if constexpr (!F64) S[j] = make_double2(S[j].x + S[j].x, S[j].y + S[j].y);
        }
        {
          const i32x4 a = r[6], b = r[7];
          lr[0] = a.x; lr[1] = a.y; lr[2] = a.z; lr[3] = a.w;
          lr[4] = b.x; lr[5] = b.y; lr[6] = b.z; lr[7] = b.w;
        }
        if constexpr (!F64) {
#pragma unroll
          for (int k = 0; k < 3; ++k) __builtin_memcpy(&cn[2 * k], &r[10 + k], 16);
        } else {
#pragma unroll
          for (int j = 0; j < G; ++j) cn[j] = 0.0;
        }
        double al, ci;
        {
          const i32x4 w8 = r[8];
          const int a2[2] = {w8.x, w8.y}, c2[2] = {w8.z, w8.w};
          __builtin_memcpy(&al, a2, 8);
          __builtin_memcpy(&ci, c2, 8);
        }
        const i32x4 w9 = r[9];
        const int node = w9.x, n = w9.y, self = w9.z;  // self: LDS offset
#pragma unroll 1
        for (int i = 0; i < NL; ++i) {
          const int k = hl + lpn * i;
          const int kc = min(k, nvc - 1);
          typename PD::St st[NV];
          {
            const RG gi = gload(self + kc);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              if constexpr (F64) div_init_w(st[v], LG::get(gi, v));
              else PD::init(st[v], LG::get(gi, v), ci);
            }
          }
          RG gn[G];
#pragma unroll
          for (int j = 0; j < G; ++j) gn[j] = gload((lr[j] & ~kLrefPole) + kc);
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const bool pole = (lr[j] & kLrefPole) != 0;
            if (j < kMinRow) {
#pragma unroll
              for (int v = 0; v < NV; ++v) {
                if constexpr (F64) div_add_half_w(st[v], LG::get(gn[j], v), S[j]);
                else PD::add(st[v], LG::get(gn[j], v), S[j], false, cn[j]);
              }
              continue;
            }
            const bool use = j < n && !pole;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
              typename PD::St tt = st[v];
              if constexpr (F64) div_add_half_w(tt, LG::get(gn[j], v), S[j]);
              else PD::add(tt, LG::get(gn[j], v), S[j], pole, cn[j]);
              PD::keep(st[v], tt, use);
            }
          }
          constexpr int WD = NV * (int)sizeof(T) / 4;
          struct Words { int v[WD]; } o;
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            const T x = PD::result(st[v], al, 0.0);
            __builtin_memcpy(&o.v[v * (int)sizeof(T) / 4], &x, sizeof(T));
          }
          if (k < nvc) *reinterpret_cast<Words *>(out + (size_t)node * L + first(kc)) = o;
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Fused Laplacian, wave-specialised: the register-staged kernel above waits
// at every parallel for the loads it issued one parallel earlier, one
// memory round trip per step.  Here, as in the wave-specialised sweep, two
// producer groups of one wavefront load straight into LDS two steps ahead
// and never store, and the consumer wavefronts only compute and store.
//
// Step q forms the gradients of the g-run of parallel q (from field runs
// q-1, q, q+1) into gradient slot q mod 4 and the Laplacian of the own
// positions of parallel q-2 (from gradient runs q-3 .. q-1, finished in
// earlier steps), so the two share the wavefronts with one barrier a step.
// Load set k = {field run k+1, records of the g-run k, its references, the
// references of the own positions of parallel k-2} is issued at step k-2 by
// group k mod 2 and waited for by that group at the end of step k-1: field
// and record rings of five slots, reference rings of three.  A position's
// record serves its gradient and, two steps later, its divergence.
// References are rows of the rings (a parallel's slot is known when the mesh
// is built), so nothing is resolved at run time.  Lanes and elements as in
// the sweep; FP64 keeps the second gradient component multiplied by
// cos(lat) (the divergence's b = v cos(lat), formed once per node), FP32
// keeps the rounded components and the nodes' cos(lat) beside them.
//
// O1280, 137 levels, against one barrier per phase, references resolved by
// the producers and selects on every row: FP64 8.26 -> 7.20 ms, FP32 6.20 ->
// 4.85; 10 levels, FP64, 1.83 -> 1.03.  With no gradients it takes 5.6 ms,
// with no divergences 5.6, with neither (loads and barriers) 3.95: the bound
// is the LDS, which serves 35 reads of a column's elements and ten of a
// record's words for each wavefront of positions and each phase.
// ---------------------------------------------------------------------------
constexpr int kLswGroupWaves = 1, kLswProducers = 2 * kLswGroupWaves;
constexpr int kLswBlock = 768;  // at most (three wavefronts per SIMD: 168 registers)
constexpr int kLswRecSlots = 5, kLswRefSlots = 3;
constexpr int kLswMaxNe = 5;

template <class T, int LPN, int NE>
__global__ void __launch_bounds__(kLswBlock) k_lsweepw(LaplView m, const int4 *__restrict__ geo,
                                                  const T *__restrict__ in, T *__restrict__ out,
                                                  int nlev, int vpc, int per_xcd) {
  using PG = Pol<T, OP_GRAD>;
  using PD = Pol<T, OP_DIV>;
  using GV = typename PD::V;                  // gradient of one level
  constexpr bool F64 = sizeof(T) == 8;
  constexpr int NV = 16 / (int)sizeof(T);     // levels per vector
  constexpr int EL = 8 / (int)sizeof(T);      // levels per element
  constexpr int NPN = 64 / LPN;               // positions per wavefront
  constexpr int GW = kSgeoWordsS;
  struct __align__(8) FElem { T v[EL]; };
  struct __align__(16) GElem { GV v[EL]; };
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int fmax = m.fmax, gmax = m.gmax, pmax = m.pmax;
  i32x4 *fbuf = reinterpret_cast<i32x4 *>(smem_raw);   // [field slots][fmax][nvc]
  i32x4 *gbuf = fbuf + kLswFieldSlots * fmax * vpc;     // [gradient slots][gmax][2 nvc]
  i32x4 *recs = gbuf + kLswGradSlots * gmax * 2 * vpc;  // [record slots][gmax][GW]
  i32x4 *gref = recs + kLswRecSlots * gmax * GW;        // [reference slots][gmax]
  i32x4 *oref = gref + kLswRefSlots * gmax;             // [reference slots][pmax]
  double *cosb = reinterpret_cast<double *>(oref + kLswRefSlots * pmax);  // FP32: [4][gmax]
  const int u = xcd_tile(blockIdx.x, per_xcd);
  const int nvec = (nlev + NV - 1) / NV;
  const int nchunk = (nvec + vpc - 1) / vpc;
  const int tile = u / nchunk;
  const int c = u - tile * nchunk;
  if (tile >= m.ntiles) return;
  const int v0 = c * vpc;
  if (v0 >= nvec) return;
  const int nvc = min(vpc, nvec - v0);
  const int k0 = cst(m.tile_seg)[tile];
  const int W = cst(m.tile_seg)[tile + 1] - k0;
  const size_t L = (size_t)nlev;
  const uint32_t col_bytes = (uint32_t)(L * sizeof(T));
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const RunTable gruns(m.gseg + k0, W, lane);  // {first, length, first reference, 0}
  const PosTable positions(m.seg_pos + k0, W, lane);
  auto glen = [&](int q) { return q < W ? gruns(q).y : 0; };
  auto own = [&](int q) { return q >= 0 && q < W ? positions(q) : make_int2(0, 0); };
  // first parallel with gradients, last with own positions
  int qa = W, qb = -1;
  for (int q = 0; q < W; ++q) {
    if (glen(q) > 0) qa = min(qa, q);
    const int2 sp = own(q);
    if (sp.y > sp.x) qb = q;
  }
  if (qb < 0) return;

  if (wave < kLswProducers) {
    const int grp = wave / kLswGroupWaves, gwave = wave % kLswGroupWaves;
    const unsigned char *field = reinterpret_cast<const unsigned char *>(in);
    const RunTable fruns(m.fseg + k0, W, lane);  // {ring offset, ring size, first, length}
    const RunLoader ld(gwave, kLswGroupWaves, lane, nvc, v0, col_bytes);
    auto load_f = [&](int q) {
      if (q >= 0 && q < W) ld.load(field, fruns(q), fbuf + (q % kLswFieldSlots) * fmax * nvc);
    };
    // records and references of set k
    auto load_g = [&](int k) {
      if (k < W) {
        const int4 f = fruns(k), g = gruns(k);
        i32x4 *slot = recs + (k % kLswRecSlots) * gmax * GW;
        const int4 *first = geo + (size_t)(f.x + g.x) * GW;
        const int head = min(g.y, f.y - g.x);  // the run may wrap round the parallel
        ld.copy(first, slot, head * GW);
        if (head < g.y) ld.copy(geo + (size_t)f.x * GW, slot + head * GW, (g.y - head) * GW);
        ld.copy(m.grefs + g.z, gref + (k % kLswRefSlots) * gmax, g.y);
      }
      const int2 sp = own(k - 2);
      ld.copy(m.orefs + sp.x, oref + (k % kLswRefSlots) * pmax, sp.y - sp.x);
    };
    // prologue: the runs before set qa, and set qa (waited), then set
    // qa + 1, each by its group
    for (int q = qa - 1; q <= qa + 1; ++q)
      if ((q & 1) == grp) load_f(q);
    if ((qa & 1) == grp) load_g(qa);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (((qa + 1) & 1) == grp) {
      load_f(qa + 2);
      load_g(qa + 1);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    for (int q = qa; q <= qb + 2; ++q) {
      if ((q & 1) == grp) {
        load_f(q + 3);
        load_g(q + 2);
      }
      // set q + 1 lands before step q + 1
      if (((q + 1) & 1) == grp) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }

  // ---- consumers ------------------------------------------------------------
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  const int cw = wave - kLswProducers, ncw = nw - kLswProducers;
  const int sub = lane / LPN, hl = lane - sub * LPN;
  const int nel = nvc * 2;  // elements in this chunk
  const uint32_t frow = (uint32_t)nvc * 16u, grow = 2 * frow;
  const unsigned char *fbase = reinterpret_cast<const unsigned char *>(fbuf) + hl * 8;
  unsigned char *gbase = reinterpret_cast<unsigned char *>(gbuf) + hl * 16;
  int off_g[NE];  // byte offset in the output row of element g
#pragma unroll
  for (int g = 0; g < NE; ++g) {
    const int e = hl + g * LPN;
    off_g[g] = (min(NV * (v0 + e / 2), nlev - NV) + EL * (e & 1)) * (int)sizeof(T);
  }
  auto rows_of = [](const i32x4 &r, uint32_t (&rw)[6]) {
    rw[0] = (uint32_t)r.y & 0xffffu; rw[1] = (uint32_t)r.y >> 16;
    rw[2] = (uint32_t)r.z & 0xffffu; rw[3] = (uint32_t)r.z >> 16;
    rw[4] = (uint32_t)r.w & 0xffffu; rw[5] = (uint32_t)r.w >> 16;
  };
  auto pair_of = [](const i32x4 &w, double &lo, double &hi) {
    const int a[2] = {w.x, w.y}, b[2] = {w.z, w.w};
    __builtin_memcpy(&lo, a, 8);
    __builtin_memcpy(&hi, b, 8);
  };
  // FULL: six incidences, none a pole edge (see k_sweepw)
  auto gradient = [&](const i32x4 *rec, const i32x4 &ref, int row, auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    if constexpr (!FULL) asm volatile("" ::: "memory");
    double al, be, cosg, pad;
    pair_of(rec[0], pad, al);
    pair_of(rec[1], be, cosg);
    uint32_t rw[6];
    rows_of(ref, rw);
    typename PG::St st[NE][EL];
    const unsigned char *self = fbase + __umul24((uint32_t)ref.x & 0xffffu, frow);
#pragma unroll
    for (int g = 0; g < NE; ++g) {
      const FElem x = *reinterpret_cast<const FElem *>(self + g * LPN * 8);
#pragma unroll
      for (int e = 0; e < EL; ++e) PG::init(st[g][e], x.v[e], 0.0);
    }
    FElem x[2][NE];
    double2 S2[2];
    auto read = [&](int j) {
      pair_of(rec[2 + j], S2[j & 1].x, S2[j & 1].y);
      const unsigned char *col = fbase + __umul24(rw[j], frow);
#pragma unroll
      for (int g = 0; g < NE; ++g)
        x[j & 1][g] = *reinterpret_cast<const FElem *>(col + g * LPN * 8);
    };
    read(0);
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (j < 5) read(j + 1);
      const double2 Sh = S2[j & 1];
      const bool pole = !FULL && j >= kMinRow && (ref.x & (kSgeoPole << j)) != 0;
      const bool use = FULL || j < kMinRow || j < ((ref.x >> 16) & 7);
#pragma unroll
      for (int g = 0; g < NE; ++g)
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          if (FULL || j < kMinRow) {
            PG::add_half(st[g][e], x[j & 1][g].v[e], Sh, false, 0.0);
          } else {
            typename PG::St tt = st[g][e];
            PG::add_half(tt, x[j & 1][g].v[e], Sh, pole, 0.0);
            PG::keep(st[g][e], tt, use);
          }
        }
      if constexpr (NE * EL >= 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < NE; ++g)
#pragma unroll
      for (int e = 0; e < EL; ++e) PG::settle(st[g][e]);
    unsigned char *dst = gbase + __umul24((uint32_t)row, grow);
#pragma unroll
    for (int g = 0; g < NE; ++g)
      if (hl + g * LPN < nel) {
        GElem o;
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          const typename PG::Out r = PG::result_half(st[g][e], al, be);
          o.v[e].x = r.x;
          if constexpr (F64) o.v[e].y = r.y * cosg;  // v cos(lat), as the divergence forms it
          else o.v[e].y = r.y;
        }
        *reinterpret_cast<GElem *>(dst + g * LPN * 16) = o;
      }
    if constexpr (!F64) {
      if (hl == 0) cosb[row] = cosg;
    }
  };
  auto divergence = [&](const i32x4 *rec, const i32x4 &ref, auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    if constexpr (!FULL) asm volatile("" ::: "memory");
    const i32x4 w0 = rec[0];
    double al, be, ci, pad;
    pair_of(w0, pad, al);
    pair_of(rec[1], be, ci);
    uint32_t rw[6];
    rows_of(ref, rw);
    typename PD::St st[NE][EL];
    const unsigned char *self = gbase + __umul24((uint32_t)ref.x & 0xffffu, grow);
#pragma unroll
    for (int g = 0; g < NE; ++g) {
      const GElem x = *reinterpret_cast<const GElem *>(self + g * LPN * 16);
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        if constexpr (F64) div_init_w(st[g][e], x.v[e]);
        else PD::init(st[g][e], x.v[e], ci);
      }
    }
    GElem x[2][NE];
    double2 S2[2];
    double cn2[2] = {0.0, 0.0};
    auto read = [&](int j) {
      pair_of(rec[2 + j], S2[j & 1].x, S2[j & 1].y);
      if constexpr (!F64) cn2[j & 1] = cosb[rw[j]];
      const unsigned char *col = gbase + __umul24(rw[j], grow);
#pragma unroll
      for (int g = 0; g < NE; ++g)
        x[j & 1][g] = *reinterpret_cast<const GElem *>(col + g * LPN * 16);
    };
    read(0);
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      if (j < 5) read(j + 1);
      const double2 Sh = S2[j & 1];
      const double cn = cn2[j & 1];
      const bool use = FULL || j < kMinRow ||
                       (j < ((ref.x >> 16) & 7) && (ref.x & (kSgeoPole << j)) == 0);
#pragma unroll
      for (int g = 0; g < NE; ++g)
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          typename PD::St tt = st[g][e];
          if constexpr (F64) div_add_half_w(tt, x[j & 1][g].v[e], Sh);
          else PD::add_half(tt, x[j & 1][g].v[e], Sh, false, cn);
          if (FULL || j < kMinRow) st[g][e] = tt;
          else PD::keep(st[g][e], tt, use);
        }
      if constexpr (NE * EL >= 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < NE; ++g)
#pragma unroll
      for (int e = 0; e < EL; ++e) PD::settle(st[g][e]);
    unsigned char *dst = reinterpret_cast<unsigned char *>(out) + (size_t)(uint32_t)w0.x * col_bytes;
#pragma unroll
    for (int g = 0; g < NE; ++g)
      if (hl + g * LPN < nel) {
        FElem o;
#pragma unroll
        for (int e = 0; e < EL; ++e) o.v[e] = PD::result_half(st[g][e], al, 0.0);
        __builtin_memcpy(dst + off_g[g], &o, sizeof(o));
      }
  };
  for (int q = qa; q <= qb + 2; ++q) {
    const int ng = glen(q);
    const int2 sp = own(q - 2);
    const int no = sp.y - sp.x;
    const int tg = (ng + NPN - 1) / NPN, td = (no + NPN - 1) / NPN;
    for (int t = cw; t < tg + td; t += ncw) {
      if (t < tg) {
        const int s = t * NPN + sub;
        if (s < ng) {
          const i32x4 ref = gref[(q % kLswRefSlots) * gmax + s];
          const i32x4 *rec = recs + ((q % kLswRecSlots) * gmax + s) * GW;
          const int row = (q % kLswGradSlots) * gmax + s;
          if (__builtin_amdgcn_ballot_w64((ref.x & kSgeoFull) == 0) == 0)
            gradient(rec, ref, row, std::true_type{});
          else
            gradient(rec, ref, row, std::false_type{});
        }
      } else {
        const int i = (t - tg) * NPN + sub, r = q - 2;
        if (i < no) {
          const i32x4 ref = oref[(q % kLswRefSlots) * pmax + i];
          // the own row's place in its run, in the record ring
          const int s = (ref.x & 0xffff) + ((r % kLswRecSlots) - (r % kLswGradSlots)) * gmax;
          const i32x4 *rec = recs + s * GW;
          if (__builtin_amdgcn_ballot_w64((ref.x & kSgeoFull) == 0) == 0)
            divergence(rec, ref, std::true_type{});
          else
            divergence(rec, ref, std::false_type{});
        }
      }
    }
    // this step's LDS accesses are done before the barrier
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// The instance for LPN lanes per position (8, 16 or 32) and NE elements per
// lane (1 .. kLswMaxNe).
template <class T, int LPN, int NE = 1>
void (*lsweepw_kernel_ne(int ne))(LaplView, const int4 *, const T *, T *, int, int, int) {
  if constexpr (NE < kLswMaxNe) {
    if (ne > NE) return lsweepw_kernel_ne<T, LPN, NE + 1>(ne);
  }
  return &k_lsweepw<T, LPN, NE>;
}
template <class T>
auto lsweepw_kernel(int lpn, int ne) {
  return lpn == 8    ? lsweepw_kernel_ne<T, 8>(ne)
         : lpn == 16 ? lsweepw_kernel_ne<T, 16>(ne)
                     : lsweepw_kernel_ne<T, 32>(ne);
}

// Packs the fused Laplacian's per-record geometry (after the scales are
// derived): gradient-node records in g-record order, own-position records
// in position order.
__global__ void k_pack_ggeo(DevMesh m, int ng, i32x4 *__restrict__ dst) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ng) return;
  const int4 gn = m.l2_gnode[g];  // {row start, row length, f self, position}
  i32x4 *o = dst + (size_t)g * kGGeoWords;
  for (int j = 0; j < 6; ++j) {  // halved normals (exact)
    const double2 h = make_double2(0.5 * m.S[gn.x + j].x, 0.5 * m.S[gn.x + j].y);
    __builtin_memcpy(&o[j], &h, 16);
  }
  __builtin_memcpy(&o[6], m.l2_glref + (size_t)g * kGRefs, 32);
  const PosRec pr = m.pos[gn.w];
  const double ab[2] = {pr.alpha, pr.beta};
  __builtin_memcpy(&o[8], ab, 16);
  const double c = m.coslat[pr.node];
  int cw[2];
  __builtin_memcpy(cw, &c, 8);
  o[9] = i32x4{gn.z, gn.y, cw[0], cw[1]};
}
__global__ void k_pack_lgeo(DevMesh m, i32x4 *__restrict__ dst) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m.V) return;
  const PosRec pr = m.pos[p];
  i32x4 *o = dst + (size_t)p * kLGeoWords;
  for (int j = 0; j < 6; ++j) {  // halved normals (exact)
    const double2 h = make_double2(0.5 * m.S[pr.r0 + j].x, 0.5 * m.S[pr.r0 + j].y);
    __builtin_memcpy(&o[j], &h, 16);
  }
  __builtin_memcpy(&o[6], m.l2_lref + pr.r0, 32);
  const double ac[2] = {pr.alpha, m.coslat[pr.node]};
  __builtin_memcpy(&o[8], ac, 16);
  o[9] = i32x4{pr.node, pr.r1 - pr.r0, m.l2_lself[p], 0};
  __builtin_memcpy(&o[10], m.ncos + pr.r0, 48);
}

// Packs the wave-specialised kernels' per-position records (after the scales
// are derived): `vec` 0 for scalar inputs, 1 for vector inputs; by position
// or by node.  Entries past a row are neutral: zero normals, cos(lat) 1.
__global__ void k_pack_sgeo(DevMesh m, int vec, int by_node, i32x4 *__restrict__ dst) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m.V) return;
  const PosRec pr = m.pos[p];
  const int n = pr.r1 - pr.r0;
  const double sc[3] = {pr.alpha, vec ? m.coslat[pr.node] : pr.beta, m.coslat[pr.node]};
  int w[6];
  __builtin_memcpy(w, sc, 24);
  i32x4 *o = dst + (size_t)(by_node ? pr.node : p) * (vec ? kSgeoWordsV : kSgeoWordsS);
  o[0] = i32x4{pr.node, 0, w[0], w[1]};
  o[1] = i32x4{w[2], w[3], w[4], w[5]};
  for (int j = 0; j < 6; ++j) {  // halved normals (exact)
    const double2 v = j < n ? make_double2(0.5 * m.S[pr.r0 + j].x, 0.5 * m.S[pr.r0 + j].y)
                            : make_double2(0.0, 0.0);
    __builtin_memcpy(&o[2 + j], &v, 16);
  }
  if (vec) {
    double cn[6];
    for (int j = 0; j < 6; ++j) cn[j] = j < n ? m.ncos[pr.r0 + j] : 1.0;
    __builtin_memcpy(&o[8], cn, 48);
  }
}

template <class T, int OP>
__global__ void __launch_bounds__(1024) k_flat(DevMesh m, const T *__restrict__ in,
                                               T *__restrict__ out, int nlev, int npb,
                                               int per_xcd) {
  int p0, p1;
  if (!tile_range(m, xcd_tile(blockIdx.x, per_xcd), npb, p0, p1)) return;
  const int nel = (p1 - p0) * nlev;
  for (int e = threadIdx.x; e < nel; e += blockDim.x) {
    const int pl = e / nlev;
    const int k = e - pl * nlev;
    const int p = p0 + pl;
    element<T, OP>(m, in, out, nlev, p, m.perm[p], m.rowp[p], m.rowp[p + 1], k);
  }
}

// ---------------------------------------------------------------------------
// Flux form, kernel 1 of 2: one value per (edge slot, level) into an
// EdgeColumns-like buffer [E + npole][nlev] (x2 for the gradient).  Slots
// E.. are the pole edges (gradient only).  FP64 fields only.
// ---------------------------------------------------------------------------
template <int OP>
__global__ void __launch_bounds__(256) k_edge_flux(DevMesh m, const double *__restrict__ in,
                                                   double *__restrict__ flux, int nlev) {
  const int nslot = (OP == OP_GRAD) ? m.E + m.npole : m.E;
  const size_t L = (size_t)nlev;
  const size_t total = (size_t)nslot * L;
  for (size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x; g < total;
       g += (size_t)gridDim.x * blockDim.x) {
    const int e = (int)(g / L);
    const int k = (int)(g - (size_t)e * L);
    const int a = m.e2n[2 * e], b = m.e2n[2 * e + 1];
    const double2 S = m.eS[e];
    if (OP == OP_GRAD) {
      const double xe = 0.5 * (in[(size_t)a * L + k] + in[(size_t)b * L + k]);
      double2 f;
      f.x = S.x * xe;
      f.y = S.y * xe;
      reinterpret_cast<double2 *>(flux)[g] = f;
    } else {
      const double2 *vin = reinterpret_cast<const double2 *>(in);
      const double2 ua = vin[(size_t)a * L + k], ub = vin[(size_t)b * L + k];
      const double ca = m.coslat[a], cb = m.coslat[b];
      const double aa = (OP == OP_DIV) ? ua.x : ua.y, ab = (OP == OP_DIV) ? ub.x : ub.y;
      const double ba = ((OP == OP_DIV) ? ua.y : ua.x) * ca;
      const double bb = ((OP == OP_DIV) ? ub.y : ub.x) * cb;
      const double ae = 0.5 * (aa + ab), be = 0.5 * (ba + bb);
      flux[g] = (OP == OP_DIV) ? S.x * ae + S.y * be : S.x * ae - S.y * be;
    }
  }
}

// Flux form, kernel 2 of 2: each node gathers its slots in the same order
// and with the same signs as the fused forms.
template <int OP>
__global__ void __launch_bounds__(1024) k_gather_flux(DevMesh m,
                                                      const double *__restrict__ flux,
                                                      double *__restrict__ out, int nlev,
                                                      int per_xcd) {
  int p0, p1;
  if (!tile_range(m, xcd_tile(blockIdx.x, per_xcd), 0, p0, p1)) return;
  const size_t L = (size_t)nlev;
  const int nel = (p1 - p0) * nlev;
  for (int e = threadIdx.x; e < nel; e += blockDim.x) {
    const int pl = e / nlev;
    const int k = e - pl * nlev;
    const int p = p0 + pl;
    const int node = m.perm[p], r0 = m.rowp[p], r1 = m.rowp[p + 1];
    if (OP == OP_GRAD) {
      double gl = 0.0, gt = 0.0;
      for (int r = r0; r < r1; ++r) {
        const uint32_t slot = (uint32_t)m.inc_edge[r];
        const bool pole = ((uint32_t)m.nbr[r] & kPoleBit) != 0;
        const double2 f = reinterpret_cast<const double2 *>(flux)[(size_t)(slot & ~kPoleBit) * L + k];
        const bool neg = (slot & kPoleBit) != 0;
        if (!pole) gl = gl + (neg ? -f.x : f.x);
        gt = gt + (neg ? -f.y : f.y);
      }
      double2 o;
      o.x = m.alpha[p] * gl;
      o.y = m.beta[p] * gt;
      reinterpret_cast<double2 *>(out)[(size_t)node * L + k] = o;
    } else {
      double acc = 0.0;
      for (int r = r0; r < r1; ++r) {
        if ((uint32_t)m.nbr[r] & kPoleBit) continue;
        const uint32_t slot = (uint32_t)m.inc_edge[r];
        const double f = flux[(size_t)(slot & ~kPoleBit) * L + k];
        acc = acc + ((slot & kPoleBit) ? -f : f);
      }
      out[(size_t)node * L + k] = m.alpha[p] * acc;
    }
  }
}

// ---------------------------------------------------------------------------
// Batched persistent form.  Workgroup b serves work queue b mod 8 (one per
// XCD); units are (item, block of positions, phase).  One launch runs one
// pass: phase 0 (every single operator, and the gradient of every
// Laplacian into its workspace), then, if any item is a Laplacian, a second
// launch runs phase 1 (the divergence of that gradient) -- the dependency is
// the launch order.  A workgroup never waits for another: it takes units
// from its queue until the queue is drained, then exits.  heads[x] is queue
// x's next unit.
// ---------------------------------------------------------------------------
// Lane vectors wider than 16 bytes: the batch kernel takes them one per
// lane only (two would not fit its register budget).
template <class T, int OP, int NV>
__host__ __device__ constexpr bool batch_wide() {
  return NV * sizeof(typename Pol<T, OP>::V) > 16;
}

// Column-form positions p0 + wave, p0 + wave + nw, ... below p1 with lane
// vectors of NV levels and nchv (1 or 2; 1 if wide) vectors per lane; false
// if that width does not exist for this dtype and operator.
template <class T, int OP, int NV>
__device__ __forceinline__ bool batch_colv(const DevMesh &m, const T *in, T *out, int nlev,
                                           int nchv, int p0, int p1, int wave, int nw, int lane) {
  if constexpr (lane_vec_ok<T, OP, NV>()) {
    for (int p = p0 + wave; p < p1; p += nw) {
      const PosRec pr = m.pos[p];
      if (batch_wide<T, OP, NV>() || nchv == 1) colv_node<T, OP, NV, 1>(m, in, out, nlev, pr, lane);
      else colv_node<T, OP, NV, 2>(m, in, out, nlev, pr, lane);
    }
    return true;
  }
  return false;
}

template <class T, int OP>
__device__ __forceinline__ void batch_unit_op(const DevMesh &m, int form, int level_vec,
                                              const T *in, T *out, int nlev, int p0, int p1) {
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (form == FORM_COLUMN) {
    // lane vectors as in the single-launch column form, up to two per lane
    // (one if wider than 16 bytes: the batch kernel's registers are sized
    // for that); wider columns and level_vec 1 take one level per lane
    const int nv = level_vec == 1 ? 0 : auto_level_vec<T, OP>(nlev, m.maxdeg, m.mindeg, level_vec);
    if (nv > 0) {
      const int nchv = ((nlev + nv - 1) / nv + 63) / 64;
      const bool wide = nv * (int)sizeof(typename Pol<T, OP>::V) > 16;
      bool done = false;
      if (nchv <= (wide ? 1 : 2)) {
        if (nv == 1) done = batch_colv<T, OP, 1>(m, in, out, nlev, nchv, p0, p1, wave, nw, lane);
        else if (nv == 2) done = batch_colv<T, OP, 2>(m, in, out, nlev, nchv, p0, p1, wave, nw, lane);
        else if (nv == 3) done = batch_colv<T, OP, 3>(m, in, out, nlev, nchv, p0, p1, wave, nw, lane);
        else done = batch_colv<T, OP, 4>(m, in, out, nlev, nchv, p0, p1, wave, nw, lane);
      }
      if (done) return;
    }
    const int nch = (nlev + 63) / 64;
    for (int p = p0 + wave; p < p1; p += nw) {
      const PosRec pr = m.pos[p];
      if (m.maxdeg <= 6 && nch == 1) column_node<T, OP, 1, 6, true>(m, in, out, nlev, pr, lane);
      else if (m.maxdeg <= 6 && nch == 2) column_node<T, OP, 2, 6, true>(m, in, out, nlev, pr, lane);
      else if (m.maxdeg <= 6 && nch == 3) column_node<T, OP, 3, 6, true>(m, in, out, nlev, pr, lane);
      else
        for (int k = lane; k < nlev; k += 64) element<T, OP>(m, in, out, nlev, p, pr.node, pr.r0, pr.r1, k);
    }
  } else {
    const int nel = (p1 - p0) * nlev;
    for (int e = threadIdx.x; e < nel; e += blockDim.x) {
      const int pl = e / nlev;
      const int k = e - pl * nlev;
      const int p = p0 + pl;
      element<T, OP>(m, in, out, nlev, p, m.perm[p], m.rowp[p], m.rowp[p + 1], k);
    }
  }
}

// waves per SIMD the batch kernel is compiled for (FP64: three, so the
// one-level-per-lane column paths keep their registers)
template <class T>
constexpr int batch_waves() { return sizeof(T) == 8 ? 3 : 4; }

template <class T>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(batch_waves<T>()))) k_batch(const BatchItem *__restrict__ items,
                                               const BatchUnit *__restrict__ units,
                                               const int *__restrict__ qbeg, int *heads) {
  // Unit indices pass through two LDS slots: while the workgroup runs unit
  // s_u[k], thread 0 already takes the next one into s_u[k ^ 1], so the
  // atomic's latency hides behind the unit and one barrier per unit
  // suffices (s_u[k] is rewritten only after every thread has passed the
  // barrier that follows its read).
  __shared__ int s_u[2];
  const int x = blockIdx.x & 7;
  const int qend = qbeg[x + 1];
  if (threadIdx.x == 0) s_u[0] = qbeg[x] + atomicAdd(&heads[x], 1);
  __syncthreads();
  for (int k = 0;; k ^= 1) {
    const int u = s_u[k];
    if (u >= qend) break;  // this queue is drained: every wave exits
    if (threadIdx.x == 0) s_u[k ^ 1] = qbeg[x] + atomicAdd(&heads[x], 1);
    const BatchUnit un = units[u];
    const BatchItem &it = items[un.item];
    const int op = it.lapl ? (un.phase ? OP_DIV : OP_GRAD) : it.op;
    const T *src = static_cast<const T *>(un.phase ? it.ws : it.in);
    T *dst = static_cast<T *>((it.lapl && un.phase == 0) ? it.ws : it.out);
    const int lv = un.phase ? it.level_vec1 : it.level_vec;
    if (op == OP_GRAD)
      batch_unit_op<T, OP_GRAD>(it.m, it.form, lv, src, dst, it.nlev, un.p0, un.p1);
    else if (op == OP_DIV)
      batch_unit_op<T, OP_DIV>(it.m, it.form, lv, src, dst, it.nlev, un.p0, un.p1);
    else
      batch_unit_op<T, OP_CURL>(it.m, it.form, lv, src, dst, it.nlev, un.p0, un.p1);
    __syncthreads();
  }
}

__global__ void k_fill(int *p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

atlas_status launch_fill(int *p, int n, int value, hipStream_t st) {
  hipLaunchKernelGGL(k_fill, dim3((n + 255) / 256), dim3(256), 0, st, p, n, value);
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

int batch_blocks_per_cu(atlas_dtype dt, int block) {
  int n = 0;
  hipError_t e = dt == ATLAS_F64
                     ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch<double>, block, 0)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch<float>, block, 0);
  return (e == hipSuccess && n > 0) ? n : 1;
}

// One batch = counter reset (a kernel, not a memset, so it can live in a
// captured graph) + the phase-0 pass + (if any) the phase-1 pass.
atlas_status launch_batch(atlas_dtype dt, const BatchItem *items, const BatchUnit *units,
                          const int *qbeg0, const int *qbeg1, bool two_pass, int *heads,
                          int grid, int block, hipStream_t st) {
  atlas_status s = launch_fill(heads, 16, 0, st);
  if (s != ATLAS_OK) return s;
  for (int pass = 0; pass < (two_pass ? 2 : 1); ++pass) {
    const int *qb = pass ? qbeg1 : qbeg0;
    int *hd = heads + 8 * pass;
    if (dt == ATLAS_F64)
      hipLaunchKernelGGL(k_batch<double>, dim3(grid), dim3(block), 0, st, items, units, qb, hd);
    else
      hipLaunchKernelGGL(k_batch<float>, dim3(grid), dim3(block), 0, st, items, units, qb, hd);
    ATLASX_HIP(hipGetLastError());
  }
  return ATLAS_OK;
}

// ---------------------------------------------------------------------------
// Streaming reference: read n, write 2n (the gradient's byte pattern).  One
// element per thread and a grid that covers the array (a grid-stride loop
// over fewer blocks reached only ~75 % of this rate on MI355X), each store
// instruction one contiguous run of 64 lane pairs.
// ---------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(256) k_stream_r1w2(const T *__restrict__ x, T *__restrict__ y,
                                                     int64_t n) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2 *yv = reinterpret_cast<v2 *>(y);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const T v = x[i];
    yv[i] = v2{v, v};
  }
}

atlas_status bandwidth_probe(const void *in, void *out, int64_t n, int elem, hipStream_t st) {
  // one thread per element up to 2^22 blocks (2^30 elements), then a loop
  const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, (int64_t)1 << 22);
  if (elem == 8)
    hipLaunchKernelGGL(k_stream_r1w2<double>, dim3(grid), dim3(256), 0, st,
                       static_cast<const double *>(in), static_cast<double *>(out), n);
  else
    hipLaunchKernelGGL(k_stream_r1w2<float>, dim3(grid), dim3(256), 0, st,
                       static_cast<const float *>(in), static_cast<float *>(out), n);
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

// ---------------------------------------------------------------------------
// Per-node scales, derived once at upload: alpha = R/V, beta = R cos/V.
// ---------------------------------------------------------------------------
__global__ void k_derive_scales(int V, const double *__restrict__ vol,
                                const double *__restrict__ cosl, double R,
                                double *__restrict__ alpha, double *__restrict__ beta,
                                PosRec *__restrict__ pos) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < V) {
    const double a = R / vol[p], b = (R * cosl[p]) / vol[p];
    alpha[p] = a;
    beta[p] = b;
    pos[p].alpha = a;
    pos[p].beta = b;
  }
}

atlas_status pack_lapl_geometry(MeshStore &m, int64_t ngrec) {
  void *g = nullptr, *l = nullptr;
  const size_t gb = std::max<size_t>(16, (size_t)ngrec * kGGeoWords * 16);
  const size_t lb = std::max<size_t>(16, (size_t)m.d.V * kLGeoWords * 16);
  if (hipMalloc(&g, gb) != hipSuccess) return fail(ATLAS_ENOMEM, "hipMalloc of mesh store failed");
  m.allocations.push_back(g);
  if (hipMalloc(&l, lb) != hipSuccess) return fail(ATLAS_ENOMEM, "hipMalloc of mesh store failed");
  m.allocations.push_back(l);
  m.bytes += gb + lb;
  if (ngrec > 0)
    hipLaunchKernelGGL(k_pack_ggeo, dim3((unsigned)((ngrec + 255) / 256)), dim3(256), 0, 0, m.d,
                       (int)ngrec, static_cast<i32x4 *>(g));
  if (m.d.V > 0)
    hipLaunchKernelGGL(k_pack_lgeo, dim3((m.d.V + 255) / 256), dim3(256), 0, 0, m.d,
                       static_cast<i32x4 *>(l));
  ATLASX_HIP(hipGetLastError());
  m.d.l2_ggeo = static_cast<const int4 *>(g);
  m.d.l2_lgeo = static_cast<const int4 *>(l);
  return ATLAS_OK;
}

atlas_status pack_sweep_geometry(MeshStore &m) {
  // by position for scalar and vector inputs, by node for the Laplacian
  const int sets = m.lcuts.empty() ? 2 : 3;
  auto words = [&](int k) { return (size_t)m.d.V * (k == 1 ? kSgeoWordsV : kSgeoWordsS); };
  size_t total = 0;
  for (int k = 0; k < sets; ++k) total += words(k) * 16;
  void *p = nullptr;
  if (hipMalloc(&p, total) != hipSuccess) {
    (void)hipGetLastError();
    return fail(ATLAS_ENOMEM, "hipMalloc of mesh store failed");
  }
  m.allocations.push_back(p);
  m.bytes += total;
  i32x4 *g = static_cast<i32x4 *>(p);
  for (int k = 0; k < sets; g += words(k), ++k) {
    hipLaunchKernelGGL(k_pack_sgeo, dim3((m.d.V + 255) / 256), dim3(256), 0, 0, m.d, k == 1,
                       k == 2 ? 1 : 0, g);
    ATLASX_HIP(hipGetLastError());
    (k == 0 ? m.d.sgeo : k == 1 ? m.d.sgeo_v : m.d.sgeo_n) = reinterpret_cast<const int4 *>(g);
  }
  return ATLAS_OK;
}

atlas_status derive_scales(MeshStore &m, const double *vol_by_pos, const double *cos_by_pos,
                           double radius) {
  const int V = m.d.V;
  hipLaunchKernelGGL(k_derive_scales, dim3((V + 255) / 256), dim3(256), 0, 0, V, vol_by_pos,
                     cos_by_pos, radius, const_cast<double *>(m.d.alpha),
                     const_cast<double *>(m.d.beta), const_cast<PosRec *>(m.d.pos));
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

// ---------------------------------------------------------------------------
// Host-side dispatch
// ---------------------------------------------------------------------------
size_t flux_ws_bytes(const MeshStore &m, atlas_op op, int nlev, atlas_dtype dt) {
  const size_t w = dt == ATLAS_F64 ? 8 : 4;
  const bool grad = op == ATLAS_OP_GRADIENT || op == ATLAS_OP_LAPLACIAN;
  const size_t slots = (size_t)m.d.E + (grad ? (size_t)m.d.npole : 0);
  return slots * (size_t)nlev * w * (grad ? 2 : 1);
}

// Built-in shape (the autotuner can replace it per mesh and class), from
// measurements: the wave-specialised sweep wherever its pieces fill the chip
// (sweepw_default).  Elsewhere, below 24 levels the flat form over blocks of
// 64 positions (512 threads; larger ones on large meshes), from 24 levels the
// column form over blocks of 16 consecutive positions (a run of one parallel,
// so the neighbour columns of consecutive blocks overlap in L2), at the
// automatic lane-vector width except the FP64 gradient to 47 levels and the
// FP32 one from there to 256 (one level per lane).  The Laplacian takes the
// fused form or each pass's own shape.
constexpr size_t kMaxLds = 160 * 1024;

// How the wave-specialised sweep runs a column: the cut of the tiles, the
// level chunks (nchunk even chunks of at most vpc 16-byte vectors), the
// lanes per position and elements per lane, and the LDS bytes.
struct SweepwPlan {
  int cut = 0, vpc = 0, nchunk = 0, lpn = 0, ne = 0, block = 0;
  size_t lds = 0;
};

// Chunk ends inside a row are what the sweep loses most by: the row's 128-byte
// lines there are written in halves by two workgroups (14.5 GB of rows cut in
// four: 3.2 TB/s, whole rows: 5.1 TB/s).  So the tiles are cut into the fewest
// parts with which a whole column fits in LDS, or that need the fewest
// chunks (O1280 FP64 gradient, 137 levels: four chunks on whole tiles 5.18
// ms, two chunks 4.77, whole columns on half tiles 4.57) -- but FP64 vector
// columns stay on whole tiles: most of their bytes are read, and narrow
// parts read more of them twice (O1280 divergence, 137 levels: three chunks
// on whole tiles 5.19 ms, whole columns on thirds 5.44).  Of a small mesh's
// cuts of the bands the one whose rounds of workgroups take the fewest
// steps (a last round that is nearly empty costs a whole one: O160, 37
// levels, FP32 divergence, 520 pieces on 512 places 33.8 us, 390 27.5, 260
// 35.6).
// `want`: at most so many vectors per chunk; epv: elements per vector.
static SweepwPlan sweepw_plan(const MeshStore &ms, bool vec, bool whole, int epv, int max_ne,
                              int nvec, int want) {
  const int most = 32 * max_ne / epv;
  const int cus = device_cu_count();
  SweepwPlan best;
  int64_t best_steps = 0;
  // tiles refused as too large: runs so long that even a one-vector chunk
  // leaves no room for the records of as many positions (above 224 nodes, 164 with
  // vector inputs; a regular grid's polar rows take half a parallel)
  const size_t seg = (size_t)max(1, ms.d.segmax);
  auto lines = [](size_t words) { return (words + 63) / 64 * 64; };
  if (16 * (kSweepwSlots * lines(seg) + kSweepwGeoSlots * lines(seg * (vec ? 14 : 10))) >
      kMaxLds) {
    best.lds = kMaxLds + 1;
    return best;
  }
  for (size_t k = 0; k < ms.cuts.size(); ++k) {
    const SweepView &v = ms.cuts[k];
    if (whole && v.parts > 1) continue;
    auto bytes = [&](int c) {
      return (size_t)16 * (kSweepwSlots * max(1, v.segmax) * c +
                           kSweepwGeoSlots * max(1, v.pmax) *
                               (1 + (vec ? kSgeoWordsV : kSgeoWordsS))) +
             kSweepwLdsTail;
    };
    SweepwPlan p;
    p.cut = (int)k;
    p.vpc = min(want > 0 ? min(want, most) : most, nvec);
    p.nchunk = (nvec + p.vpc - 1) / p.vpc;
    p.vpc = (nvec + p.nchunk - 1) / p.nchunk;
    while (p.vpc > 1 && bytes(p.vpc) > kMaxLds) {
      ++p.nchunk;
      p.vpc = (nvec + p.nchunk - 1) / p.nchunk;
    }
    p.nchunk = (nvec + p.vpc - 1) / p.vpc;
    p.lds = bytes(p.vpc);
    if (k > 0 && (p.nchunk > best.nchunk ||
                  (p.nchunk == best.nchunk && v.parts > ms.cuts[best.cut].parts)))
      continue;
    // lanes per position and elements per lane: the cheapest pair that
    // holds the chunk, a wavefront's cost being its elements and a fixed part
    // (the record's decoding, about three elements' worth) over its positions
    const int nel = p.vpc * epv;
    int cost = INT_MAX;
    for (int l : {8, 16, 32}) {
      const int e = (nel + l - 1) / l;
      if (e <= max_ne && (e + 3) * l < cost) {
        cost = (e + 3) * l;
        p.lpn = l;
        p.ne = e;
      }
    }
    // the producers, and consumers for one position per lane group a step
    // (where two workgroups share a compute unit, for one position less: few
    // runs have pmax)
    const int npn = 64 / p.lpn;
    const int own = max(1, 2 * p.lds <= kMaxLds ? v.pmax - 1 : v.pmax);
    const int waves = min(16, kSweepwGroups * kSweepwGroupWaves + (own + npn - 1) / npn);
    p.block = 64 * waves;
    // steps until the last round of workgroups is done (four for each
    // one's start); waves a compute unit holds by the kernels' registers
    const int held = p.ne <= 2 ? 32 : p.ne == 3 ? 24 : p.ne == 4 ? 20 : 16;
    const int64_t places =
        (int64_t)cus * max(1, min((int)(kMaxLds / p.lds), held / max(8, waves)));
    const int64_t units = (int64_t)v.ntiles * p.nchunk;
    const int64_t steps = (units + places - 1) / places * (v.rings + 4);
    if (k == 0 || p.nchunk < best.nchunk || v.parts < ms.cuts[best.cut].parts ||
        steps < best_steps) {
      best = p;
      best_steps = steps;
    }
  }
  return best;
}
template <class T, int OP, bool DC>
static SweepwPlan sweepw_plan(const MeshStore &m, int nlev, int level_chunk) {
  constexpr int nv16 = 16 / (int)sizeof(typename Pol<T, OP>::V);
  return sweepw_plan(m, Pol<T, OP>::kVecIn, Pol<T, OP>::kVecIn && sizeof(T) == 8,
                     nv16 / sweepw_elem_levels<T, DC>(), sweepw_max_ne<T, OP, DC>(),
                     (nlev + nv16 - 1) / nv16, (level_chunk + nv16 - 1) / nv16);
}

// Where the wave-specialised sweep is the built-in shape: on large meshes, and
// wherever its pieces fill the chip.  Columns that leave room for two
// workgroups per compute unit ask for 64 tiles (in up to six bands each;
// O160 has 130: 37 levels, FP32 divergence 27.5 against 35.6 us for the column
// form; O80 has 39: 16 against 11 us), longer ones and those above 48 levels
// (O160, 91 levels, FP32 gradient: 43 against 34 us) for 600 pieces and chunks
// of whole bands (O320 has 460 tiles: 920 pieces, 137 levels, FP64 gradient
// 335 against 466 us; O200 has 194, 582 pieces: FP64 divergence 195 against
// 190 us).
//
// Short columns leave it bound by what a piece costs whatever its levels: the
// records of its nodes, 144 bytes each, which the flat form's blocks read
// less of and share in the caches, and each tile's walk (O320 cut in 3360
// tiles of 125 nodes, 4 levels: 45 us against 32 for the flat form).  `pair`: for
// two results (the one-pass divergence and curl, which the flat form takes twice
// as long for: O500, 2 levels, 71 against 155 us), from its first vector on.
// For one: from a few levels and a number of values that grows with the tiles
// (inputs that are not in the caches; FP64 gradient: O320 4 levels 31 against
// 30 us, O400 39 against 45; O500 3 levels 61 against 57, but the Laplacian's two
// passes 129 against 144; 3360 tiles, 8 levels 49
// against 50, 10: 55 against 64; divergence: O320 4 levels 29 against 34; 3360
// tiles, 5 levels 44 against 42, 7: 45 against 54; FP32 gradient: O160 14 levels
// 16 against 18, O256 6 levels 24 against 22, 7: 24 against 26; 3360 tiles, 8
// levels 49 against 42, 10: 49 against 54; divergence: 3360 tiles, 6 levels 46
// against 44, 7: 46 against 52).  On meshes above 1.5 M nodes, whose geometry the
// caches no longer hold, from a little less (O640, FP32 divergence 2 levels 90
// against 80 us, FP64 gradient 3 levels 89 against 98; O900 2 levels 155 against
// 171), and vector columns in FP64 at once (O1280, one level, 304 against 377 us).
//
// Tiles of fewer than 96 nodes read more records than columns: they are left
// to the other forms (O160 in tiles of 61 nodes, FP32, 60 levels: divergence 49
// against 39 us, gradient 52 against 36; FP64: divergence 57 against 53), except
// where those read the columns in several passes or parts (sweepw_least_nodes).
static int sweepw_least_nodes(bool pair, bool grad, bool f32, int nlev) {
  if (pair) {
    // no one-pass column form from 16 to 47 levels (tiles of 32, O320: FP64, 37
    // levels, 257 against 354 us), nor a flat one (tiles of 61, O160: 14 levels
    // 47 against 53); FP64 above 256: columns in parts (323 against 692)
    if ((nlev >= 16 && nlev < 48) || (!f32 && nlev > 256)) return 30;
    return nlev >= 5 && nlev < 16 ? 48 : 96;
  }
  if (!grad) {
    // FP64 above 256 levels: parts again (tiles of 61: 217 against 348); FP32 from 13
    // to 16, which the flat form takes in two passes (O640 in tiles of 63: 283
    // against 411, 20: 581 against 516)
    if (!f32 && nlev > 256) return 30;
    return f32 && nlev > 12 && nlev <= 16 ? 48 : 96;
  }
  // gradients: FP64 from 20 levels (O640 in tiles of 63: 20 levels 396 against 495
  // us, 37: 674 against 688, 60: 674 against 924; of 32 nodes, O320: 91 levels 252
  // against 290, 137: 471 against 444), FP32 from 161 to 240 (tiles of 61: 170
  // levels 61 against 73, 137: 73 against 61)
  if (f32) return nlev > 160 && nlev <= 240 ? 48 : 96;
  if (nlev >= 42) return nlev <= 112 ? 30 : 48;
  return nlev >= 20 && nlev <= 24 ? 48 : 96;
}
static bool sweepw_default(const MeshStore &ms, atlas_op op, atlas_dtype dt, int nlev, bool pair,
                           LaunchShape *s) {
  const DevMesh &m = ms.d;
  const bool grad = op == ATLAS_OP_GRADIENT;
  if (!grad && op != ATLAS_OP_DIVERGENCE && op != ATLAS_OP_CURL) return false;
  const int nv = dt == ATLAS_F64 ? (grad ? 2 : 1) : (grad ? 4 : 2);  // levels per vector
  if (nlev < nv || m.ntiles < kSweepFewTiles) return false;
  const bool large = m.ntiles >= kSweepMinTiles;
  const bool f32 = dt == ATLAS_F32;
  const int64_t values = (int64_t)m.V * nlev, tiles = m.ntiles;
  if (m.V < sweepw_least_nodes(pair, grad, f32, nlev) * tiles) return false;
  // (FP32 vector columns of several chunks on tiles of fewer than 192 nodes,
  // where the column form's two or four levels per lane hold the whole column:
  // O320 in tiles of 125, 104 levels, 209 against 180 us, 137: 259 against 272,
  // 200: 398 against 346; one pass: 104 levels 366 against 238, 200: 640 against
  // 423)
  if (f32 && !grad && m.V < 192 * tiles &&
      (pair ? nlev > 96 : (nlev > 96 && nlev <= 128) || (nlev > 192 && nlev <= 256)))
    return false;
  if (pair) {
    if (!large && values < 1500000) return false;
  } else if (m.V >= 1500000) {
    if (values < (f32 || grad ? 3000000 : 0) + 600 * tiles) return false;
  } else if (grad ? nlev < (f32 ? 5 : m.V >= 750000 ? 3 : 4) || values < (f32 ? 1400000 + 800 * tiles
                                                          : 1300000 + 700 * tiles)
                  : nlev < (f32 ? 5 : 3) || values < (f32 ? 1300000 + 470 * tiles
                                                          : 1150000 + 400 * tiles)) {
    return false;
  }
  const SweepwPlan p = dt == ATLAS_F64 ? (grad ? sweepw_plan<double, OP_GRAD, false>(ms, nlev, 0)
                                               : sweepw_plan<double, OP_DIV, false>(ms, nlev, 0))
                                       : (grad ? sweepw_plan<float, OP_GRAD, false>(ms, nlev, 0)
                                               : sweepw_plan<float, OP_DIV, false>(ms, nlev, 0));
  if (p.lds > kMaxLds) return false;
  // (several chunks make several pieces of a part, but FP32 columns have the
  // column form's lane vectors beside them, which hold up to 256 levels: there on
  // 250000 nodes and more, or above that, and where the last round of pieces is not
  // too empty: O256 200 levels 202 against 227 us, O220 184 against 170, 280 levels
  // 241 against 262; O200's 776 pieces are a little more than three rounds: 178
  // against 154, 280 levels 224 against 217)
  const int64_t parts = (int64_t)m.ntiles * ms.cuts[p.cut].parts;
  const int64_t pieces = parts * p.nchunk, cus = device_cu_count();
  const bool chunks = !f32 || ((m.V >= 250000 || nlev >= 256) &&
                               9 * pieces >= 7 * cus * ((pieces + cus - 1) / cus));
  if (!large && (nlev > 48 || 2 * p.lds > kMaxLds) && (chunks ? pieces : parts) < 600)
    return false;
  s->variant = ATLAS_VARIANT_SWEEP;
  s->block = max(512, p.block);
  s->nodes_per_block = 0;
  s->level_chunk = 0;
  s->blocks_per_cu = 0;
  s->level_vec = 0;
  return true;
}

// The wave-specialised sweep needs the packed records, rows of 4..6, and runs
// about as long as a tile's own rows: a regular grid's polar rows refer to the
// far half of their parallel, and rings of such runs leave no room for columns
// (F640, 20 levels: FP64 gradient 2.95 against 1.06 ms for the flat form,
// divergence 6.3 against 1.12).
static bool sweepw_builtin(const MeshStore &m, atlas_op op, atlas_dtype dt, int nlev, bool pair,
                           LaunchShape *s) {
  return m.d.sgeo && !m.cuts.empty() && m.d.mindeg >= kMinRow &&
         max(1, m.d.segmax) * kGeoWords <= 768 && sweepw_default(m, op, dt, nlev, pair, s);
}

struct FusedwPlan {
  int cut = 0, vpc = 0, nchunk = 0, lpn = 0, ne = 0, block = 0;
  size_t lds = 0;
};
template <class T>
static bool fusedw_plan(const MeshStore &ms, int nlev, const LaunchShape &sh, FusedwPlan *fp);

// `packed`: the mesh's packed records may be used (they hold the physical
// scales).
LaunchShape default_shape(const MeshStore &m, atlas_op op, int nlev, atlas_dtype dt,
                          bool packed) {
  LaunchShape s;
  s.variant = nlev >= 24 ? ATLAS_VARIANT_COLUMN : ATLAS_VARIANT_FLAT;
  s.block = nlev >= 24 ? 256 : 512;
  s.nodes_per_block = nlev >= 24 ? 16 : 64;
  s.level_vec = 0;
  if (nlev < 24 && m.d.ntiles >= kSweepMinTiles) {
    // large meshes have blocks enough: more positions in each fetch fewer
    // neighbours from other blocks (O1280, FP32 gradient, 3 levels: 426 us at
    // 64 positions on 512 threads, 372 at 256 on 1024; one level, FP64: 333,
    // 321 at 128, 341 at 256; F640, FP64 gradient, 2 levels 190 and 170), but
    // from 5 levels no more than one value per thread: 256 positions of 5 leave
    // three quarters of the second pass idle (O500, FP32 gradient: 73.1 us, 69.7
    // at 64 on 512 threads, 64.6 at 204; F640 288, 279, 236; 9 levels 450, 447,
    // 394; FP64, 20 levels 992, 1060, 958).  (Smaller meshes in smaller tiles:
    // O320 one level 21.3 us, 23.8 at 128, 22.0 at 256.)
    s.block = 1024;
    s.nodes_per_block = nlev == 1 && m.d.V >= 750000 ? 128 : min(256, 1024 / nlev);
  }
  // (the register-staged sweep; on tiles of 250 nodes O640, 60 levels, FP64
  // gradient 1177 against 765 us for the column form)
  const bool sweep_fits = m.d.sweep_ok && m.d.ntiles >= kSweepMinTiles &&
                          m.d.V >= 512 * (int64_t)m.d.ntiles &&
                          max(1, m.d.segmax) * kGeoWords <= 768;
  auto staged = [](LaunchShape v) {
    v.variant = ATLAS_VARIANT_SWEEP;
    v.block = 768;
    v.nodes_per_block = 0;
    v.blocks_per_cu = 1;
    v.level_vec = 0;
    return v;
  };
  if (op == ATLAS_OP_LAPLACIAN) {
    // the fused one-pass form, wave-specialised, where it beats the two
    // passes on their own shapes: on large meshes from 4 levels in FP64
    // (O1280, 10 levels: 1.03 against 1.09 ms, 137: 7.2 against 9.4) and from
    // 33 in FP32 (24 levels: 1.46 against 1.22 ms, 40: 1.78 against 1.75,
    // 63: 2.19 against 3.15, 137: 4.85 against 5.65; it needs no workspace);
    // on small ones with work enough to hide its longer walk and pieces enough
    // to fill the chip (FP64: O320, 37 levels, 149 against 292 us; O120, 62000
    // nodes: 80 levels 86 against 85, 96: 86 against 97, 137: 114 against 144;
    // O160 60 levels 102 against 110, 128 161 against 206; O180 37 levels, 5 M
    // values, 89 against 77, 47: 88 against 118; FP32: O320, 64 levels 158 against
    // 274, 40: 131 against 127; O220 112 levels, 23 M values, 165 against 175, 137:
    // 187 against 244; O160 240 levels, 26 M, 205 against 199, 300 235 against
    // 271)
    const bool f64 = dt == ATLAS_F64;
    const int64_t values = (int64_t)m.d.V * nlev;
    const bool worth =
        m.d.ntiles >= kSweepMinTiles ? nlev >= (f64 ? 4 : 33)
        : f64 ? values >= 5000000 : values >= 25000000 && nlev >= 64;
    // (Also where tiles are so small that most gradients are formed several times:
    // O320 in tiles of 16 nodes, FP64, 37 levels 519 against 337 us.  The two
    // passes need the gradient's memory, which callers of such meshes do without.)
    FusedwPlan fw;
    LaunchShape fs;
    fs.variant = ATLAS_VARIANT_FUSED;
    fs.block = kLswBlock;
    if (worth && m.d.ntiles >= kSweepFewTiles &&
        (f64 ? fusedw_plan<double>(m, nlev, fs, &fw) : fusedw_plan<float>(m, nlev, fs, &fw))) {
      fs.block = max(512, fw.block);
      return fs;
    }
    s.per_pass = 1;
    return s;
  }
  if (packed && sweepw_builtin(m, op, dt, nlev, false, &s)) return s;
  // Without the packed records the sweep is the register-staged one: one
  // workgroup per tile and level chunk, each walking its band's parallels in
  // turn, so only a mesh of many tiles fills the chip (O160, 37 levels, FP64
  // gradient: 100 us on 130 tiles, 30 for the column form), and only columns
  // long enough to hide each step's loads repay the walk.  FP32 gradient:
  // 20 to 79 levels (O1280: 16 levels 1560 against 1370 us for the flat form,
  // 20: 1589 against 1785, 37: 1590 against 2177 for the column form, 64: 1834
  // against 2380, 80: 2706 against 2683); FP64 gradient from 48 (below).
  if (dt == ATLAS_F32 && op == ATLAS_OP_GRADIENT && sweep_fits && nlev >= 20 && nlev < 80)
    return staged(s);
  // The derivatives in longitude and latitude also take it for longer columns,
  // from levels that grow as the tiles get fewer -- but not from 241 to 256
  // levels, whose last chunk is short (FP32, O640, 240 levels 1011 against 1273
  // us, 256: 1868 against 1354; FP64, O320, 879 against 681).  FP32: from 161
  // levels, up to 256 of which the column form holds in one level per lane
  // (O500, 160 levels 612 against 553, 185: 622 against 666; O640 892 against
  // 1090; O320 170 levels 246 against 257, 280: 481 against 515; O256 240 levels
  // 272 against 227); on more than 1.5 M nodes from 100 (O640, 120 levels 772
  // against 799; O900 91 levels 1450 against 1337), 4 M from 80 (O1280, 120 levels
  // 2887 against 3136).  On tiles of fewer than 512 nodes later (O320 in tiles of
  // 367: FP32, 185 levels 278 against 275, 240: 312 against 336; FP64, 80 levels
  // 257 against 252, 120: 298 against 344).  FP64: O400, 60 levels 332 against
  // 350; O320, 97 levels 265 against 295, 120: 280 against 357; O256, 160 levels
  // 329 against 319, 200: 353 against 378; O220, 210 levels 255 against 294.
  const bool f32 = dt == ATLAS_F32;
  if (!packed && op == ATLAS_OP_GRADIENT && m.d.sweep_ok &&
      max(1, m.d.segmax) * kGeoWords <= 768 && (nlev <= 240 || nlev > 256) &&
      m.d.V >= (nlev > (f32 ? 200 : 90) ? 320 : 512) * (int64_t)m.d.ntiles) {
    const int t = m.d.ntiles;
    if (f32 ? t >= 400 && nlev >= (m.d.V >= 4000000 ? 80 : m.d.V >= 1500000 ? 100 : 161)
            : t >= 220 && nlev >= (t >= kSweepMinTiles ? 48 : t >= 650 ? 60
                                   : t >= 400 ? 100 : 180))
      return staged(s);
  }
  if (nlev < 24) return s;
  if (nlev < 48) {
    if (dt == ATLAS_F64 && op == ATLAS_OP_GRADIENT) {
      // one level per lane (O100, 30 levels, 14.4 against 15.7 us); FP32 takes
      // lane vectors (F300, 37 levels, gradient 155 against 172 us; F640, 47
      // levels, divergence 1197 against 1286)
      s.level_vec = 1;
    }
    return s;
  }
  // FP32 gradient: one level per lane to 256 levels (F640, 137 levels, 1566
  // against 1652 us on lane vectors, 256: 2692 against 2945); above, that form
  // walks the column in single steps (300: 7765 against 4222)
  if (dt == ATLAS_F32 && op == ATLAS_OP_GRADIENT && nlev <= 256) s.level_vec = 1;
  if (dt == ATLAS_F64 && op == ATLAS_OP_GRADIENT && sweep_fits) {
    // (O1280: 64 levels 2953 against 3205 us for the column form, 137: 5891
    // against 7185)
    return staged(s);
  }
  return s;
}


int device_cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Levels per chunk of the sweep form: at most 64 (one per lane), split
// evenly (137 -> 46, 46, 45).
static int sweep_chunk(int nlev, int want) {
  if (want > 0) return min(want, 64);
  const int n = (nlev + 63) / 64;
  return (nlev + n - 1) / n;
}

// Whether a sweep shape runs the wave-specialised kernel: blocks_per_cu 0,
// the packed geometry, 16-byte lane vectors, rows of 4..6 incidences and a
// block of at least 512 threads.
template <class T, int OP>
static bool sweepw_applies(const DevMesh &m, int nlev, const LaunchShape &sh) {
  constexpr int nv16 = 16 / (int)sizeof(typename Pol<T, OP>::V);
  return sh.blocks_per_cu == 0 && m.sgeo && (sh.level_vec == 0 || sh.level_vec == nv16) &&
         nlev >= nv16 && m.maxdeg <= 6 && m.mindeg >= kMinRow && sh.block >= 512 &&
         sh.block % 64 == 0;
}

// The wave-specialised sweep of `sh` (sweepw_applies); DC: the divergence
// and, into out2, the curl of the same field in one pass.
template <class T, int OP, bool DC>
static atlas_status launch_sweepw(const MeshStore &ms, const T *in, T *out, T *out2, int nlev,
                                  const LaunchShape &sh, hipStream_t st) {
  const DevMesh &m = ms.d;
  const SweepwPlan p = sweepw_plan<T, OP, DC>(ms, nlev, sh.level_chunk);
  if (p.lds > kMaxLds) return fail(ATLAS_EINVAL, "sweep tile too large for LDS");
  const SweepView &v = ms.cuts[p.cut];
  const int64_t units = (int64_t)v.ntiles * p.nchunk;
  const int per = (int)((units + 7) / 8);
  auto kern = sweepw_kernel<T, OP, DC>(p.lpn, p.ne);
  ATLASX_HIP(hipFuncSetAttribute((const void *)kern,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds));
  hipLaunchKernelGGL(kern, dim3(per * 8), dim3(sh.block), p.lds, st, v,
                     Pol<T, OP>::kVecIn ? m.sgeo_v : m.sgeo, in, out, out2, nlev, p.vpc, per);
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

template <class T, int OP>
static atlas_status launch_typed(const MeshStore &ms, const T *in, int nlev, T *out, void *ws,
                                 const LaunchShape &sh, hipStream_t st,
                                 const DevMesh *dm = nullptr) {
  const DevMesh &m = dm ? *dm : ms.d;
  const int ntiles = sh.nodes_per_block > 0 ? (m.V + sh.nodes_per_block - 1) / sh.nodes_per_block
                                            : m.ntiles;
  const int per_xcd = (ntiles + 7) / 8;
  const dim3 grid(per_xcd * 8), block(sh.block);
  if (sh.nodes_per_block > 0 && (int64_t)sh.nodes_per_block * nlev * 2 >= ((int64_t)1 << 31))
    return fail(ATLAS_EINVAL, "nodes_per_block * nlev too large");
  switch (sh.variant) {
    case ATLAS_VARIANT_COLUMN: {
      if (sh.block > 512 && sh.level_chunk == 0)
        return fail(ATLAS_EINVAL, "the column form takes at most 512 threads per block");
      if (sh.level_chunk > 0) {
        const int nchunk = (nlev + sh.level_chunk - 1) / sh.level_chunk;
        if ((int64_t)ntiles * nchunk * sh.block >= ((int64_t)1 << 32))
          return fail(ATLAS_EINVAL, "too many work units: raise nodes_per_block or level_chunk");
        const int units = ntiles * nchunk;
        const int per = (units + 7) / 8;
        hipLaunchKernelGGL((k_column_chunked<T, OP>), dim3(per * 8), block, 0, st, m, in, out,
                           nlev, sh.nodes_per_block, sh.level_chunk, ntiles, per);
        break;
      }
      const int nch = (nlev + 63) / 64;
      // persistent grid: blocks_per_cu workgroups on every compute unit
      const int cyc = sh.blocks_per_cu > 0 ? sh.blocks_per_cu * device_cu_count() / 8 : 0;
      const dim3 cgrid = cyc > 0 ? dim3(8 * cyc) : grid;
      // level_vec: 0 = widest lane vector, 2 / 4 = at most that many levels
      // per lane, 1 = the one-level-per-lane kernel
      if (sh.level_vec < 0 || sh.level_vec > 4)
        return fail(ATLAS_EINVAL, "level_vec must be in [0, 4]");
      const int nv = sh.level_vec == 1 ? 0
                                       : auto_level_vec<T, OP>(nlev, m.maxdeg, m.mindeg,
                                                               sh.level_vec);
      if (nv > 0) {
        const int nchv = (nlev + 64 * nv - 1) / (64 * nv);
        void (*kern)(DevMesh, const T *, T *, int, int, int, int) = nullptr;
#define ATLASX_COLV(NV)                                                     \
  if constexpr (lane_vec_ok<T, OP, NV>()) {                                 \
    if (nchv == 1) kern = k_colv<T, OP, NV, 1>;                             \
    else if (nchv == 2) kern = k_colv<T, OP, NV, 2>;                        \
    else if (nchv == 3) kern = k_colv<T, OP, NV, 3>;                        \
    else kern = k_colv<T, OP, NV, 4>;                                       \
  }
        if (nv == 1) {
          ATLASX_COLV(1)
        } else if (nv == 2) {
          ATLASX_COLV(2)
        } else if (nv == 3) {
          ATLASX_COLV(3)
        } else {
          ATLASX_COLV(4)
        }
#undef ATLASX_COLV
        if (!kern) return fail(ATLAS_EINVAL, "level_vec not available for this dtype and operator");
        hipLaunchKernelGGL(kern, cgrid, block, 0, st, m, in, out, nlev, sh.nodes_per_block,
                           per_xcd, cyc);
        break;
      }
#define ATLASX_COL(N)                                                                  \
  do {                                                                                 \
    if (m.maxdeg <= 6)                                                                 \
      hipLaunchKernelGGL((k_column<T, OP, N, 6>), cgrid, block, 0, st, m, in, out, nlev, \
                         sh.nodes_per_block, per_xcd, cyc);                            \
    else                                                                               \
      hipLaunchKernelGGL((k_column<T, OP, N, 8>), cgrid, block, 0, st, m, in, out, nlev, \
                         sh.nodes_per_block, per_xcd, cyc);                            \
  } while (0)
      if (nch == 1) ATLASX_COL(1);
      else if (nch == 2) ATLASX_COL(2);
      else if (nch == 3) ATLASX_COL(3);
      else if (nch == 4) ATLASX_COL(4);
      else ATLASX_COL(0);
#undef ATLASX_COL
      break;
    }
    case ATLAS_VARIANT_FLAT:
      hipLaunchKernelGGL((k_flat<T, OP>), grid, block, 0, st, m, in, out, nlev,
                         sh.nodes_per_block, per_xcd);
      break;
    case ATLAS_VARIANT_FLUX: {
      if constexpr (sizeof(T) == 4) {
        // the terms of an FP32 field's sums are FP64: the column form
        // computes them (the workspace stays as it is)
        LaunchShape col;
        col.nodes_per_block = 16;
        return launch_typed<T, OP>(ms, in, nlev, out, ws, col, st, dm);
      } else {
        T *flux = static_cast<T *>(ws);
        const size_t nslot = (size_t)m.E + (OP == OP_GRAD ? m.npole : 0);
        const size_t total = nslot * (size_t)nlev;
        const unsigned nb = (unsigned)std::min<size_t>((total + 255) / 256, 256 * 1024);
        hipLaunchKernelGGL((k_edge_flux<OP>), dim3(nb), dim3(256), 0, st, m, in, flux, nlev);
        const int per = (m.ntiles + 7) / 8;
        hipLaunchKernelGGL((k_gather_flux<OP>), dim3(per * 8), block, 0, st, m, (const T *)flux,
                           out, nlev, per);
        break;
      }
    }
    case ATLAS_VARIANT_SWEEP: {
      if (!m.sweep_ok) return fail(ATLAS_EINVAL, "the sweep form needs a mesh of parallels");
      if (sh.nodes_per_block > 0)
        return fail(ATLAS_EINVAL, "the sweep form runs on the mesh's tiles (nodes_per_block = 0)");
      // the chunk shrinks until a parallel's run fits the staging registers
      // (16 elements per thread) and four runs fit in LDS
      if (sh.level_vec < 0 || sh.level_vec > 4)
        return fail(ATLAS_EINVAL, "level_vec must be in [0, 4]");
      // the level-vector sweep stages each position's geometry with one
      // thread per 16-byte word: it needs a block of segmax * kGeoWords
      // threads, else the one-level-per-lane sweep runs (same results)
      // wave-specialised sweep (blocks_per_cu == 0): 16-byte lane vectors
      if (sweepw_applies<T, OP>(m, nlev, sh)) {
        atlas_status s = launch_sweepw<T, OP, false>(ms, in, out, nullptr, nlev, sh, st);
        if (s != ATLAS_OK) return s;
        break;
      }
      int nv = sh.level_vec == 1 ? 0
                                 : auto_level_vec<T, OP>(nlev, m.maxdeg, m.mindeg, sh.level_vec);
      if (sh.block < max(1, m.segmax) * kGeoWords) nv = 0;
      if (nv > 0) {
        // level chunk: vpc lane vectors per workgroup pass, at most 64, split
        // evenly; it shrinks until four runs fit the LDS budget (two
        // workgroups per compute unit) and a run fits the staging registers
        const int nvec = (nlev + nv - 1) / nv;
        int vpc = sh.level_chunk > 0 ? min(64, (sh.level_chunk + nv - 1) / nv) : 64;
        vpc = min(vpc, nvec);
        {
          const int nchunk = (nvec + vpc - 1) / vpc;
          vpc = (nvec + nchunk - 1) / nchunk;
        }
        const size_t seg = (size_t)max(1, m.segmax);
        const size_t rb = (size_t)nv * sizeof(typename Pol<T, OP>::V);  // lane-vector bytes
        // geometry staged per run: 2 record words and up to kGeoWords row
        // words per position, one of each kind per thread
        const size_t geo = 4 * seg * (2 + kGeoWords) * 16;
        const size_t budget = sh.block > 512 ? kMaxLds : kMaxLds / 2;
        // (staging: at most kSweepEpt lane vectors per thread and run)
        while (vpc > 1 && (4 * seg * vpc * rb + geo > budget ||
                           (int)((seg * vpc + sh.block - 1) / sh.block) > kSweepEpt))
          vpc = (vpc + 1) / 2;
        const int ept = (int)((seg * vpc + sh.block - 1) / sh.block);
        if (4 * seg * vpc * rb + geo > kMaxLds || ept > kSweepEpt)
          return fail(ATLAS_EINVAL, "sweep tile too large for LDS or the block size");
        const int nchunk = (nvec + vpc - 1) / vpc;
        const size_t lds = 4 * seg * vpc * rb + geo;
        const int units = m.ntiles * nchunk;
        const int per = (units + 7) / 8;
        void (*kern)(DevMesh, const T *, T *, int, int, int, int) = nullptr;
#define ATLASX_SWV(NV)                                              \
  if constexpr (lane_vec_ok<T, OP, NV>()) kern = k_sweepv<T, OP, NV, kSweepEpt>;
        if (nv == 1) {
          ATLASX_SWV(1)
        } else if (nv == 2) {
          ATLASX_SWV(2)
        } else if (nv == 3) {
          ATLASX_SWV(3)
        } else {
          ATLASX_SWV(4)
        }
#undef ATLASX_SWV
        if (!kern) return fail(ATLAS_EINVAL, "level_vec not available for this dtype and operator");
        ATLASX_HIP(hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, dim3(per * 8), block, lds, st, m, in, out, nlev, vpc, m.ntiles,
                           per);
        break;
      }
      // wavefront w stages nodes w, w + nw, ... of a run: EPT >= segmax / nw;
      // four runs of kc levels must fit in LDS (the chunk shrinks if needed)
      const size_t vbytes = sizeof(T) * (OP == OP_GRAD ? 1 : 2);
      int kc = sweep_chunk(nlev, sh.level_chunk);
      kc = min(kc, (int)(kMaxLds / (4 * vbytes * (size_t)max(1, m.segmax))));
      if (kc < 1) return fail(ATLAS_EINVAL, "sweep tile too large for LDS");
      const int nchunk = (nlev + kc - 1) / kc;
      const size_t lds = (size_t)4 * m.segmax * kc * vbytes;
      const int need = (m.segmax + (sh.block >> 6) - 1) / (sh.block >> 6);
      const int units = m.ntiles * nchunk;
      const int per = (units + 7) / 8;
      void (*kern)(DevMesh, const T *, T *, int, int, int, int) = nullptr;
      if (need <= 4) kern = k_sweep<T, OP, 4>;
      else if (need <= 8) kern = k_sweep<T, OP, 8>;
      else if (need <= 16) kern = k_sweep<T, OP, 16>;
      else if (need <= 32) kern = k_sweep<T, OP, 32>;
      else return fail(ATLAS_EINVAL, "sweep tile too large for the block size");
      ATLASX_HIP(hipFuncSetAttribute((const void *)kern,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      hipLaunchKernelGGL(kern, dim3(per * 8), block, lds, st, m, in, out, nlev, kc, m.ntiles, per);
      break;
    }
    case ATLAS_VARIANT_FUSED:
      return fail(ATLAS_EINVAL, "the fused variant is for the Laplacian only");
    default:
      return fail(ATLAS_EINVAL, "unknown launch variant");
  }
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

template <class T>
static atlas_status launch_dtype(const MeshStore &ms, atlas_op op, const void *in, int nlev,
                                 void *out, void *ws, const LaunchShape &sh, hipStream_t st) {
  const T *i = static_cast<const T *>(in);
  T *o = static_cast<T *>(out);
  switch (op) {
    case ATLAS_OP_GRADIENT: return launch_typed<T, OP_GRAD>(ms, i, nlev, o, ws, sh, st);
    case ATLAS_OP_DIVERGENCE: return launch_typed<T, OP_DIV>(ms, i, nlev, o, ws, sh, st);
    case ATLAS_OP_CURL: return launch_typed<T, OP_CURL>(ms, i, nlev, o, ws, sh, st);
    default: return fail(ATLAS_EINVAL, "unknown operator");
  }
}

// Shape of one Laplacian pass: the autotuned one for that operator, else the
// built-in one.
static LaunchShape pass_shape(const MeshStore &ms, atlas_op op, int nlev, atlas_dtype dt) {
  LaunchShape s;
  return tuned_shape(ms, op, nlev, dt, &s) ? s : default_shape(ms, op, nlev, dt);
}

// Laplacian: gradient into the workspace [V][nlev][2], then its divergence;
// the flux form needs its flux buffer behind the gradient.
// Divergence and curl of one field in one pass (column form, level-vector
// lanes of the divergence's automatic width).  Short columns (below 48
// levels) and meshes outside the level-vector form run the two operators
// one after the other with their own shapes (same results).
template <class T>
static atlas_status launch_div_curl_typed(const MeshStore &ms, atlas_dtype dt, const T *in,
                                          int nlev, T *od, T *oc, hipStream_t st) {
  const DevMesh &m = ms.d;
  {
    // where the wave-specialised sweep pays for the divergence, or for the
    // two together, the curl rides on the same loads (a tuned divergence keeps
    // its form)
    LaunchShape sh;
    if (!tuned_shape(ms, ATLAS_OP_DIVERGENCE, nlev, dt, &sh) &&
        !sweepw_builtin(ms, ATLAS_OP_DIVERGENCE, dt, nlev, true, &sh))
      sh = default_shape(ms, ATLAS_OP_DIVERGENCE, nlev, dt);
    if (sh.variant == ATLAS_VARIANT_SWEEP && sweepw_applies<T, OP_DIV>(m, nlev, sh)) {
      // (FP32 columns of several chunks: on large meshes (O1280, 137 levels 4.93
      // against 5.31 ms for the column form, O320 380 against 345 us); on smaller
      // ones where that form's three levels per lane are nearly used up or it
      // reads the column in parts: O320 in tiles of 367 nodes, 137 levels 347
      // against 333 us, 185: 357 against 413, 200: 504 against 431, 260: 526
      // against 667)
      const SweepwPlan p = sweepw_plan<T, OP_DIV, true>(ms, nlev, sh.level_chunk);
      if (p.lds <= kMaxLds && (p.nchunk == 1 || sizeof(T) == 8 || m.V >= 750000 ||
                               (nlev > 160 && nlev <= 192) || nlev > 256)) {
        sh.block = max(512, p.block);
        return launch_sweepw<T, OP_DIV, true>(ms, in, od, oc, nlev, sh, st);
      }
    }
  }
  const int nv = nlev >= 48 ? auto_level_vec<T, OP_DIV>(nlev, m.maxdeg, m.mindeg) : 0;
  if (nv == 0) {
    for (atlas_op op : {ATLAS_OP_DIVERGENCE, ATLAS_OP_CURL}) {
      LaunchShape sh = shape_from(nullptr, ms, op, nlev, dt);
      if (sh.variant == ATLAS_VARIANT_FLUX) sh = default_shape(ms, op, nlev, dt);
      atlas_status s = launch_op(ms, op, dt, in, nlev, op == ATLAS_OP_CURL ? (void *)oc : (void *)od,
                                 nullptr, sh, st);
      if (s != ATLAS_OK) return s;
    }
    return ATLAS_OK;
  }
  const int nvec = (nlev + nv - 1) / nv, nch = (nvec + 63) / 64;
  constexpr int kNpb = 16;
  const int ntiles = (m.V + kNpb - 1) / kNpb;
  const int per_xcd = (ntiles + 7) / 8;
  void (*kern)(DevMesh, const T *, T *, T *, int, int, int) = nullptr;
#define ATLASX_DC(NV)                                                  \
  if constexpr (lane_vec_ok<T, OP_DIV, NV>()) {                          \
    if (nch == 1) kern = k_colv_dc<T, NV, 1>;                            \
    else if (nch == 2) kern = k_colv_dc<T, NV, 2>;                       \
    else if (nch == 3) kern = k_colv_dc<T, NV, 3>;                       \
    else kern = k_colv_dc<T, NV, 4>;                                     \
  }
  if (nv == 1) {
    ATLASX_DC(1)
  } else if (nv == 2) {
    ATLASX_DC(2)
  } else if (nv == 3) {
    ATLASX_DC(3)
  } else {
    ATLASX_DC(4)
  }
#undef ATLASX_DC
  if (!kern || nch > 4) return fail(ATLAS_EINVAL, "no level-vector width for this column");
  hipLaunchKernelGGL(kern, dim3(per_xcd * 8), dim3(256), 0, st, m, in, od, oc, nlev, kNpb,
                     per_xcd);
  ATLASX_HIP(hipGetLastError());
  return ATLAS_OK;
}

atlas_status launch_div_curl(const MeshStore &ms, atlas_dtype dt, const void *in, int nlev,
                             void *out_div, void *out_curl, hipStream_t st) {
  if (dt == ATLAS_F64)
    return launch_div_curl_typed<double>(ms, dt, static_cast<const double *>(in), nlev,
                                         static_cast<double *>(out_div),
                                         static_cast<double *>(out_curl), st);
  return launch_div_curl_typed<float>(ms, dt, static_cast<const float *>(in), nlev,
                                      static_cast<float *>(out_div),
                                      static_cast<float *>(out_curl), st);
}

// The fused Laplacian's launch plan: lane width, level chunk and LDS bytes;
// false where the plan or the kernel's assumptions do not hold (no plan,
// rows outside 4..6 incidences, a block too small for the staging, runs too
// long for LDS).
struct FusedPlan {
  int nv, vpc, nchunk;
  size_t lds;
};
template <class T>
static bool fused_plan(const MeshStore &ms, int nlev, const LaunchShape &sh, FusedPlan *fp) {
  const DevMesh &m = ms.d;
  if (!m.l2_ok || m.maxdeg > 6 || m.mindeg < kMinRow) return false;
  constexpr int NVW = (int)(16 / sizeof(T));  // 16-byte field lanes
  const int nv = (nlev >= NVW && sh.level_vec != 1) ? NVW : 1;
  const int nvec = (nlev + nv - 1) / nv;
  const size_t fb = (size_t)nv * sizeof(T), gb = 2 * fb;  // lane-vector bytes
  const size_t per_vec = 4 * (size_t)m.l2_fmax * fb + 4 * (size_t)m.l2_gmax * gb;
  // two slots of packed geometry; a thread stages at most kGeoEpt words
  const size_t geo_words = (size_t)m.l2_gmax * kGGeoWords +
                           (size_t)m.l2_pmax * (sizeof(T) == 8 ? kLGeoWords64 : kLGeoWords);
  const size_t geo = 2 * geo_words * 16;
  if (geo_words > (size_t)kGeoEpt * sh.block) return false;
  int vpc = sh.level_chunk > 0 ? min(64, (sh.level_chunk + nv - 1) / nv) : 64;
  vpc = min(vpc, nvec);
  {
    const int nchunk = (nvec + vpc - 1) / vpc;
    vpc = (nvec + nchunk - 1) / nchunk;
  }
  // the chunk shrinks until both rings fit in LDS and a field run fits the
  // staging registers (kLsweepEpt lane vectors per thread)
  while (vpc > 1 && (per_vec * vpc + geo > kMaxLds ||
                     ((size_t)m.l2_fmax * vpc + sh.block - 1) / sh.block > (size_t)kLsweepEpt))
    vpc = (vpc + 1) / 2;
  if (per_vec * vpc + geo > kMaxLds ||
      ((size_t)m.l2_fmax * vpc + sh.block - 1) / sh.block > (size_t)kLsweepEpt)
    return false;
  fp->nv = nv;
  fp->vpc = vpc;
  fp->nchunk = (nvec + vpc - 1) / vpc;
  fp->lds = per_vec * vpc + geo;
  return true;
}

// The wave-specialised fused Laplacian's plan (blocks_per_cu 0, 16-byte
// vectors, at least one consumer wavefront): the cut of the tiles with the
// fewest level chunks (then the fewest parts, then the fewest steps until
// the last round of workgroups is done), and chunks for two workgroups per
// compute unit before that; false where none fits in LDS.
// (nodes_per_block 4 and 5 chose a ring in earlier forms and are taken as 0.)
template <class T>
static bool fusedw_plan(const MeshStore &ms, int nlev, const LaunchShape &sh, FusedwPlan *fp) {
  const DevMesh &m = ms.d;
  constexpr int NVW = (int)(16 / sizeof(T));
  if (ms.lcuts.empty() || m.mindeg < kMinRow || !m.sgeo_n) return false;
  if (sh.blocks_per_cu != 0 || sh.level_vec == 1 || nlev < NVW) return false;
  if (sh.block < 320) return false;
  if (sh.nodes_per_block != 0 && sh.nodes_per_block != 4 && sh.nodes_per_block != 5) return false;
  // (field runs far longer than the tiles' own rows, as a regular grid's
  // polar rows need, leave room for a level or two: F640, 37 levels, 17.2
  // against 2.8 ms for the two passes)
  if (ms.lcuts[0].fmax > 2 * ms.lcuts[0].pmax + 16) return false;
  const int nvec = (nlev + NVW - 1) / NVW;
  const int most = 32 * kLswMaxNe / 2;
  const int want = sh.level_chunk > 0 ? (sh.level_chunk + NVW - 1) / NVW : most;
  const int cus = device_cu_count();
  int64_t best_steps = 0;
  bool any = false;
  bool two = false;  // the plan so far lets two workgroups share a compute unit
  for (size_t k = 0; k < ms.lcuts.size(); ++k) {
    const LaplView &v = ms.lcuts[k];
    auto bytes = [&](int c) {
      return (size_t)16 * ((size_t)kLswFieldSlots * v.fmax * c +
                           (size_t)kLswGradSlots * v.gmax * 2 * c +
                           (size_t)kLswRecSlots * v.gmax * kSgeoWordsS +
                           (size_t)kLswRefSlots * (v.gmax + v.pmax)) +
             (sizeof(T) == 4 ? (size_t)8 * kLswGradSlots * v.gmax : 0) + kSweepwLdsTail;
    };
    // (a field run is loaded by one wavefront's kRunLoads instructions)
    auto fits = [&](int c) {
      return bytes(c) <= kMaxLds && v.fmax * c <= kRunLoads * 64 * kLswGroupWaves;
    };
    int vpc = min(min(want, most), nvec);
    int nchunk = (nvec + vpc - 1) / vpc;
    vpc = (nvec + nchunk - 1) / nchunk;
    while (vpc > 1 && !fits(vpc)) {
      ++nchunk;
      vpc = (nvec + nchunk - 1) / nchunk;
    }
    nchunk = (nvec + vpc - 1) / vpc;
    if (!fits(vpc)) continue;
    // One workgroup on a compute unit waits out each step's barrier and
    // loads; two of eight wavefronts hide them.  A column that one or two more
    // chunks bring down to 13 to 16 vectors (two elements on 16 lanes; 17 and
    // 18 leave a third of the lanes idle) takes them, on the cut where two
    // such workgroups fit (O1280: FP64, 80 levels in three chunks of 14 on half
    // tiles 4.47 ms, two of 20 5.60; 60 levels 3.02 against 3.19, 120 5.96 against
    // 6.41; 100 levels in three of 17 8.01 against 6.36, in four of 13 5.96; FP32,
    // 170 levels 5.82 against 7.04, 100 3.91 against 4.20).  Not three for one (75
    // levels, one of 38 3.68 ms, three of 13 4.43; FP32, 150: 4.88 against 5.84),
    // and not on tiles of fewer than 512 nodes, whose halves form more gradients
    // twice (O320 in tiles of 368: FP32, 100 levels, 341 against 359 us).
    bool pair = false;
    if (sh.level_chunk == 0 && m.V >= 512 * (int64_t)m.ntiles && 2 * bytes(vpc) > kMaxLds) {
      for (int n = nchunk + 1; n <= min(nchunk + 2, 2 * nchunk) && !pair; ++n) {
        const int c = (nvec + n - 1) / n;
        if (c >= 13 && c <= 16 && fits(c) && 2 * bytes(c) <= kMaxLds) {
          vpc = c;
          pair = true;
        }
      }
      if (pair) nchunk = (nvec + vpc - 1) / vpc;
    }
    FusedwPlan p;
    p.cut = (int)k;
    p.vpc = vpc;
    p.nchunk = nchunk;
    p.lds = bytes(vpc);
    const bool better = !any || pair > two ||
                        (pair == two && (nchunk < fp->nchunk ||
                                         (nchunk == fp->nchunk &&
                                          v.parts < ms.lcuts[fp->cut].parts)));
    if (!better && (pair < two || nchunk > fp->nchunk || v.parts > ms.lcuts[fp->cut].parts))
      continue;
    // Lanes per position and elements per lane: the cheapest pair that holds
    // the chunk, as in the sweep -- but not eight lanes with four elements or
    // more: eight positions a wavefront leave a run of 34 to four or five of
    // the wavefronts, each with a long chain (O1280, 30 levels, 1.91 ms, on 16
    // lanes 1.60; O500, 37 levels, 522 against 468 us; FP32, 80 levels, O640 1062
    // against 949) -- except 34 to 36 elements in FP32, of which 16 lanes take
    // three with a quarter of them idle (O640, 72 levels, 655 against 698 us;
    // FP64, 36 levels, 545 against 527).
    const int nel = p.vpc * 2;
    int cost = INT_MAX;
    for (int l : {8, 16, 32}) {
      const int e = (nel + l - 1) / l;
      const bool lanes8 = e <= 3 || (sizeof(T) == 4 && e == 5 && nel <= 36);
      if ((l > 8 || lanes8) && e <= kLswMaxNe && (e + 3) * l < cost) {
        cost = (e + 3) * l;
        p.lpn = l;
        p.ne = e;
      }
    }
    const int npn = 64 / p.lpn;
    const int tasks = (v.gmax + npn - 1) / npn + (v.pmax + npn - 1) / npn;
    p.block = pair ? 512 : min(kLswBlock, 64 * (kLswProducers + tasks));
    const int64_t places = (int64_t)cus * max(1, min((int)(kMaxLds / p.lds), 1024 / p.block));
    const int64_t steps =
        ((int64_t)v.ntiles * p.nchunk + places - 1) / places * (v.rings + 6);
    if (better || steps < best_steps) {
      *fp = p;
      best_steps = steps;
      two = pair;
      any = true;
    }
  }
  return any;
}

int lapl_fused_block(const MeshStore &ms, int nlev, atlas_dtype dt, const LaunchShape &sh) {
  if (sh.variant != ATLAS_VARIANT_FUSED) return 0;
  FusedPlan fp;
  FusedwPlan fw;
  if (dt == ATLAS_F64 ? fusedw_plan<double>(ms, nlev, sh, &fw)
                      : fusedw_plan<float>(ms, nlev, sh, &fw))
    return min(sh.block, kLswBlock);
  return (dt == ATLAS_F64 ? fused_plan<double>(ms, nlev, sh, &fp)
                          : fused_plan<float>(ms, nlev, sh, &fp)) ? sh.block : 0;
}

bool lapl_fused_runs(const MeshStore &ms, int nlev, atlas_dtype dt, const LaunchShape &sh) {
  return lapl_fused_block(ms, nlev, dt, sh) != 0;
}

// The fused Laplacian on the two-ring plan; *ran = false (nothing
// launched) where fused_plan refuses.
template <class T>
atlas_status launch_lapl_fused(const MeshStore &ms, const T *in, int nlev, T *out,
                               const LaunchShape &sh, hipStream_t st, bool *ran) {
  const DevMesh &m = ms.d;
  *ran = false;
  constexpr int NVW = (int)(16 / sizeof(T));
  FusedwPlan fw;
  if (fusedw_plan<T>(ms, nlev, sh, &fw)) {
    const LaplView &v = ms.lcuts[fw.cut];
    const int64_t units = (int64_t)v.ntiles * fw.nchunk;
    const int per = (int)((units + 7) / 8);
    auto kern = lsweepw_kernel<T>(fw.lpn, fw.ne);
    ATLASX_HIP(hipFuncSetAttribute((const void *)kern,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)fw.lds));
    hipLaunchKernelGGL(kern, dim3(per * 8), dim3(min(sh.block, kLswBlock)), fw.lds, st, v, m.sgeo_n, in, out, nlev,
                       fw.vpc, per);
    ATLASX_HIP(hipGetLastError());
    *ran = true;
    return ATLAS_OK;
  }
  FusedPlan fp;
  if (!fused_plan<T>(ms, nlev, sh, &fp)) return ATLAS_OK;
  const int nv = fp.nv, vpc = fp.vpc, nchunk = fp.nchunk;
  const size_t lds = fp.lds;
  const int units = m.ntiles * nchunk;
  const int per = (units + 7) / 8;
  // each lane walks nl lane vectors of a node (blocks_per_cu 1..3 picks
  // nl; 0: one), so a node takes lpn = vpc / nl lanes (rounded up) and a
  // wavefront 64 / lpn nodes
  const int nl = sh.blocks_per_cu >= 1 && sh.blocks_per_cu <= 3 ? sh.blocks_per_cu : 1;
  const int lpn = (vpc + nl - 1) / nl;
  void (*kern)(DevMesh, const T *, T *, int, int, int, int, int) = nullptr;
  if (nv == 1)
    kern = nl == 1 ? k_lsweep<T, 1, kLsweepEpt, 1>
           : nl == 2 ? k_lsweep<T, 1, kLsweepEpt, 2> : k_lsweep<T, 1, kLsweepEpt, 3>;
  else
    kern = nl == 1 ? k_lsweep<T, NVW, kLsweepEpt, 1>
           : nl == 2 ? k_lsweep<T, NVW, kLsweepEpt, 2> : k_lsweep<T, NVW, kLsweepEpt, 3>;
  ATLASX_HIP(hipFuncSetAttribute((const void *)kern,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kern, dim3(per * 8), dim3(sh.block), lds, st, m, in, out, nlev, vpc,
                     m.ntiles, per, lpn);
  ATLASX_HIP(hipGetLastError());
  *ran = true;
  return ATLAS_OK;
}

// Scales of the derivatives in the computational plane: d/dlon = R cos(lat)
// times the zonal component, d/dlat = R times the meridional one, i.e. both
// sums over the node's edges divided by its (lon, lat) dual area
// A_i = V_i / (R^2 cos lat_i): alpha = beta = R beta_i.
__global__ void k_comp_scales(int V, double R, const PosRec *__restrict__ pos,
                              double *__restrict__ alpha, double *__restrict__ beta,
                              PosRec *__restrict__ pos_c) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < V) {
    PosRec r = pos[p];
    const double s = R * r.beta;
    r.alpha = s;
    r.beta = s;
    alpha[p] = s;
    beta[p] = s;
    pos_c[p] = r;
  }
}

atlas_status gradient_lonlat(MeshStore &ms, atlas_dtype dt, const void *in, int nlev, void *out,
                             hipStream_t st) {
  {
    std::lock_guard<std::mutex> g(ms.comp_mu);
    if (!ms.comp_ready) {
      const int V = ms.d.V;
      void *p = nullptr, *a = nullptr, *b = nullptr;
      if (hipMalloc(&p, sizeof(PosRec) * (size_t)V) != hipSuccess)
        return fail(ATLAS_ENOMEM, "derivative scales");
      ms.allocations.push_back(p);
      if (hipMalloc(&a, sizeof(double) * (size_t)V) != hipSuccess)
        return fail(ATLAS_ENOMEM, "derivative scales");
      ms.allocations.push_back(a);
      if (hipMalloc(&b, sizeof(double) * (size_t)V) != hipSuccess)
        return fail(ATLAS_ENOMEM, "derivative scales");
      ms.allocations.push_back(b);
      ms.bytes += (sizeof(PosRec) + 16) * (size_t)V;
      hipLaunchKernelGGL(k_comp_scales, dim3((V + 255) / 256), dim3(256), 0, 0, V, ms.radius,
                         ms.d.pos, static_cast<double *>(a), static_cast<double *>(b),
                         static_cast<PosRec *>(p));
      ATLASX_HIP(hipGetLastError());
      ATLASX_HIP(hipDeviceSynchronize());
      ms.dcomp = ms.d;
      ms.dcomp.pos = static_cast<const PosRec *>(p);
      ms.dcomp.alpha = static_cast<const double *>(a);
      ms.dcomp.beta = static_cast<const double *>(b);
      ms.dcomp.sgeo = nullptr;  // packed geometry holds the physical scales
      ms.dcomp.l2_ok = 0;
      ms.comp_ready = true;
    }
  }
  // the built-in gradient shape among the forms that read the scales by
  // position
  const LaunchShape sh = default_shape(ms, ATLAS_OP_GRADIENT, nlev, dt, false);
  if (dt == ATLAS_F64)
    return launch_typed<double, OP_GRAD>(ms, static_cast<const double *>(in), nlev,
                                         static_cast<double *>(out), nullptr, sh, st, &ms.dcomp);
  return launch_typed<float, OP_GRAD>(ms, static_cast<const float *>(in), nlev,
                                      static_cast<float *>(out), nullptr, sh, st, &ms.dcomp);
}

atlas_status launch_op(const MeshStore &ms, atlas_op op, atlas_dtype dt, const void *in,
                       int nlev, void *out, void *ws, const LaunchShape &sh, hipStream_t st) {
  if (op == ATLAS_OP_LAPLACIAN && sh.variant == ATLAS_VARIANT_FUSED) {
    bool ran = false;
    const atlas_status s =
        dt == ATLAS_F64
            ? launch_lapl_fused<double>(ms, static_cast<const double *>(in), nlev,
                                        static_cast<double *>(out), sh, st, &ran)
            : launch_lapl_fused<float>(ms, static_cast<const float *>(in), nlev,
                                       static_cast<float *>(out), sh, st, &ran);
    if (s != ATLAS_OK || ran) return s;
    // otherwise the two passes with their built-in shapes (same results)
    if (!ws) return fail(ATLAS_EINVAL, "the two-pass Laplacian needs a workspace");
    LaunchShape two = sh;
    two.variant = ATLAS_VARIANT_COLUMN;
    two.per_pass = 1;
    return launch_op(ms, op, dt, in, nlev, out, ws, two, st);
  }
  if (op == ATLAS_OP_LAPLACIAN) {
    if (!ws) return fail(ATLAS_EINVAL, "the two-pass Laplacian needs a workspace");
    const size_t w = dt == ATLAS_F64 ? 8 : 4;
    char *grad = static_cast<char *>(ws);
    void *flux = grad + (size_t)ms.d.V * nlev * 2 * w;
    const LaunchShape sg = sh.per_pass ? pass_shape(ms, ATLAS_OP_GRADIENT, nlev, dt) : sh;
    const LaunchShape sd = sh.per_pass ? pass_shape(ms, ATLAS_OP_DIVERGENCE, nlev, dt) : sh;
    atlas_status s = launch_op(ms, ATLAS_OP_GRADIENT, dt, in, nlev, grad, flux, sg, st);
    if (s != ATLAS_OK) return s;
    return launch_op(ms, ATLAS_OP_DIVERGENCE, dt, grad, nlev, out, flux, sd, st);
  }
  if (dt == ATLAS_F64) return launch_dtype<double>(ms, op, in, nlev, out, ws, sh, st);
  return launch_dtype<float>(ms, op, in, nlev, out, ws, sh, st);
}

}  // namespace atlasx
