// Small levels of the V-cycle (vertex smoother, subdomains of 2 x 2 x 2 elements).
//
// On levels of up to 32^3 elements the separate kernels of a smoothing step (residual,
// condensation, patch products, interface sum) and of the transfers take 4 to 7 us each, for
// work of well under 1 us: each is a chain of two to four dependent memory round trips behind
// a launch.  Here a launch does as much as one exchange between work items allows, and a
// block or wavefront owns one item:
//   k_small_patch     one block per vertex: everything the patch of a vertex V needs lies in
//                     the 4^3 elements around V (108 inner edges, 300 edges in all).  The
//                     block loads z and g there (and the coarse correction, which it
//                     prolongs), forms the residual on the 108 inner edges, condenses it
//                     onto the 60 slots, and multiplies by S_type^{-1}, one result row per
//                     lane.  Each inner edge is computed by the up to 8 patches that hold it.
//   k_small_pull      one wavefront per subdomain: sums the patch results on its 48 boundary
//                     edges, extends them into its interior and updates its 24 unknowns.
//   k_small_restrict  one block per coarse node: the 54 fine residuals its three edges
//                     restrict, then the weighted sums.
// All loads that do not depend on one another go out before the first wait, the convergence
// flag's among them (tested before the first store).  What bounds them is latency: launch,
// one or two round trips and the LDS phases.  Measured at 16^3 in FP32: 5.8 us for
// prolongation, residual, condensation and patch products (separate kernels 19), 4.6 for
// condensation and patch products (10), 3.5 for the interface sum (7), 3.9 for residual and
// restriction (9).  A level takes 5 launches instead of 10.  One wavefront per vertex instead
// of a block measured slower (6.9 us at 10^3: about 900 instructions one after another); so
// did the condensed residual as a launch of its own before the MFMA patch products at every
// size.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "apply_lds.hpp"
#include "ndmg_internal.hpp"
#include "small.hpp"

namespace ndmg {

namespace {

__device__ __forceinline__ int64_t lin(const DGeom& g, int i, int j, int k) {
  return (int64_t)k * g.plane + (int64_t)j * g.P + i;
}

// contiguous ranges of logical blocks per XCD (hardware deals blocks to the 8 XCDs in turn)
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, i = b >> 3;
  return x * q + min(x, r) + i;
}

// keeps the loads above it from sinking below a branch
__device__ __forceinline__ void issue_barrier() { __asm__ volatile("" ::: "memory"); }

// The cube of a block: the nodes around its vertices, 2 V - 2 .. 2 V + 2 of each axis (one
// vertex, CX = 5 nodes along x; two neighbours along x, CX = 7), an array [3][5][5][CX] of
// edges by their first node.
template <int CX>
struct CubeShape {
  static constexpr int N = 25 * CX;                       // entries per direction
  static constexpr int st[3] = {1, CX, 5 * CX};
  static __device__ __forceinline__ int at(int x, int y, int z) { return x + CX * y + 5 * CX * z; }
  static __device__ __forceinline__ void pos(int m, int& x, int& y, int& z) {
    z = m / (5 * CX);
    const int q = m - z * 5 * CX;
    y = q / CX;
    x = q - y * CX;
  }
};

// Lower node of a cube in the level.
struct Cube {
  int x0, y0, z0, n;
  __device__ __forceinline__ bool inside(int x, int y, int z) const {
    return (unsigned)(x0 + x) <= (unsigned)n && (unsigned)(y0 + y) <= (unsigned)n && (unsigned)(z0 + z) <= (unsigned)n;
  }
  // the edge of direction d at cube node (x, y, z) is an unknown
  __device__ __forceinline__ bool unknown(int d, int x, int y, int z) const {
    return x0 + x >= (d != 0) && y0 + y >= (d != 1) && z0 + z >= (d != 2) && x0 + x < n && y0 + y < n && z0 + z < n;
  }
};

// entry m of direction d of v on the cube; 0 outside [0, n]^3
template <int CX, typename T>
__device__ __forceinline__ T load_cube(const T* __restrict__ v, const DGeom& g, const Cube& q, int d, int m) {
  int x, y, z;
  CubeShape<CX>::pos(m, x, y, z);
  const bool ok = q.inside(x, y, z);
  const T t = v[ok ? d * g.B + lin(g, q.x0 + x, q.y0 + y, q.z0 + z) : 0];
  return ok ? t : T(0);
}

// the same at position p of direction D of a cube, every stride a constant
template <int D, int CX, bool COEF, typename T>
__device__ __forceinline__ T apply_cube(const T* L, int p, T ah, T h3, T c00, T c10, T c01, T c11) {
  using S = CubeShape<CX>;
  return apply_lds<COEF>(L + D * S::N + p, L + (D + 1) % 3 * S::N + p, L + (D + 2) % 3 * S::N + p, S::st[D],
                         S::st[(D + 1) % 3], S::st[(D + 2) % 3], ah, h3, c00, c10, c01, c11);
}

// Coefficient boxes: the factor of cell m of a cube (CX - 1 cells along x, 4 x 4 across), 0
// outside the level (and in the boxes outside a domain: no unknown touches such a cell).
template <int CX>
__device__ __forceinline__ double load_cell(const Bat& bt, const Cube& q, const BoxDiv& dv, int m) {
  const int cz = m / (4 * (CX - 1)), cq = m - cz * 4 * (CX - 1), cy = cq / (CX - 1), cx = cq - cy * (CX - 1);
  const int x = q.x0 + cx, y = q.y0 + cy, z = q.z0 + cz;
  const bool ok = (unsigned)x < (unsigned)q.n && (unsigned)y < (unsigned)q.n && (unsigned)z < (unsigned)q.n;
  const int r = bt.coef_r;
  const double f = bt.coef[ok ? (dv.box(z >> 1) * r + dv.box(y >> 1)) * r + dv.box(x >> 1) : 0];
  return ok ? f : 0.0;
}

struct Pos {
  int x, y, z;
};
// edge of direction d at offset a along it and b, c across (axes d + 1, d + 2)
__device__ __forceinline__ Pos edge_pos(int d, int a, int b, int c) {
  return d == 0 ? Pos{a, b, c} : (d == 1 ? Pos{c, a, b} : Pos{b, c, a});
}
// factors of the four cells around the edge of direction d at p, from the cube's cells
template <int CX, typename T>
__device__ __forceinline__ void edge_cells(const T* fL, int d, const Pos& p, T& c00, T& c10, T& c01, T& c11) {
  const int cell = p.x + (CX - 1) * (p.y + 4 * p.z);
  const int sx = 1, sy = CX - 1, sz = 4 * (CX - 1);
  const int sb = d == 0 ? sy : (d == 1 ? sz : sx), sc = d == 0 ? sz : (d == 1 ? sx : sy);
  c00 = fL[cell - sb - sc];
  c10 = fL[cell - sc];
  c01 = fL[cell - sb];
  c11 = fL[cell];
}

// I zc at the edge of direction D at cube node (x, y, z), from the coarse cube cL
// ([3][3][3][CC], from the node half the cube's lower node): weight 1/2 each side across an
// axis at an odd offset (the cube's lower node is even)
template <int D, int CC, typename T>
__device__ __forceinline__ T prolong_cube(const T* cL, int x, int y, int z) {
  const int o[3] = {x, y, z};
  constexpr int st[3] = {1, CC, 3 * CC};
  const int ob = o[(D + 1) % 3] & 1, oc = o[(D + 2) % 3] & 1;
  const int sb = ob * st[(D + 1) % 3], sc = oc * st[(D + 2) % 3];
  const T* e = cL + 9 * CC * D + (x >> 1) + CC * (y >> 1) + 3 * CC * (z >> 1);
  const T wb0 = ob ? T(0.5) : T(1), wb1 = ob ? T(0.5) : T(0);
  const T wc0 = oc ? T(0.5) : T(1), wc1 = oc ? T(0.5) : T(0);
  const T lo = wb0 * e[0] + wb1 * e[sb], hi = wb0 * e[sc] + wb1 * e[sb + sc];
  return wc0 * lo + wc1 * hi;
}

// One block per NV vertices V, V + e_x (NV = 2: the pairs (2 p - 1, 2 p), which share their
// cube's residuals and, inside a type's range, S^{-1}; a pair's vertex outside 0 .. nH is
// computed from zeros and not stored).  Wave d < 3 works on the edges of direction d.
// MODE 0: r = g; 1: r = g - A z; 2: r = g - A (z + I zc).  COEF: coefficient boxes, with the
// patch type from the vertex's class triple (BoxPatches) and X_T from each subdomain's box.
template <typename T, int MODE, bool COEF, int NV>
__global__ void __launch_bounds__(256) k_small_patch(const T* __restrict__ g, const T* __restrict__ z,
                                                     const T* __restrict__ zc, SmallSub<T> s, DGeom gc, Bat bt) {
  constexpr int NG = 60, NPAD = 64, NX = 288, NC = NG / 4;
  constexpr int CX = 3 + 2 * NV, CC = 2 + NV;
  using S = CubeShape<CX>;
  constexpr int NL = (S::N + 63) / 64, NF = (16 * (CX - 1) + 63) / 64;
  __shared__ T zL[MODE ? 3 * S::N : 1];
  __shared__ T rL[3 * S::N];
  __shared__ T cL[MODE == 2 ? 27 * CC : 1];
  __shared__ T xL[COEF ? 1 : NX];
  __shared__ T fL[COEF ? 64 * NF : 1];
  __shared__ T gL[NV][NPAD];
  __shared__ T pL[NV][4][NPAD];
  const int nv = s.nH + 1, nv3 = nv * nv * nv, nb = NV == 1 ? nv : nv / 2 + 1;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int pair = lb / (nb * nv * nv), v = lb - pair * (nb * nv * nv);
  const int vx = NV == 1 ? v % nb : 2 * (v % nb) - 1, vy = (v / nb) % nv, vz = v / (nb * nv);
  const int act = bt.act ? bt.act[pair] : 1;
  const int prob = pair / bt.nrhs;
  const T ah = MODE ? (T)(bt.alpha[prob] * s.h) : T(0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t off = (int64_t)pair * 3 * s.g.B;
  const Cube q{2 * vx - 2, 2 * vy - 2, 2 * vz - 2, s.g.n};
  T zv[NL], cv = T(0), gv = T(0), xv[COEF ? 6 * NV : 5], sv[NC];
  double fv[NF];
  // condensation: four lanes per slot, one subdomain each
  const uint32_t* __restrict__ tab = s.tab + kSmallSlots + 5 * min(tid >> 2, NG - 1);
  const uint32_t slot = tab[0], code = tab[1 + (tid & 3)];
  // patch type of vertex j
  auto type_of = [&](int j) {
    const int x = min(max(vx + j, 0), s.nH);
    if constexpr (COEF) {
      const int K = 2 * bt.coef_r + 1;
      auto cls = [&](int u) {
        const int b = s.dv.box(u);
        return 2 * b + (u != b * s.dv.w ? 1 : 0);
      };
      return s.cls[2 * ((cls(vz) * K + cls(vy)) * K + cls(x)) + 1];
    } else {
      return (x == 0 ? 0 : (x == s.nH ? 2 : 1)) + 3 * (vy == 0 ? 0 : (vy == s.nH ? 2 : 1)) +
             9 * (vz == 0 ? 0 : (vz == s.nH ? 2 : 1));
    }
  };
  int type[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) type[j] = type_of(j);
  // this lane's inner edge of direction `wave`: nodes 1 .. 3 (along x: CX - 2) across it
  const int nx = wave == 0 ? CX - 1 : CX - 2;           // positions along x
  const int ninner = wave == 0 ? 9 * (CX - 1) : 12 * (CX - 2);
  const int il = min(lane, ninner - 1);
  const int ix = il % nx, iq = il / nx;
  const Pos ip = wave == 0 ? Pos{ix, 1 + iq % 3, 1 + iq / 3}
                           : (wave == 1 ? Pos{1 + ix, iq & 3, 1 + iq / 4} : Pos{1 + ix, 1 + iq % 3, iq / 3});
  const bool iu = wave < 3 && q.unknown(wave, ip.x, ip.y, ip.z);
  if (wave < 3) {
    if constexpr (MODE != 0) {
#pragma unroll
      for (int i = 0; i < NL; ++i) zv[i] = load_cube<CX>(z + off, s.g, q, wave, min(lane + 64 * i, S::N - 1));
    }
    if constexpr (MODE == 2) {
      const int m = min(lane, 9 * CC - 1), w = m / (3 * CC), y = m / CC % 3, x = m % CC;
      const bool ok = (unsigned)(vx - 1 + x) <= (unsigned)gc.n && (unsigned)(vy - 1 + y) <= (unsigned)gc.n &&
                      (unsigned)(vz - 1 + w) <= (unsigned)gc.n;
      const T t = zc[(int64_t)pair * 3 * gc.B + (ok ? wave * gc.B + lin(gc, vx - 1 + x, vy - 1 + y, vz - 1 + w) : 0)];
      cv = ok ? t : T(0);
    }
    gv = g[off + (iu ? wave * s.g.B + lin(s.g, q.x0 + ip.x, q.y0 + ip.y, q.z0 + ip.z) : 0)];
  } else if constexpr (COEF) {
#pragma unroll
    for (int i = 0; i < NF; ++i) fv[i] = load_cell<CX>(bt, q, s.dv, min(lane + 64 * i, 16 * (CX - 1) - 1));
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) xv[i] = s.XT[(int64_t)prob * NX + min(lane + 64 * i, NX - 1)];
  }
  // subdomain (of the 8 around a vertex) and boundary edge of this lane's condensation term
  const bool on = code != 0xffff;
  const int sx = code & 1, sy = (code >> 1) & 1, sz = (code >> 2) & 1, ce = on ? (int)(code >> 3) : 0;
  if constexpr (COEF) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      // (a subdomain outside the cube has no term: its slots are absent)
      const int r = bt.coef_r, m = s.nH - 1;
      const int a = min(max(vx + j - 1 + sx, 0), m), b = min(max(vy - 1 + sy, 0), m), c = min(max(vz - 1 + sz, 0), m);
      const T* __restrict__ X = s.XT + ((s.dv.box(c) * r + s.dv.box(b)) * r + s.dv.box(a)) * NX + ce;
#pragma unroll
      for (int t = 0; t < 6; ++t) xv[6 * j + t] = X[t * 48];
    }
  }
  // S^{-1} is symmetric: column k of this lane's row is entry (k, lane); wave w takes the
  // columns 15 w .. 15 w + 14
  auto load_s = [&](int ty) {
    const T* __restrict__ Sm = s.Sinv + prob * s.sstride + (int64_t)ty * NPAD * NPAD + wave * NC * NPAD + lane;
#pragma unroll
    for (int k = 0; k < NC; ++k) sv[k] = Sm[k * NPAD];
  };
  load_s(type[0]);
  issue_barrier();
  if (act == 0) return;
  if (wave == 3) {
    if constexpr (COEF) {
#pragma unroll
      for (int i = 0; i < NF; ++i) fL[lane + 64 * i] = (T)fv[i];
    } else {
#pragma unroll
      for (int i = 0; i < 5; ++i)
        if (lane + 64 * i < NX) xL[lane + 64 * i] = xv[i];
    }
  } else if constexpr (MODE == 0) {
    // (entries off the unknowns of a domain are zero in every residual)
    if (lane < ninner) rL[wave * S::N + S::at(ip.x, ip.y, ip.z)] = iu ? gv : T(0);
  } else if constexpr (MODE == 1) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (lane + 64 * i < S::N) zL[wave * S::N + lane + 64 * i] = zv[i];
  } else {
    if (lane < 9 * CC) cL[9 * CC * wave + lane] = cv;
    // (a wave prolongs its own direction from the coarse entries it has just written)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    auto prolong = [&](auto dir) {
      constexpr int D = decltype(dir)::value;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int m = min(lane + 64 * i, S::N - 1);
        int x, y, w;
        S::pos(m, x, y, w);
        // (an entry past the last element along its direction is not an edge of the cube)
        const T add = (D == 0 ? x < CX - 1 : (D == 1 ? y < 4 : w < 4)) ? prolong_cube<D, CC>(cL, x, y, w) : T(0);
        if (lane + 64 * i < S::N) zL[D * S::N + m] = zv[i] + add;
      }
    };
    if (wave == 0) prolong(std::integral_constant<int, 0>{});
    if (wave == 1) prolong(std::integral_constant<int, 1>{});
    if (wave == 2) prolong(std::integral_constant<int, 2>{});
  }
  __syncthreads();
  if constexpr (MODE != 0) {
    const T h3 = (T)(s.h * s.h * s.h);
    const int p = S::at(ip.x, ip.y, ip.z);
    T ax = T(0), c00 = T(1), c10 = T(1), c01 = T(1), c11 = T(1);
    if constexpr (COEF) edge_cells<CX>(fL, wave, ip, c00, c10, c01, c11);
    if (wave == 0) ax = apply_cube<0, CX, COEF>(zL, p, ah, h3, c00, c10, c01, c11);
    if (wave == 1) ax = apply_cube<1, CX, COEF>(zL, p, ah, h3, c00, c10, c01, c11);
    if (wave == 2) ax = apply_cube<2, CX, COEF>(zL, p, ah, h3, c00, c10, c01, c11);
    const bool in = iu && c00 > T(0) && c10 > T(0) && c01 > T(0) && c11 > T(0);
    if (wave < 3 && lane < ninner) rL[wave * S::N + p] = in ? gv - ax : T(0);
    __syncthreads();
  }
  {
    // interior unknown t of a subdomain: a constant offset from its lower node
    constexpr int io[6] = {6 * CX,             1 + 6 * CX,         S::N + 1 + 5 * CX,
                           S::N + 1 + 6 * CX,  2 * S::N + 1 + CX,  2 * S::N + 1 + 6 * CX};
    const int pos = (slot & 3) * S::N + S::at((slot >> 2) & 7, (slot >> 5) & 7, (slot >> 8) & 7);
    const T* rs = rL + S::at(2 * sx, 2 * sy, 2 * sz);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      T c = T(0);
#pragma unroll
      for (int t = 0; t < 6; ++t) c += (COEF ? xv[COEF ? 6 * j + t : 0] : xL[COEF ? 0 : t * 48 + ce]) * rs[2 * j + io[t]];
      c = on ? c : T(0);
      c += __shfl_xor(c, 1, 64);
      c += __shfl_xor(c, 2, 64);
      if ((tid & 3) == 0) gL[j][tid >> 2] = tid < 4 * NG ? rL[pos + 2 * j] - c : T(0);
    }
  }
  if constexpr (MODE != 0) {
    // r on the interiors of the subdomains whose lower corners are the vertices
    const int j = lane / 6, t = lane - 6 * j, a = vx + j;
    if (wave == 1 && lane < 6 * NV && a >= 0 && a < s.nH && vy < s.nH && vz < s.nH) {
      const int d = t >> 1, f = t & 1;   // (order of interior_dofs)
      const int ex = d == 0 ? f : 1, ey = d == 1 ? f : 1, ez = d == 2 ? f : 1;
      s.r[off + d * s.g.B + lin(s.g, 2 * a + ex, 2 * vy + ey, 2 * vz + ez)] =
          rL[d * S::N + S::at(2 + 2 * j + ex, 2 + ey, 2 + ez)];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j > 0 && type[j] != type[0]) load_s(type[j]);
    T y = T(0);
#pragma unroll
    for (int k = 0; k < NC; ++k) y += sv[k] * gL[j][wave * NC + k];
    pL[j][wave][lane] = y;
  }
  __syncthreads();
  if (wave < NV && vx + wave >= 0 && vx + wave <= s.nH)
    s.Y[((int64_t)pair * nv3 + (vz * nv + vy) * nv + vx + wave) * NPAD + lane] =
        (pL[wave][0][lane] + pL[wave][1][lane]) + (pL[wave][2][lane] + pL[wave][3][lane]);
}

// Lane e < 48: boundary edge e of the subdomain; lanes 48 .. 53: its interior unknowns.
// Bound by latency: one round trip for the table, one for everything else.
template <typename T>
__global__ void __launch_bounds__(64) k_small_pull(const T* __restrict__ r, T* z, const T* __restrict__ zc,
                                                   int assign, SmallSub<T> s, DGeom gc, Bat bt) {
  constexpr int NPAD = 64, NX = 288;
  __shared__ T wL[48];
  const int nH = s.nH, nv = nH + 1, nv3 = nv * nv * nv, ns = nH * nH * nH;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int pair = lb / ns, u = lb - pair * ns;
  const int a = u % nH, b = (u / nH) % nH, c = u / (nH * nH);
  const int act = bt.act ? bt.act[pair] : 1;
  // factors of the problem, or of the subdomain's box
  int prob = pair / bt.nrhs;
  if (bt.coef) prob = (s.dv.box(c) * bt.coef_r + s.dv.box(b)) * bt.coef_r + s.dv.box(a);
  const int lane = threadIdx.x;
  const int64_t off = (int64_t)pair * 3 * s.g.B;
  const uint32_t* __restrict__ tab = s.tab + kSmallEdges + 5 * min(lane, 53);
  const uint32_t tx = tab[0], c0 = tab[1], c1 = tab[2], c2 = tab[3], c3 = tab[4];
  // interior rows: lane 8 t + p takes columns 6 p .. 6 p + 5 of row t of X_T, and column p
  // of A_T^{-1}
  const int t = min(lane >> 3, 5), p = lane & 7;
  T xr[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) xr[i] = s.XT[(int64_t)prob * NX + t * 48 + 6 * p + i];
  const T ai = s.ATinv[(int64_t)prob * 36 + 6 * t + min(p, 5)];
  T ri;
  {
    const int q = min(p, 5), d = q >> 1, f = q & 1;
    ri = r[off + d * s.g.B + lin(s.g, 2 * a + (d == 0 ? f : 1), 2 * b + (d == 1 ? f : 1), 2 * c + (d == 2 ? f : 1))];
  }
  const int d = tx & 3, ox = (tx >> 2) & 3, oy = (tx >> 4) & 3, oz = (tx >> 6) & 3;
  const bool mine = (tx >> 8) & 1;
  const int64_t at = off + d * s.g.B + lin(s.g, 2 * a + ox, 2 * b + oy, 2 * c + oz);
  const T zo = assign ? T(0) : z[at];
  T pe[4] = {T(0), T(0), T(0), T(0)};
  const int ob = (d == 0 ? oy : (d == 1 ? oz : ox)) & 1, oc = (d == 0 ? oz : (d == 1 ? ox : oy)) & 1;
  if (zc) {
    const int64_t st[3] = {1, (int64_t)gc.P, gc.plane};
    const int64_t sb = ob ? (d == 0 ? st[1] : (d == 1 ? st[2] : st[0])) : 0;
    const int64_t sc = oc ? (d == 0 ? st[2] : (d == 1 ? st[0] : st[1])) : 0;
    const T* e = zc + (int64_t)pair * 3 * gc.B + d * gc.B + lin(gc, a + (ox >> 1), b + (oy >> 1), c + (oz >> 1));
    pe[0] = e[0];
    pe[1] = e[sb];
    pe[2] = e[sc];
    pe[3] = e[sb + sc];
  }
  const T* __restrict__ Yp = s.Y + (int64_t)pair * nv3 * NPAD;
  auto patch = [&](unsigned code) {
    const bool on = code != 0xffff;
    const int q = code & 7, slot = on ? (int)(code >> 3) : 0;
    const int x = a + (q & 1), y = b + ((q >> 1) & 1), w = c + (q >> 2);
    const T val = Yp[((w * nv + y) * nv + x) * NPAD + slot];
    return on ? val : T(0);
  };
  const T y0 = patch(c0), y1 = patch(c1), y2 = patch(c2), y3 = patch(c3);
  issue_barrier();
  if (act == 0) return;
  const T w = ((y0 + y1) + y2) + y3;
  if (lane < 48) wL[lane] = w;
  __syncthreads();
  T sum = p < 6 ? ai * ri : T(0);
#pragma unroll
  for (int i = 0; i < 6; ++i) sum -= xr[i] * wL[6 * p + i];
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) sum += __shfl_xor(sum, m, 64);
  const T zi = __shfl(sum, 8 * max(min(lane - 48, 5), 0), 64);
  const T wb0 = ob ? T(0.5) : T(1), wb1 = ob ? T(0.5) : T(0), wc0 = oc ? T(0.5) : T(1), wc1 = oc ? T(0.5) : T(0);
  const T pro = wc0 * (wb0 * pe[0] + wb1 * pe[1]) + wc1 * (wb0 * pe[2] + wb1 * pe[3]);
  if (mine && lane < 54) z[at] = (zo + pro) + (T)s.eta * (lane < 48 ? w : zi);
}

// Lane: direction, offset 0 / 1 along it, -1 .. 1 across, of the 54 fine edges that the three
// coarse edges of node V restrict.  (A wave per direction, with constant strides, measured
// slower: 8.6 against 5.7 us at 32^3 in FP64, 4.4 against 3.9 at 16^3.)
template <typename T, bool COEF>
__global__ void __launch_bounds__(64) k_small_restrict(const T* __restrict__ g, const T* __restrict__ z,
                                                       T* __restrict__ out, DGeom f, double h, DGeom c, BoxDiv dv,
                                                       Bat bt) {
  using S = CubeShape<5>;
  constexpr int NL = (3 * S::N + 63) / 64;
  __shared__ T zL[3 * S::N];
  __shared__ T rL[54];
  __shared__ T fL[COEF ? 64 : 1];
  const int nc = c.n, nc3 = nc * nc * nc;
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int pair = lb / nc3, v = lb - pair * nc3;
  const int vx = v % nc, vy = (v / nc) % nc, vz = v / (nc * nc);
  const int act = bt.act ? bt.act[pair] : 1;
  const T ah = (T)(bt.alpha[pair / bt.nrhs] * h), h3 = (T)(h * h * h);
  const int lane = threadIdx.x;
  const int64_t off = (int64_t)pair * 3 * f.B;
  const Cube q{2 * vx - 2, 2 * vy - 2, 2 * vz - 2, f.n};
  T zv[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int m = min(lane + 64 * i, 3 * S::N - 1), d = m / S::N;
    zv[i] = load_cube<5>(z + off, f, q, d, m - d * S::N);
  }
  const int l = min(lane, 53), d = l / 18, e18 = l - 18 * d;
  const Pos e = edge_pos(d, 2 + (e18 & 1), 1 + (e18 >> 1) % 3, 1 + e18 / 6);
  const bool on = q.unknown(d, e.x, e.y, e.z);
  const T gv = g[off + (on ? d * f.B + lin(f, q.x0 + e.x, q.y0 + e.y, q.z0 + e.z) : 0)];
  double fv = 0.0;
  if constexpr (COEF) fv = load_cell<5>(bt, q, dv, lane);
  issue_barrier();
  if (act == 0) return;
  if constexpr (COEF) fL[lane] = (T)fv;
#pragma unroll
  for (int i = 0; i < NL; ++i)
    if (lane + 64 * i < 3 * S::N) zL[lane + 64 * i] = zv[i];
  __syncthreads();
  T c00 = T(1), c10 = T(1), c01 = T(1), c11 = T(1);
  if constexpr (COEF) edge_cells<5>(fL, d, e, c00, c10, c01, c11);
  const int sa = d == 0 ? 1 : (d == 1 ? 5 : 25), sb = d == 0 ? 5 : (d == 1 ? 25 : 1), sc = d == 0 ? 25 : (d == 1 ? 1 : 5);
  const T* zp = zL + S::at(e.x, e.y, e.z);
  const T ax = apply_lds<COEF>(zp + d * S::N, zp + (d == 2 ? 0 : d + 1) * S::N, zp + (d == 0 ? 2 : d - 1) * S::N, sa, sb,
                               sc, ah, h3, c00, c10, c01, c11);
  const bool in = on && c00 > T(0) && c10 > T(0) && c01 > T(0) && c11 > T(0);
  if (lane < 54) rL[lane] = in ? gv - ax : T(0);
  __syncthreads();
  if (lane < 3) {
    const T* s = rL + 18 * lane;
    T acc = T(0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {   // the two fine edges along the coarse one
      const T mid = T(0.5) * (s[k + 2] + s[k + 14]) + s[k + 8];
      const T lo = T(0.5) * (s[k] + s[k + 12]) + s[k + 6];
      const T hi = T(0.5) * (s[k + 4] + s[k + 16]) + s[k + 10];
      acc += T(0.5) * (lo + hi) + mid;
    }
    bool cin = vx >= (lane != 0) && vy >= (lane != 1) && vz >= (lane != 2);
    if constexpr (COEF) {   // the coarse edge's cells are those around its first fine edge
      edge_cells<5>(fL, lane, Pos{2, 2, 2}, c00, c10, c01, c11);
      cin = cin && c00 > T(0) && c10 > T(0) && c01 > T(0) && c11 > T(0);
    }
    out[(int64_t)pair * 3 * c.B + lane * c.B + lin(c, vx, vy, vz)] = cin ? acc : T(0);
  }
}

}  // namespace

namespace {

std::vector<uint32_t> make_tables() {
  std::vector<uint32_t> t(kSmallWords, 0);
  auto set = [&](int at, uint32_t x, const std::vector<uint32_t>& codes) {
    t[at] = x;
    for (size_t i = 0; i < 4; ++i) t[at + 1 + i] = i < codes.size() ? codes[i] : 0xffff;
  };
  const std::vector<Slot> bd = boundary_dofs(2), in = interior_dofs(2), sl = vertex_slots(2);
  const std::vector<int> bp = boundary_patch_table();
  auto word = [](const Slot& q, bool own) {
    return (uint32_t)(q.d | q.dx << 2 | q.dy << 4 | q.dz << 6 | (own ? 1 : 0) << 8);
  };
  for (size_t e = 0; e < bd.size(); ++e) {
    std::vector<uint32_t> codes;
    for (int k = 0; k < 4; ++k) {
      const int code = bp[4 * e + k];
      if (code >= 0) codes.push_back((uint32_t)(code & ~(1 << 30)));
    }
    set(kSmallEdges + 5 * (int)e, word(bd[e], bd[e].dx <= 1 && bd[e].dy <= 1 && bd[e].dz <= 1), codes);
  }
  for (size_t i = 0; i < in.size(); ++i) set(kSmallEdges + 5 * (48 + (int)i), word(in[i], true), {});
  for (size_t i = 0; i < sl.size(); ++i) {
    const int o[3] = {2 + sl[i].dx, 2 + sl[i].dy, 2 + sl[i].dz};
    std::vector<uint32_t> codes;
    for (int q = 0; q < 8; ++q)
      for (size_t e = 0; e < bd.size(); ++e)
        if (bd[e].d == sl[i].d && 2 * (q & 1) + bd[e].dx == o[0] && 2 * ((q >> 1) & 1) + bd[e].dy == o[1] &&
            2 * (q >> 2) + bd[e].dz == o[2])
          codes.push_back((uint32_t)(q | (int)e << 3));
    set(kSmallSlots + 5 * (int)i, (uint32_t)(sl[i].d | o[0] << 2 | o[1] << 5 | o[2] << 8), codes);
  }
  return t;
}

}  // namespace

const std::vector<uint32_t>& small_tables() {
  static const std::vector<uint32_t> t = make_tables();
  return t;
}

// Measured on MI355X (us per CG iteration of one problem, large-level kernels / these, the
// levels below on these): 16^3 FP32 79 / 56, FP64 85 / 56; 24^3 97 / 78, 104 / 83; 32^3 105 /
// 94, 119 / 107 (Fichera domain 117 / 101, 133 / 118); 40^3 135 / 134, 157 / 162; 48^3 146 /
// 164.  The work grows with the vertices of all pairs, each reading its S^{-1} and repeating
// its neighbours' residuals, while the large-level kernels' time below 32^3 is their round
// trips; the two cross between 17^3 and 21^3 vertices.
bool small_level(int nH, int count) {
  const int64_t nv = nH + 1;
  return nv * nv * nv * count <= 6000;
}

// Two vertices per block where the blocks outnumber the compute units: they share S^{-1}, whose
// loads bound the launch from 24^3 on (32^3 FP64 107 against 116 us per iteration, 20^3 86 /
// 88, equal at 16^3); with fewer vertices one per block (10^3 63 against 64).
static bool small_pairs(int nH, int count) {
  const int64_t nv = nH + 1;
  return nv * nv * nv * count > 500;
}

template <typename T>
hipError_t launch_small_patch(int mode, const T* g, const T* z, const T* zc, const SmallSub<T>& s, const DGeom& gc,
                              const Bat& bt, hipStream_t st) {
  const int nv = s.nH + 1;
  const bool two = small_pairs(s.nH, bt.count);
  const dim3 grid((unsigned)((two ? nv / 2 + 1 : nv) * nv * nv * bt.count));
  auto launch = [&](auto coef, auto pairs) {
    constexpr bool C = decltype(coef)::value;
    constexpr int NV = decltype(pairs)::value ? 2 : 1;
    if (mode == 0)
      hipLaunchKernelGGL((k_small_patch<T, 0, C, NV>), grid, dim3(256), 0, st, g, z, zc, s, gc, bt);
    else if (mode == 1)
      hipLaunchKernelGGL((k_small_patch<T, 1, C, NV>), grid, dim3(256), 0, st, g, z, zc, s, gc, bt);
    else
      hipLaunchKernelGGL((k_small_patch<T, 2, C, NV>), grid, dim3(256), 0, st, g, z, zc, s, gc, bt);
  };
  auto with_coef = [&](auto pairs) {
    if (bt.coef)
      launch(std::true_type{}, pairs);
    else
      launch(std::false_type{}, pairs);
  };
  if (two)
    with_coef(std::true_type{});
  else
    with_coef(std::false_type{});
  return hipGetLastError();
}

template <typename T>
hipError_t launch_small_pull(const T* r, T* z, const T* zc, int assign, const SmallSub<T>& s, const DGeom& gc,
                             const Bat& bt, hipStream_t st) {
  hipLaunchKernelGGL((k_small_pull<T>), dim3((unsigned)(s.nH * s.nH * s.nH * bt.count)), dim3(64), 0, st, r, z, zc,
                     assign, s, gc, bt);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_small_restrict(const T* g, const T* z, T* out, const DGeom& f, double h, const DGeom& c,
                                 const Bat& bt, hipStream_t st) {
  const dim3 grid((unsigned)(c.n * c.n * c.n * bt.count));
  const BoxDiv dv = bt.coef ? BoxDiv(c.n / bt.coef_r) : BoxDiv();
  if (bt.coef)
    hipLaunchKernelGGL((k_small_restrict<T, true>), grid, dim3(64), 0, st, g, z, out, f, h, c, dv, bt);
  else
    hipLaunchKernelGGL((k_small_restrict<T, false>), grid, dim3(64), 0, st, g, z, out, f, h, c, dv, bt);
  return hipGetLastError();
}

#define NDMG_SMALL(T)                                                                                            \
  template hipError_t launch_small_patch<T>(int, const T*, const T*, const T*, const SmallSub<T>&, const DGeom&, \
                                            const Bat&, hipStream_t);                                            \
  template hipError_t launch_small_pull<T>(const T*, T*, const T*, int, const SmallSub<T>&, const DGeom&,        \
                                           const Bat&, hipStream_t);                                             \
  template hipError_t launch_small_restrict<T>(const T*, const T*, T*, const DGeom&, double, const DGeom&,       \
                                               const Bat&, hipStream_t);
NDMG_SMALL(double)
NDMG_SMALL(float)

}  // namespace ndmg
