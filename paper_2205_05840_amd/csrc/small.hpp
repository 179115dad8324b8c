// The vertex smoother (subdomains of 2^3 elements) and the transfers of a small level, one
// block or wavefront per vertex, subdomain or coarse node: three launches down and two up.
#pragma once

#include <cstdint>

#include "kernels.hpp"

namespace ndmg {

// Box of a subdomain along an axis, u / w by a multiplication (exact for u w < 2^16).
struct BoxDiv {
  int w = 1, m = 65536;
  BoxDiv() = default;
  explicit BoxDiv(int w_) : w(w_), m((65536 + w_ - 1) / w_) {}
  __host__ __device__ int box(int u) const { return (u * m) >> 16; }
};

// One smoothed level as the small-level kernels take it.  Factors of problem p follow each
// other (36, 288 and sstride elements per problem); with coefficient boxes (one problem)
// A_T^{-1} and X_T hold a block per box, zero outside the domain.  Y: the patch results by vertex,
// [(nH+1)^3][64] per pair.
template <typename T>
struct SmallSub {
  DGeom g;
  double h;
  int nH;
  const uint32_t* tab;  // small_tables()
  const int* cls;       // class triples of the vertices (BoxPatches), with coefficient boxes
  const T* ATinv;
  const T* XT;
  const T* Sinv;
  int64_t sstride;
  T* Y;
  T* r;                 // interior residuals of the subdomains (modes with a residual)
  double eta;
  BoxDiv dv;            // with coefficient boxes
};

// Packed tables of the 2 x 2 x 2 subdomain, built from the host's slot rules, five words per
// entry.  kSmallEdges: the 48 boundary edges of a subdomain, then its 6 interior unknowns:
// direction | offsets << 2, 4, 6 | 1 << 8 where the subdomain writes the unknown, then the
// patch results it sums (corner | slot << 3, 0xffff none).  kSmallSlots: the 60 slots of a
// vertex patch: direction | node in the patch's cube << 2, 5, 8 (x, y, z; the vertex at 2, 2,
// 2), then the subdomains of the patch whose boundary holds the edge (subdomain | boundary
// edge << 3).
constexpr int kSmallEdges = 0, kSmallSlots = 5 * 54, kSmallWords = 5 * 114;
const std::vector<uint32_t>& small_tables();   // built once

// Whether the V-cycle steps of a level of nH subdomains per axis take these kernels when
// `count` pairs are in flight.
bool small_level(int nH, int count);

// Patch products Y of the condensed residual of r = g (mode 0), r = g - A z (mode 1) or
// r = g - A (z + I zc) (mode 2, zc on the coarser level); modes 1 and 2 also write r on the
// subdomain interiors.
template <typename T>
hipError_t launch_small_patch(int mode, const T* g, const T* z, const T* zc, const SmallSub<T>& s, const DGeom& gc,
                              const Bat& bt, hipStream_t st);
// z (assign: =, else +=) M^{-1} r from the patch results and r on the interiors; with zc
// z += I zc as well.
template <typename T>
hipError_t launch_small_pull(const T* r, T* z, const T* zc, int assign, const SmallSub<T>& s, const DGeom& gc,
                             const Bat& bt, hipStream_t st);
// gc = I^T (g - A z)
template <typename T>
hipError_t launch_small_restrict(const T* g, const T* z, T* out, const DGeom& f, double h, const DGeom& c,
                                 const Bat& bt, hipStream_t st);

}  // namespace ndmg
