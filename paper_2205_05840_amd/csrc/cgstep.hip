// The vector work of one CG iteration of a small problem (n <= 12) as one block per pair.
//
// At 8^3 an iteration ran six launches besides the V-cycle (dot products, direction, operator,
// dot product, update, convergence test), 3 to 4 us each for vectors of 31 KB: latency only.
// Here one block of 1024 lanes keeps p in LDS, so the operator and the three reductions need
// block barriers instead of launches.  Lanes take unknowns, not entries of the padded vector
// (30 % of it at 8^3).  Bound by latency and by one compute unit's LDS: one round trip for the
// vectors, three block reductions, 2 (8^3) to 5 (12^3) edges of 33 LDS reads per lane.  Measured
// at 8^3: 8.0 us per iteration (six launches 21); whole solves (us, before / after) 8^3 FP64
// 985 / 508, 10^3 1344 / 1062, 12^3 1350 / 1220.  14^3 would need 7 edges per lane: launches.
#include <hip/hip_runtime.h>

#include "apply_lds.hpp"
#include "cgstep.hpp"

namespace ndmg {

namespace {

// e / x by a multiplication, exact for e x < 2^32 (m = ceil(2^32 / x); 0 stands for x = 1)
struct Div {
  unsigned m;
  __device__ __forceinline__ unsigned div(unsigned e) const { return m ? __umulhi(e, m) : e; }
};

// sums over the block of two values, to every lane, in a fixed order (sh: 16 pairs)
__device__ __forceinline__ void block_sum2(double& a, double& b, double2* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_double2(a, b);
  __syncthreads();
  a = b = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    a += sh[w].x;
    b += sh[w].y;
  }
}

// Unknown t of the level (direction-major, then x fastest) as its direction, its node's offset
// and its place in the padded vector.
struct Unknowns {
  int n, per;        // per: n (n - 1)^2, the unknowns of one direction
  Div n0, n1;        // by n and by n - 1
  int P, plane, B;
  __device__ __forceinline__ int node(int t, int& d) const {
    d = (t >= per) + (t >= 2 * per);
    const int q = t - d * per;
    const int row = (int)(d == 0 ? n0 : n1).div(q), i = q - row * (d == 0 ? n : n - 1);
    const int k = (int)(d == 1 ? n0 : n1).div(row), j = row - k * (d == 1 ? n : n - 1);
    return (k + (d != 2)) * plane + (j + (d != 1)) * P + i + (d != 0);
  }
};

// NE unknowns per lane: t = lane + 1024 i of the N
template <typename TZ, int NE>
__global__ void __launch_bounds__(1024) k_cg_step(const TZ* __restrict__ z, CgStep s, Unknowns un, double h, int count,
                                                  Bat bt) {
  extern __shared__ __attribute__((aligned(16))) unsigned char step_smem[];
  const int N = 3 * un.per, len = 3 * un.B;
  double* pL = reinterpret_cast<double*>(step_smem);   // p, padded (zeros off the unknowns)
  double* qL = pL + len;                                // A p, by unknown
  __shared__ double2 sh[3][16];
  const int pair = blockIdx.x, tid = threadIdx.x;
  const int act = s.act[pair];
  const int64_t off = (int64_t)pair * len;
  z += off;
  double* __restrict__ r = s.r + off;
  double* __restrict__ p = s.p + off;
  double* __restrict__ q = s.q + off;
  double* __restrict__ u = s.u + off;
  double* sc = s.scal + (int64_t)pair * kScalStride;
  const double ah = bt.alpha[pair / bt.nrhs] * h, h3 = h * h * h;
  int at[NE];
  double rz = 0.0, zq = 0.0, rv[NE], pv[NE], zv[NE], uv[NE];
  {
    double qv[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      int d;
      const int node = un.node(min(tid + 1024 * i, N - 1), d);
      at[i] = node + d * un.B;
      zv[i] = (double)z[at[i]];
      rv[i] = r[at[i]];
      pv[i] = p[at[i]];
      qv[i] = q[at[i]];
      uv[i] = u[at[i]];
    }
    __asm__ volatile("" ::: "memory");   // (the loads stay above the test)
    if (act == 0) {
      if (count == 1 && tid == 0) s.nact[0] = 0;
      return;
    }
    for (int e = tid; e < len; e += 1024) pL[e] = 0.0;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const bool in = tid + 1024 * i < N;
      rz += in ? zv[i] * rv[i] : 0.0;
      zq += in ? zv[i] * qv[i] : 0.0;
    }
  }
  block_sum2(rz, zq, sh[0]);
  if (s.first) {
#pragma unroll
    for (int i = 0; i < NE; ++i) pv[i] = zv[i];
  } else {
    const double beta = s.flexible ? -(sc[s.i_an] / sc[kS_PQ]) * zq / sc[s.i_den] : rz / sc[s.i_den];
    const double al = sc[kS_AL];   // the pending update's (an active pair always has one here)
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      if (tid + 1024 * i < N) u[at[i]] = uv[i] + al * pv[i];
      pv[i] = zv[i] + beta * pv[i];
    }
  }
#pragma unroll
  for (int i = 0; i < NE; ++i)
    if (tid + 1024 * i < N) {
      p[at[i]] = pv[i];
      pL[at[i]] = pv[i];
    }
  __syncthreads();   // (and every lane has read the scalars that lane 0 replaces below)
  // (one edge at a time: its 33 entries fill the registers)
  double pq = 0.0;
#pragma unroll 1
  for (int t = tid; t < N; t += 1024) {
    int d;
    const double* base = pL + un.node(t, d);
    const int sa = d == 0 ? 1 : (d == 1 ? un.P : un.plane), sb = d == 0 ? un.P : (d == 1 ? un.plane : 1),
              scs = d == 0 ? un.plane : (d == 1 ? 1 : un.P);
    const double* ua = base + d * un.B;
    const double ax = apply_lds<false>(ua, base + (d == 2 ? 0 : d + 1) * un.B, base + (d == 0 ? 2 : d - 1) * un.B, sa, sb,
                                       scs, ah, h3, 1.0, 1.0, 1.0, 1.0);
    qL[t] = ax;
    pq += ax * ua[0];
  }
  double none = 0.0;
  block_sum2(pq, none, sh[1]);
  const double alpha = rz / pq;
  double rr = 0.0;
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int t = tid + 1024 * i;
    if (t < N) {
      const double qe = qL[t], v = rv[i] - alpha * qe;
      rr += v * v;
      r[at[i]] = v;
      q[at[i]] = qe;
      if (s.r32) s.r32[off + at[i]] = (float)v;
    }
  }
  none = 0.0;
  block_sum2(rr, none, sh[2]);
  if (tid != 0) return;
  sc[s.i_num] = rz;
  if (s.flexible && !s.first) sc[s.i_zq] = zq;
  sc[kS_PQ] = pq;
  sc[kS_AL] = alpha;
  sc[kS_PEND] = 1.0;
  if (count > 1) {
    s.rr_part[(int64_t)pair * s.pstride] = rr;
    return;
  }
  // the convergence test, as launch_pcg_check has it
  sc[kS_RR] = rr;
  const int it = s.iters[0];
  if (it < kHistCap) {
    s.hist[2 * it] = rz;
    s.hist[2 * it + 1] = pq;
  }
  s.iters[0] = it + 1;
  const double rel = sqrt(rr) / sqrt(sc[kS_BB]);
  sc[kS_REL] = rel;
  int active = 0;
  if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rr) || !isfinite(rz)) {
    s.act[0] = 0;
    s.status[0] = kPairBroken;
  } else if (rel <= sc[kS_TOL]) {
    s.act[0] = 0;
    s.status[0] = kPairDone;
  } else {
    active = 1;
  }
  s.nact[0] = active;
}

Div make_div(int x) { return Div{x > 1 ? (unsigned)(((uint64_t(1) << 32) + x - 1) / x) : 0}; }

}  // namespace

template <typename TZ>
hipError_t launch_cg_step(const TZ* z, const CgStep& s, const Geom& g, const Bat& bt, hipStream_t st) {
  if (g.n < 2 || g.n > kCgStepMaxN || bt.coef) return hipErrorInvalidValue;
  const int n = g.n, per = n * (n - 1) * (n - 1);
  const Unknowns un{n, per, make_div(n), make_div(n - 1), g.P, (int)g.plane, (int)g.B};
  const size_t lds = ((size_t)g.len + 3 * per) * sizeof(double);
  const dim3 grid((unsigned)bt.count);
  if (3 * per <= 2048)
    hipLaunchKernelGGL((k_cg_step<TZ, 2>), grid, dim3(1024), lds, st, z, s, un, g.h, bt.count, bt);
  else if (3 * per <= 3072)
    hipLaunchKernelGGL((k_cg_step<TZ, 3>), grid, dim3(1024), lds, st, z, s, un, g.h, bt.count, bt);
  else
    hipLaunchKernelGGL((k_cg_step<TZ, 5>), grid, dim3(1024), lds, st, z, s, un, g.h, bt.count, bt);
  return hipGetLastError();
}

template hipError_t launch_cg_step<double>(const double*, const CgStep&, const Geom&, const Bat&, hipStream_t);
template hipError_t launch_cg_step<float>(const float*, const CgStep&, const Geom&, const Bat&, hipStream_t);

}  // namespace ndmg
