// The operator at one edge from entries in LDS, shared by the small-level and small-CG kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace ndmg {

// (A u)_e at an edge of direction a: ua, ub, uc its entry and those of the next two
// directions at its first node in LDS, sa, sb, sc the strides along and across it.  The
// factorised form alpha h C^T M_F C + h^3 M_E, the 33 entries read once; COEF: c_{db dc} the
// factors of the cells at -1 + db, -1 + dc across.
template <bool COEF, typename T>
__device__ __forceinline__ T apply_lds(const T* ua, const T* ub, const T* uc, int sa, int sb, int sc, T ah, T h3, T c00,
                                       T c10, T c01, T c11) {
  const T t6 = T(1) / T(6), t23 = T(2) / T(3), t3 = T(1) / T(3);
  T A[3][3], Ub[2][3][2], Uc[2][3][2];   // offsets [b][c]; [b: -1, 0][c][a]; [c: -1, 0][b][a]
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) A[i][j] = ua[(i - 1) * sb + (j - 1) * sc];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        Ub[i][j][e] = ub[(i - 1) * sb + (j - 1) * sc + e * sa];
        Uc[i][j][e] = uc[(i - 1) * sc + (j - 1) * sb + e * sa];
      }
  // faces of normal b at (c offset i - 1, b offset j - 1), and of normal c likewise
  T Fb[2][3], Fc[2][3];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Fb[i][j] = (A[j][i + 1] - A[j][i]) - (Uc[i][j][1] - Uc[i][j][0]);
      Fc[i][j] = (Ub[i][j][1] - Ub[i][j][0]) - (A[i + 1][j] - A[i][j]);
    }
  // a face between the cells of factors m (below along its normal) and p
  const T bm[2] = {c00, c01}, bp[2] = {c10, c11}, cm[2] = {c00, c10}, cp[2] = {c01, c11};
  T Gb[2], Gc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (COEF) {
      Gb[i] = t6 * (bm[i] * Fb[i][0] + bp[i] * Fb[i][2]) + t3 * (bm[i] + bp[i]) * Fb[i][1];
      Gc[i] = t6 * (cm[i] * Fc[i][0] + cp[i] * Fc[i][2]) + t3 * (cm[i] + cp[i]) * Fc[i][1];
    } else {
      Gb[i] = t6 * (Fb[i][0] + Fb[i][2]) + t23 * Fb[i][1];
      Gc[i] = t6 * (Fc[i][0] + Fc[i][2]) + t23 * Fc[i][1];
    }
  }
  const T curl = (Gb[0] - Gb[1]) - (Gc[0] - Gc[1]);
  T row[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) row[i] = t6 * (A[i][0] + A[i][2]) + t23 * A[i][1];
  const T mass = t6 * (row[0] + row[2]) + t23 * row[1];
  return ah * curl + h3 * mass;
}
}  // namespace ndmg
