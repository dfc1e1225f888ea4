// train_device.hpp -- device helpers shared by the training kernels, templated on
// the arithmetic.
#pragma once

#include "train.hpp"

namespace nepmi {

// Symmetric 3x3 as (xx, yy, zz, xy, xz, yz); full-matrix gradient convention
// dE = sum_ab M_ab dA_ab.  A_n from S_n2m (l = 2 content of S).
template <class R>
__device__ __forceinline__ void sym_from_s2(const R* s2, R (&A)[6]) {
  const R azz = s2[0] * (R(1.0) / (R(3.0) * ShC<R>::k20));
  const R dif = s2[3] * (R(1.0) / ShC<R>::k22);
  A[0] = R(0.5) * (dif - azz);
  A[1] = -R(0.5) * (dif + azz);
  A[2] = azz;
  A[3] = s2[4] * (R(1.0) / ShC<R>::k21);
  A[4] = s2[1] * (R(1.0) / ShC<R>::k21);
  A[5] = s2[2] * (R(1.0) / ShC<R>::k21);
}

template <class R>
__device__ __forceinline__ void sym_mul_sym(const R (&A)[6], const R (&B)[6], R (&C)[9]) {
  // C = A B (general 3x3, row-major)
  const R a[9] = {A[0], A[3], A[4], A[3], A[1], A[5], A[4], A[5], A[2]};
  const R b[9] = {B[0], B[3], B[4], B[3], B[1], B[5], B[4], B[5], B[2]};
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) C[3 * i + j] = a[3 * i] * b[j] + a[3 * i + 1] * b[3 + j] + a[3 * i + 2] * b[6 + j];
}

// sum_ab M_ab N_ab for symmetric M, N
template <class R>
__device__ __forceinline__ R sym_dot(const R (&M)[6], const R (&N)[6]) {
  return M[0] * N[0] + M[1] * N[1] + M[2] * N[2] + R(2.0) * (M[3] * N[3] + M[4] * N[4] + M[5] * N[5]);
}

// Gradient with respect to S_n2m of a function whose gradient w.r.t. A is M.
template <class R>
__device__ __forceinline__ void chain_s2(const R (&M)[6], R (&g)[5]) {
  g[0] = (M[2] - R(0.5) * (M[0] + M[1])) * (R(1.0) / (R(3.0) * ShC<R>::k20));
  g[1] = R(2.0) * M[4] * (R(1.0) / ShC<R>::k21);
  g[2] = R(2.0) * M[5] * (R(1.0) / ShC<R>::k21);
  g[3] = R(0.5) * (M[0] - M[1]) * (R(1.0) / ShC<R>::k22);
  g[4] = R(2.0) * M[3] * (R(1.0) / ShC<R>::k21);
}

template <class R>
__device__ __forceinline__ void sym_sq6(const R (&A)[6], R (&B)[6]) {
  const R xx = A[0], yy = A[1], zz = A[2], xy = A[3], xz = A[4], yz = A[5];
  B[0] = xx * xx + xy * xy + xz * xz;
  B[1] = xy * xy + yy * yy + yz * yz;
  B[2] = xz * xz + yz * yz + zz * zz;
  B[3] = xx * xy + xy * yy + xz * yz;
  B[4] = xx * xz + xy * yz + xz * zz;
  B[5] = xy * xz + yy * yz + yz * zz;
}

template <class R>
__device__ __forceinline__ void load_cell9(const CfgDev* __restrict__ cfgs, int c, R (&H)[9]) {
#pragma unroll
  for (int x = 0; x < 9; ++x) H[x] = c >= 0 ? cell_rows(cfgs[c], R())[x] : R(0);
}

template <class R>
struct PV {
  R rx, ry, rz, d2;
  int q, zj;
};

// Pair vector of list entry e whose neighbour position xq is already loaded.
template <class R>
__device__ __forceinline__ PV<R> pvec_at(uint32_t e, Vec4<R> xq, Vec4<R> xi, const R (&H)[9]) {
  PV<R> v;
  v.q = (int)(e & kNbrMask);
  R sx, sy, sz;
  image_shift(H, e >> kNbrShift, sx, sy, sz);
  v.rx = (xq.x - xi.x) + sx;
  v.ry = (xq.y - xi.y) + sy;
  v.rz = (xq.z - xi.z) + sz;
  v.d2 = pair_d2(v.rx, v.ry, v.rz);
  v.zj = species_of(xq);
  return v;
}

template <class R>
__device__ __forceinline__ PV<R> pvec(const Vec4<R>* __restrict__ pos4, uint32_t e, Vec4<R> xi, const R (&H)[9]) {
  return pvec_at(e, pos4[e & kNbrMask], xi, H);
}

}  // namespace nepmi
