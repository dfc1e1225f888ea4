// nep_device.hpp -- device helpers shared by the evaluation kernels that give one
// thread to an atom (nep_kernels.hip) and those that give it a wavefront
// (nep_wave.hip): both forms compute every value with the same operations in
// the same order.
#pragma once

#include "nep_kernels.hpp"

namespace nepmi {

// Pair vector r_ij = (x_j - x_i) + image shift, computed with the same
// rounding from either side so that r_ji = -r_ij exactly.
struct PairVec {
  float rx, ry, rz, d2;
  int q, zj;
};

// Lattice-vector multiples (w0, w1, w2) of the 27 image codes (see
// image_shift), in LDS: one read per pair instead of the integer decode.
struct ImageTable {
  float4 w[32];
  __device__ void fill() {
    if (threadIdx.x < 27) {
      const int c = threadIdx.x;
      w[c] = make_float4((float)(c / 9 - 1), (float)((c / 3) % 3 - 1), (float)(c % 3 - 1), 0.f);
    }
  }
};

__device__ __forceinline__ PairVec pair_vec(uint32_t e, float4 xq, float4 xi, const float (&H)[9],
                                            const ImageTable& it) {
  PairVec v;
  v.q = (int)(e & kNbrMask);
  // the same expression as image_shift, so the shift of code 26 - c is again
  // exactly the negative of the shift of c
  const float4 w = it.w[e >> kNbrShift];
  const float sx = w.x * H[0] + w.y * H[3] + w.z * H[6];
  const float sy = w.x * H[1] + w.y * H[4] + w.z * H[7];
  const float sz = w.x * H[2] + w.y * H[5] + w.z * H[8];
  v.rx = (xq.x - xi.x) + sx;
  v.ry = (xq.y - xi.y) + sy;
  v.rz = (xq.z - xi.z) + sz;
  v.d2 = pair_d2(v.rx, v.ry, v.rz);
  v.zj = __float_as_int(xq.w);
  return v;
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Groups of four list entries fill by shifting entries in from the top
// (register moves, no selects), so a full group holds them in order; a
// partly filled one holds its r entries in the top r components, which
// front4 moves to the front (the rest repeat the last entry, a real one).
__device__ __forceinline__ void shift_in4(uint4& v, uint32_t e) { v = make_uint4(v.y, v.z, v.w, e); }
__device__ __forceinline__ uint4 front4(uint4 g, int r) {
  return r == 1 ? make_uint4(g.w, g.w, g.w, g.w) : r == 2 ? make_uint4(g.z, g.w, g.w, g.w)
                                                           : make_uint4(g.y, g.z, g.w, g.w);
}

// One neighbour's radial adjoint row (B_R floats).
template <int BR>
struct AdjRow {
  float4 v[BR / 4];
};

// Network dimensions padded to the 4-wide groups of the matrix instructions.
template <class S>
struct MlpPad {
  static constexpr int HP = (S::H + 3) / 4 * 4;
  static constexpr int DP = (S::D + 3) / 4 * 4;
};

// tanh(x) = 1 - 2 / (1 + e^{2x}) with the hardware exp2 and reciprocal
// (absolute error a few 1e-7; saturates to +-1 for large |x|).
__device__ __forceinline__ float tanh_fast(float x) {
  const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);  // 2 log2(e)
  return fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + e), 1.0f);
}


__device__ __forceinline__ void load_cell(const CfgDev* __restrict__ cfgs, int c, float (&H)[9]) {
  if (c >= 0) {
#pragma unroll
    for (int x = 0; x < 9; ++x) H[x] = cfgs[c].H[x];
  } else {
#pragma unroll
    for (int x = 0; x < 9; ++x) H[x] = 0.f;
  }
}

// The operations below are written out as fused multiply-adds: left to the
// compiler, which product of a sum gets fused depends on the code around the
// call, and the two forms of a kernel would differ in the last bit.

// S_n2m -> symmetric traceless A_n = sum_j g_n (u u^T - I/3) (l = 2 content).
// Returns A as (xx, yy, zz, xy, xz, yz).
__device__ __forceinline__ void a_from_s2(const float* s2, float (&A)[6]) {
  const float azz = s2[0] * (1.0f / (3.0f * sh::k20));
  A[0] = 0.5f * fmaf(s2[3], 1.0f / sh::k22, -azz);
  A[1] = -0.5f * fmaf(s2[3], 1.0f / sh::k22, azz);
  A[2] = azz;
  A[3] = s2[4] * (1.0f / sh::k21);
  A[4] = s2[1] * (1.0f / sh::k21);
  A[5] = s2[2] * (1.0f / sh::k21);
}

// A^2 as (xx, yy, zz, xy, xz, yz)
__device__ __forceinline__ void sym_sq(const float (&A)[6], float (&B)[6]) {
  const float xx = A[0], yy = A[1], zz = A[2], xy = A[3], xz = A[4], yz = A[5];
  B[0] = fmaf(xz, xz, fmaf(xx, xx, xy * xy));
  B[1] = fmaf(yz, yz, fmaf(yy, yy, xy * xy));
  B[2] = fmaf(zz, zz, fmaf(xz, xz, yz * yz));
  B[3] = fmaf(xz, yz, fmaf(xy, xx, xy * yy));
  B[4] = fmaf(xz, zz, fmaf(xx, xz, xy * yz));
  B[5] = fmaf(yz, zz, fmaf(xy, xz, yy * yz));
}

// f4 A^2 (B = A^2) contracted with dA/dS_2m is s4_scale(m) s4[m], m = 0..4.
__device__ __forceinline__ void s4_from_sq(const float (&B)[6], float f4, float (&s4)[5]) {
  const float b1 = f4 * B[1];
  s4[0] = fmaf(f4, B[2], -0.5f * fmaf(f4, B[0], b1));
  s4[1] = 2.0f * (f4 * B[4]);
  s4[2] = 2.0f * (f4 * B[5]);
  s4[3] = 0.5f * fmaf(f4, B[0], -b1);
  s4[4] = 2.0f * (f4 * B[3]);
}
__device__ __forceinline__ constexpr float s4_scale(int m) {
  return m == 0 ? 1.0f / (3.0f * sh::k20) : (m == 3 ? 1.0f / sh::k22 : 1.0f / sh::k21);
}

// tr(A^3) = sum_ab (A^2)_ab A_ab for symmetric A
__device__ __forceinline__ float tr_cube(const float (&A)[6]) {
  float B[6];
  sym_sq(A, B);
  const float diag = fmaf(A[2], B[2], fmaf(A[0], B[0], A[1] * B[1]));
  const float off = fmaf(A[5], B[5], fmaf(A[3], B[3], A[4] * B[4]));
  return fmaf(2.0f, off, diag);
}

}  // namespace nepmi
