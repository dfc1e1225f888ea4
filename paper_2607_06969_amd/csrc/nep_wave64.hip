// nep_wave64.hip -- the float64 evaluation with one wavefront per atom, for
// batches too small to fill the chip with one thread per atom.
//
//   k_atom64  an atom's descriptors, network, site energy, radial adjoint rows
//             atil_i[b][k] = sum_n dE_i/dq_n c[Z_i][b][n][k], sigma = dE_i/dS_i and
//             from it dE_i/dr_ij of the angular descriptors for every entry of
//             the angular part of its list
//   k_pair64  an atom's force and virial from its own and its neighbours' parts
//
// The lanes take what a phase has most of, as in the float32 kernels
// (nep_wave.hip), and hand over through LDS.
#include "train_device.hpp"

namespace nepmi {

__device__ __forceinline__ double sum64(double v, int from) {
  for (int o = 32; o >= from; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

constexpr int kAtomWaves = 4;  // wavefronts (atoms) per block

// Bound by the latency of its phases: eight wavefronts per compute unit share its
// LDS (12 KB each, and the first-layer weights of the block's species).  2,000
// atoms of the Ge-Sb-Te model: 242 us in five kernels with a thread per atom, 30.5
// here.
template <class S>
__global__ __launch_bounds__(64 * kAtomWaves) void k_atom64(TrainIOT<double> io, CutoffsT<double> cut,
                                                            const double* __restrict__ params,
                                                            const uint32_t* __restrict__ nbrTA, int rowTA,
                                                            const int* __restrict__ cntAV, double4* __restrict__ fA,
                                                            double* __restrict__ aR) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K, D = S::D, H = S::H;
  constexpr int PC = 16;                                    // angular pairs in LDS at a time
  constexpr int RW = BR | 1, QW = (2 * BA) | 1, YW = K | 1, GW = NA | 1, WW = D | 1;
  constexpr int kRad = 64 * RW, kAng = PC * (QW + YW + 2 * GW + 4);
  constexpr int LQ = 64 / K, R = NA / LQ;                   // lanes per lm, functions per lane
  constexpr int NG = 64 / PC, NH = NA / NG;                 // lanes per pair, functions of each
  static_assert(T * BR <= 64 && D <= 64 && H <= 64 && NA * L <= 64 && NA % LQ == 0 && NA % NG == 0, "one lane each");
  struct Wave {
    double buf[kRad > kAng ? kRad : kAng];  // radial rows, the radial sums, the angular chunk
    double S_[NA * K], q[64], z[64], s4[NA * 5];
  };
  __shared__ Wave waves[kAtomWaves];
  __shared__ double W0s[H * WW];
  const int64_t ns = io.ns;
  const int64_t p0 = xcd_tile() * kAtomWaves;
  if (p0 >= ns || io.cfg_of[p0] < 0) return;  // padding ends a species: the block has no atom
  const int lane = threadIdx.x & 63, w = (int)threadIdx.x >> 6;
  const int64_t p = p0 + w;
  const int c = p < ns ? io.cfg_of[p] : -1;
  const int Zi = __builtin_amdgcn_readfirstlane(species_of(io.pos4[p0]));
  const double* W0 = params + S::PCR + S::PCA + (int64_t)Zi * S::PMLP;
  const double* b0 = W0 + H * D;
  const double* w1 = b0 + H;
  for (int t = threadIdx.x; t < H * D; t += 64 * kAtomWaves) W0s[t / D * WW + t % D] = W0[t];
  __syncthreads();
  if (c < 0) return;
  Wave& m = waves[w];
  double* qS = m.buf;            // [pair] Q_k, Q'_k
  double* yS = qS + PC * QW;     // [pair] Y_lm
  double* gS = yS + PC * YW;     // [pair] g_n
  double* dS = gS + PC * GW;     // [pair] g'_n
  double* uS = dS + PC * GW;     // [pair] u, 1/d
  double* cS = m.z;              // [pair] species (while z is not in use)
  const double4 xi = io.pos4[p];
  double Hc[9];
  load_cell9(io.cfgs, c, Hc);
  const double rcR_inv = 1.0 / cut.rcR, rcA_inv = 1.0 / cut.rcA;

  // ---- radial sums P_b[k], accumulator (b, k) in lane b B_R + k
  double P = 0.0;
  const int n = io.cntR[p];
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int k = k0 + lane;
    const uint32_t e = io.nbrR[group_index(ns, p, k < n ? k : n - 1)];
    const PV<double> v = pvec(io.pos4, e, xi, Hc);
    const bool in = k < n && v.d2 < cut.rcR2;
    int row = 0, rows = 0, j0 = 0, nj = 0;  // rows by species
#pragma unroll
    for (int b = 0; b < T; ++b) {
      const uint64_t mb = __ballot(in && (T == 1 || v.zj == b));
      const int nb = __builtin_popcountll(mb);
      if (T == 1 || v.zj == b) row = rows + lanes_below(mb);
      if (lane / BR == b) {
        j0 = rows;
        nj = nb;
      }
      rows += nb;
    }
    wave_fence();
    if (in) {
      double Q[BR], dQ[BR];
      cheb_basis_d<BR>(sqrt_(v.d2), rcR_inv, Q, dQ);
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) m.buf[row * RW + kk] = Q[kk];
    }
    wave_fence();
#pragma unroll 4
    for (int j = 0; j < nj; ++j) P += m.buf[(j0 + j) * RW + lane % BR];
  }
  wave_fence();
  if (lane < T * BR) m.buf[lane] = P;
  wave_fence();
  if (lane < NR) {
    double a = 0.0;
#pragma unroll
    for (int b = 0; b < T; ++b)
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) a = fma(params[((Zi * T + b) * NR + lane) * BR + kk], m.buf[b * BR + kk], a);
    m.q[lane] = a;
  }

  // ---- angular pairs a0 .. a0 + np - 1 of the angular part of the list; entries
  //      beyond rc_angular count zero
  const uint32_t* list = nbrTA + p * rowTA;
  const int nA = cntAV[p];
  auto chunk = [&](int a0, int np) {
    wave_fence();
    if (lane < np) {
      const PV<double> v = pvec(io.pos4, list[a0 + lane], xi, Hc);
      const double d = sqrt_(v.d2), inv = 1.0 / d;
      double Q[BA], dQ[BA], Y[K];
#pragma unroll
      for (int kk = 0; kk < BA; ++kk) Q[kk] = dQ[kk] = 0.0;
      if (v.d2 < cut.rcA2) cheb_basis_d<BA>(d, rcA_inv, Q, dQ);
      real_sph<L>(v.rx * inv, v.ry * inv, v.rz * inv, Y);
#pragma unroll
      for (int kk = 0; kk < BA; ++kk) {
        qS[lane * QW + kk] = Q[kk];
        qS[lane * QW + BA + kk] = dQ[kk];
      }
#pragma unroll
      for (int lm = 0; lm < K; ++lm) yS[lane * YW + lm] = Y[lm];
      uS[lane * 4] = v.rx * inv;
      uS[lane * 4 + 1] = v.ry * inv;
      uS[lane * 4 + 2] = v.rz * inv;
      uS[lane * 4 + 3] = inv;
      cS[lane] = (double)v.zj;
    }
    wave_fence();
    for (int it = lane; it < np * NA; it += 64) {
      const int j = it / NA, nn = it % NA;
      const double* cl = params + S::PCR + ((Zi * T + (int)cS[j]) * NA + nn) * BA;
      double g = 0.0, gp = 0.0;
#pragma unroll
      for (int kk = 0; kk < BA; ++kk) {
        g = fma(cl[kk], qS[j * QW + kk], g);
        gp = fma(cl[kk], qS[j * QW + BA + kk], gp);
      }
      gS[j * GW + nn] = g;
      dS[j * GW + nn] = gp;
    }
    wave_fence();
  };
  auto chunk_len = [&](int a0) { return nA - a0 < PC ? nA - a0 : PC; };
  const int lm = lane % K, ll = lm < 3 ? 1 : (lm < 8 ? 2 : (lm < 15 ? 3 : 4));
  const bool own = lane / K < LQ;
  const int n0 = (own ? lane / K : LQ - 1) * R;
  double Sv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) Sv[r] = 0.0;
  for (int a0 = 0; a0 < nA; a0 += PC) {
    const int np = chunk_len(a0);
    chunk(a0, np);
#pragma unroll 4
    for (int j = 0; j < np; ++j) {
      const double y = yS[j * YW + lm];
#pragma unroll
      for (int r = 0; r < R; ++r) Sv[r] = fma(gS[j * GW + n0 + r], y, Sv[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (own) m.S_[(n0 + r) * K + lm] = Sv[r];
  wave_fence();

  // ---- descriptors (A and A^2 of the 4-body terms stay with their function's lane)
  double A2[6];
  if (lane < NA * L) {
    const int l = lane / NA + 1, nn = lane % NA;
    const double* Sn = m.S_ + nn * K + l * l - 1;
    double s = 0.0;
    for (int x = 0; x < 2 * l + 1; ++x) s = fma(Sn[x], Sn[x], s);
    m.q[NR + lane] = s;
    if constexpr (S::F5)
      if (l == 1) m.q[S::OFF5 + nn] = s * s;
  }
  if constexpr (S::F4) {
    if (lane < NA) {
      double A[6];
      sym_from_s2(m.S_ + lane * K + 3, A);
      sym_sq6(A, A2);
      m.q[S::OFF4 + lane] = sym_dot(A2, A);
    }
  }
  wave_fence();

  // ---- network: a hidden unit, then a descriptor, per lane
  const int h = lane < H ? lane : H - 1;
  double a = b0[h];
#pragma unroll 8
  for (int d = 0; d < D; ++d) a = fma(W0s[h * WW + d], m.q[d], a);
  const double t = tanh_(a), w1h = w1[h];
  const double E = sum64(lane < H ? w1h * t : 0.0, 1) + w1[H];
  m.z[lane] = w1h * (1.0 - t * t);
  if (lane == 0 && io.Ei) io.Ei[io.orig[p]] = E;
  const double q1 = m.q[NR + (lane < NA ? lane : 0)];  // sum of squares of l = 1
  wave_fence();
  const int d0 = lane < D ? lane : D - 1;
  double Fp = 0.0;
#pragma unroll 8
  for (int x = 0; x < H; ++x) Fp = fma(m.z[x], W0s[x * WW + d0], Fp);
  wave_fence();
  m.q[lane] = Fp;
  wave_fence();
  if (lane < T * BR) {
    const int b = lane / BR, kk = lane % BR;
    double acc = 0.0;
#pragma unroll
    for (int nn = 0; nn < NR; ++nn) acc = fma(m.q[nn], params[((Zi * T + b) * NR + nn) * BR + kk], acc);
    aR[((int64_t)b * ns + p) * BR + kk] = acc;
  }
  if (nA == 0) return;

  // ---- sigma = dE/dS in place of S
  if (lane < NA) {
    if constexpr (S::F4) {
      double M[6], g4[5];
#pragma unroll
      for (int x = 0; x < 6; ++x) M[x] = 3.0 * m.q[S::OFF4 + lane] * A2[x];
      chain_s2(M, g4);
#pragma unroll
      for (int x = 0; x < 5; ++x) m.s4[lane * 5 + x] = g4[x];
    }
    // of l = 1, with the 5-body part
    m.z[lane] = 2.0 * m.q[NR + lane] + (S::F5 ? 4.0 * m.q[S::F5 ? S::OFF5 + lane : 0] * q1 : 0.0);
  }
  wave_fence();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int nn = n0 + r;
    double s = Sv[r] * (ll == 1 ? m.z[nn] : 2.0 * m.q[NR + (ll - 1) * NA + nn]);
    if constexpr (S::F4)
      if (ll == 2) s += m.s4[nn * 5 + lm - 3];
    if (own) m.S_[nn * K + lm] = s;
  }

  // ---- pair forces: NH functions of a pair per lane,
  //      u sum_n g'_n Z_n + (I - u u^T) grad_u(sum_lm G_lm P_lm) / d with
  //      Z_n = sum_lm sigma_nlm Y_lm, G_lm = sum_n sigma_nlm g_n
  for (int a0 = 0; a0 < nA; a0 += PC) {
    const int np = chunk_len(a0);
    if (nA > PC) chunk(a0, np);
    wave_fence();
    const int j = lane % PC, f0 = lane / PC * NH;
    double fx = 0.0, fy = 0.0, fz = 0.0;
    if (j < np) {
      const double ux = uS[j * 4], uy = uS[j * 4 + 1], uz = uS[j * 4 + 2], inv = uS[j * 4 + 3];
      double G[K], s = 0.0;
#pragma unroll
      for (int x = 0; x < K; ++x) G[x] = 0.0;
#pragma unroll
      for (int f = 0; f < NH; ++f) {
        const double g = gS[j * GW + f0 + f];
        double Z = 0.0;
#pragma unroll
        for (int x = 0; x < K; ++x) {
          const double sg = m.S_[(f0 + f) * K + x];
          Z = fma(sg, yS[j * YW + x], Z);
          G[x] = fma(sg, g, G[x]);
        }
        s = fma(dS[j * GW + f0 + f], Z, s);
      }
      double gx, gy, gz;
      real_sph_grad_dot<L>(ux, uy, uz, G, gx, gy, gz);
      const double ug = ux * gx + uy * gy + uz * gz;
      fx = s * ux + (gx - ug * ux) * inv;
      fy = s * uy + (gy - ug * uy) * inv;
      fz = s * uz + (gz - ug * uz) * inv;
    }
    fx = sum64(fx, PC);
    fy = sum64(fy, PC);
    fz = sum64(fz, PC);
    if (lane < np) fA[(int64_t)(a0 + lane) * ns + p] = make_double4(fx, fy, fz, 0.0);
  }
}

// A list entry per lane: the radial pair in both directions through the two
// adjoint rows, the own angular part (also into the virial) and minus the
// neighbour's, found through the reverse index (see k_force64).  Bound by the
// latency of the gathers of the neighbours' rows and forces (2,000 atoms: 51 us
// with a thread per atom, 9.5 here).
template <class S>
__global__ __launch_bounds__(64) void k_pair64(TrainIOT<double> io, CutoffsT<double> cut,
                                               const double* __restrict__ aR, const uint32_t* __restrict__ vrev,
                                               const double4* __restrict__ fA, double* __restrict__ F,
                                               double* __restrict__ W) {
  constexpr int T = S::T, BR = S::BR;
  __shared__ double own_s[T * BR];
  const int64_t ns = io.ns;
  const int64_t p = xcd_tile();
  const int c = io.cfg_of[p];
  if (c < 0) return;
  const int lane = threadIdx.x;
  const double4 xi = io.pos4[p];
  const int Zi = __builtin_amdgcn_readfirstlane(species_of(xi));
  if (lane < T * BR) own_s[lane] = aR[((int64_t)(lane / BR) * ns + p) * BR + lane % BR];
  double Hc[9];
  load_cell9(io.cfgs, c, Hc);
  const double rcR_inv = 1.0 / cut.rcR;
  wave_fence();
  double acc[12];  // force, virial
#pragma unroll
  for (int x = 0; x < 12; ++x) acc[x] = 0.0;
  const int n = io.cntR[p];
  int ka0 = 0;  // entries of the angular part seen
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int k = k0 + lane;
    const bool valid = k < n;
    const int64_t gk = group_index(ns, p, valid ? k : n - 1);
    const uint32_t rv = valid ? vrev[gk] : 0xFFFFFFFFu;
    const PV<double> v = pvec(io.pos4, io.nbrR[gk], xi, Hc);
    const uint64_t mp = __ballot(rv != 0xFFFFFFFFu);
    const int ka = ka0 + lanes_below(mp);
    ka0 += __builtin_popcountll(mp);
    double f[3] = {0.0, 0.0, 0.0};  // dE_i/dr_ij
    if (valid && v.d2 < cut.rcR2) {
      const double d = sqrt_(v.d2), inv = 1.0 / d;
      double Q[BR], dQ[BR];
      cheb_basis_d<BR>(d, rcR_inv, Q, dQ);
      const double* aj = aR + ((int64_t)Zi * ns + v.q) * BR;
      const double* ai = own_s + (T == 1 ? 0 : v.zj * BR);
      double own = 0.0, rev = 0.0;
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) {
        own = fma(ai[kk], dQ[kk], own);
        rev = fma(aj[kk], dQ[kk], rev);
      }
      const double u[3] = {v.rx * inv, v.ry * inv, v.rz * inv};
#pragma unroll
      for (int x = 0; x < 3; ++x) {
        f[x] = own * u[x];
        acc[x] += rev * u[x];  // minus dE_j/dr_ji (r_ji = -r_ij)
      }
    }
    if (rv != 0xFFFFFFFFu) {
      const double4 o = fA[(int64_t)ka * ns + p];
      f[0] += o.x;
      f[1] += o.y;
      f[2] += o.z;
      // a partner that was not found (0xFFFFFFFE) has made the list build fail
      // already; the test only keeps the read in bounds
      if (rv <= 0xFFFFu) {
        const double4 b = fA[(int64_t)rv * ns + v.q];
        acc[0] -= b.x;
        acc[1] -= b.y;
        acc[2] -= b.z;
      }
    }
    const double r[3] = {v.rx, v.ry, v.rz};
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      acc[x] += f[x];
#pragma unroll
      for (int y = 0; y < 3; ++y) acc[3 + 3 * x + y] -= f[x] * r[y];
    }
  }
#pragma unroll
  for (int x = 0; x < 12; ++x) acc[x] = sum64(acc[x], 1);
  const int64_t i = io.orig[p];
  double out = 0.0;
#pragma unroll
  for (int x = 0; x < 12; ++x) out = lane == x ? acc[x] : out;
  if (lane < 3) F[3 * i + lane] = out;
  else if (lane < 12) W[9 * i + lane - 3] = out;
}

template <class S>
int Wave64<S>::forward(hipStream_t st, const TrainIOT<double>& io, const CutoffsT<double>& cut, const F64Args& a,
                       double* forces) {
  hipLaunchKernelGGL(k_atom64<S>, dim3((unsigned)((io.ns + kAtomWaves - 1) / kAtomWaves)), dim3(64 * kAtomWaves), 0, st,
                     io, cut, a.params, a.nbrTA, a.rowTA, a.cntAV, a.fA, a.aR);
  hipLaunchKernelGGL(k_pair64<S>, dim3((unsigned)io.ns), dim3(64), 0, st, io, cut, a.aR, a.vrev, a.fA, forces, a.Wi);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template struct Wave64<ShapeSmall>;
template struct Wave64<ShapeGST>;
template struct Wave64<ShapeTable2>;

}  // namespace nepmi
