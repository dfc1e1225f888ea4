// train_wave.hip -- the parameter gradient in one kernel, one wavefront per atom
// at a time.
//
// For every atom the kernel runs the tangent pass (radial and angular sums and
// their derivatives along t_ij = lambda_j - lambda_i + mu r_ij), the network's
// second-order adjoint, sigma = dE/dS and Sbar = dj/dS, and the angular
// coefficient pass (see train.hip for the formulas), handing over through LDS,
// and adds the atom's share of every parameter's gradient to accumulators that
// the lanes hold over all atoms of their wavefront: lane h the row h of the
// first layer, and so on.  Nothing per atom goes through memory.
//
// A wavefront's atoms are of one species: some 12 at the largest batches (48 in
// float64), up to 16 (80) of a species whose share of the blocks is rounded down to
// one.  Their shares are summed in the wavefront's arithmetic; the block's
// wavefronts are then added in float64, in order, and the blocks by
// k_train_final, in order: the order depends on the batch only.
#include "train_device.hpp"

namespace nepmi {

constexpr int kTWaves = 4;  // wavefronts per block

// Blocks of species s, of about `want` in all: in proportion to its slots,
// rounded down (one block over what the chip holds at once would run alone
// after the others), but one if it has any (want + n_species blocks suffice).
__device__ __forceinline__ int species_blocks(const int* __restrict__ base, int n_species, int want, int s) {
  const int64_t mine = base[s + 1] - base[s], all = base[n_species] - base[0];
  const int n = mine > 0 ? (int)(want * mine / all) : 0;
  return mine > 0 && n < 1 ? 1 : n;
}

// Entries of a species' gradient, in the order of a block's partial sums.
template <class S>
struct GradEntries {
  static constexpr int W0 = 0, CR = W0 + S::H * S::D, CA = CR + S::NR * S::T * S::BR, B0 = CA + S::T * S::NA * S::BA,
                       W1 = B0 + S::H, B1 = W1 + S::H, N = B1 + 1;
};

// Bound by the latency of its phases at two wavefronts per SIMD (255 registers,
// 11.5 KB of LDS each; the vector units are busy 40 % of the time), some 2,300
// vector and 500 LDS instructions per atom.  Loss gradient of 9,031 atoms of the
// Ge-Sb-Te model: 165 us in seven kernels, 83 in this one and the sum.
template <class S, class R>
__global__ __launch_bounds__(64 * kTWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_train_wave(
    TrainIOT<R> io, CutoffsT<R> cut, const R* __restrict__ params, const int* __restrict__ base, int want,
    double* __restrict__ part) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K, D = S::D, H = S::H;
  using G = GradEntries<S>;
  constexpr int PC = 16;                                         // angular pairs in LDS at a time
  constexpr int RR = 32;                                         // radial rows in LDS at a time
  constexpr int RW = (2 * BR) | 1, YW = K | 1, GW = (NA + 3) / 4 * 4, QW = (2 * BA) | 1, AW = 7;
  constexpr int LQ = 64 / K, NS = NA / LQ;                       // lanes per lm, S accumulators per lane
  constexpr int NC = (NR * T * BR + 63) / 64, NG = (NA * BA + 63) / 64;
  constexpr int kAng = PC * (2 * YW + 2 * GW + QW + 2), kRad = RR * RW;
  constexpr int kBuf = kAng > kRad ? kAng : kRad;
  constexpr int WD = D | 1;
  static_assert(H <= 64 && D <= 64 && T * BR <= 64 && NA * L <= 64 && NR <= 64, "one lane each");
  struct Wave {
    R buf[kBuf];
    R angr[64 * AW];
    R S_[NA * K], Sd[NA * K];
    R P[T * BR], Pd[T * BR];
    R q[64], qd[64], ab[64], z[64], qb[64], Fp[64];
    R g4s[NA * 5], g4b[NA * 5];
  };
  __shared__ __align__(16) char raw[sizeof(Wave) * kTWaves];
  __shared__ R W0s[H * WD];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  Wave& m = reinterpret_cast<Wave*>(raw)[wv];

  // this block's species and share
  int s = 0, j = (int)blockIdx.x, nb = 0;
  for (; s < T; ++s) {
    nb = species_blocks(base, T, want, s);
    if (j < nb) break;
    j -= nb;
  }
  if (s == T) return;
  const int Zs = s;
  const R* W0g = params + S::PCR + S::PCA + (int64_t)Zs * S::PMLP;
#pragma unroll
  for (int u = 0; u < (H * D + 64 * kTWaves - 1) / (64 * kTWaves); ++u) {  // every load before the first store
    const int t = threadIdx.x + u * 64 * kTWaves;
    if (t < H * D) W0s[(t / D) * WD + t % D] = W0g[t];
  }
  __syncthreads();
  const R* b0g = W0g + H * D;
  const R* w1g = b0g + H;
  const R b0 = lane < H ? b0g[lane] : R(0), w1 = lane < H ? w1g[lane] : R(0);
  const R* cR = params + (int64_t)Zs * (T * NR * BR);
  const R* cA = params + S::PCR + (int64_t)Zs * (T * NA * BA);
  const int64_t ns = io.ns;
  const R rcR_inv = R(1.0) / cut.rcR, rcA_inv = R(1.0) / cut.rcA;

  R gW[D], gC[NC], gA[T][NG], gb = R(0), gw = R(0), ge = R(0);
#pragma unroll
  for (int d = 0; d < D; ++d) gW[d] = R(0);
#pragma unroll
  for (int r = 0; r < NC; ++r) gC[r] = R(0);
#pragma unroll
  for (int b = 0; b < T; ++b)
#pragma unroll
    for (int r = 0; r < NG; ++r) gA[b][r] = R(0);

  R* yS = m.buf;                // [pair][lm] Y
  R* lS = yS + PC * YW;         // [pair][lm] grad Y . t
  R* gS = lS + PC * YW;         // [pair][n] g_n, later alpha + gamma
  R* dS = gS + PC * GW;         // [pair][n] g'_n (u.t), later beta
  R* qS = dS + PC * GW;         // [pair] Q_k, dQ_k
  R* uS = qS + PC * QW;         // [pair] u.t
  R* zS = uS + PC;              // [pair] species

  const int n_slots = base[s + 1] - base[s], nw = nb * kTWaves;
  const int each = (n_slots + nw - 1) / nw, w = j * kTWaves + wv;
  const int p_lo = base[s] + w * each, p_hi = min(p_lo + each, base[s + 1]);
  // The next atom's first round of list entries and their positions are loaded
  // during the present atom's work, a step at a time (configuration and list
  // length, entries, positions), so that an atom does not begin with a chain of
  // memory latencies.
  struct Ahead {
    int c, n;
    uint32_t e;          // first round: entry of this lane
    Vec4<R> x, l;        // position and lambda of its neighbour
    Vec4<R> xi, li;      // the atom's own
  };
  auto ahead_count = [&](Ahead& a, int p) {
    a.c = io.cfg_of[p];
    a.n = io.cntR[p];
  };
  auto ahead_entry = [&](Ahead& a, int p) {
    const int k = lane < a.n ? lane : a.n - 1;
    a.e = a.n > 0 ? io.nbrR[group_index(ns, p, k)] : (uint32_t)p;
  };
  auto ahead_pos = [&](Ahead& a, int p) {
    a.x = io.pos4[a.e & kNbrMask];
    a.l = io.lam4[a.e & kNbrMask];
    a.xi = io.pos4[p];
    a.li = io.lam4[p];
  };
  Ahead cur, nxt;
  if (p_lo < p_hi) {
    ahead_count(nxt, p_lo);
    ahead_entry(nxt, p_lo);
    ahead_pos(nxt, p_lo);
  }
#pragma unroll 1
  for (int p = p_lo; p < p_hi; ++p) {
    cur = nxt;
    const int pn = p + 1 < p_hi ? p + 1 : p;
    ahead_count(nxt, pn);
    const int c = cur.c;
    if (c < 0) {  // padding
      ahead_entry(nxt, pn);
      ahead_pos(nxt, pn);
      continue;
    }
    const Vec4<R> xi = cur.xi, li = cur.li;
    const R eb = (R)io.ebar[c];
    R Hc[9], mu[9];
    load_cell9(io.cfgs, c, Hc);
#pragma unroll
    for (int x = 0; x < 9; ++x) mu[x] = (R)io.mu[9 * c + x];
    const int n = cur.n;
    const int lm = lane % K, n0 = (lane / K < LQ ? lane / K : LQ - 1) * NS;  // S accumulators: lm, n0 ..
    R P = R(0), Pd = R(0), Sa[NS], Sb[NS];
#pragma unroll
    for (int r = 0; r < NS; ++r) Sa[r] = Sb[r] = R(0);

    // geometry and harmonics of pairs a0 .. a0 + np - 1 of the round, one per lane
    auto chunk = [&](int a0, int np) {
      wave_fence();
      if (lane < np) {
        const R* row = m.angr + (a0 + lane) * AW;
        const R rx = row[0], ry = row[1], rz = row[2], tx = row[3], ty = row[4], tz = row[5];
        const R d = sqrt_(pair_d2(rx, ry, rz)), inv = R(1.0) / d;
        const R ux = rx * inv, uy = ry * inv, uz = rz * inv;
        const R ut = ux * tx + uy * ty + uz * tz;
        {
          R Q[BA], dQ[BA];
          cheb_basis_d<BA>(d, rcA_inv, Q, dQ);
#pragma unroll
          for (int k = 0; k < BA; ++k) {
            qS[lane * QW + k] = Q[k];
            qS[lane * QW + BA + k] = dQ[k];
          }
        }
        {
          R Y[K];
          real_sph<L>(ux, uy, uz, Y);
#pragma unroll
          for (int lm = 0; lm < K; ++lm) yS[lane * YW + lm] = Y[lm];
        }
        {
          // grad_r Y_lm . t = grad P_lm . (t - (u.t) u) / d
          R Dl[K];
          real_sph_dir<L>(ux, uy, uz, (tx - ut * ux) * inv, (ty - ut * uy) * inv, (tz - ut * uz) * inv, Dl);
#pragma unroll
          for (int lm = 0; lm < K; ++lm) lS[lane * YW + lm] = Dl[lm];
        }
        uS[lane] = ut;
        zS[lane] = row[6];
      }
      wave_fence();
    };
    // the list in rounds of 64 entries: the angular pairs of each round go to
    // m.angr; radial(in, v, ut): the radial pairs; angular(np): a chunk of
    // angular pairs ready in LDS
    int n_ang = 0;
    auto walk = [&](auto&& radial, auto&& angular) {
      n_ang = 0;
      for (int k0 = 0; k0 < n; k0 += 64) {
        const int k = k0 + lane;
        uint32_t e = cur.e;
        Vec4<R> xq = cur.x, lj = cur.l;
        if (k0 > 0) {
          e = io.nbrR[group_index(ns, p, k < n ? k : n - 1)];
          xq = io.pos4[e & kNbrMask];
          lj = io.lam4[e & kNbrMask];
        }
        const PV<R> v = pvec_at(e, xq, xi, Hc);
        const R tx = lj.x - li.x + mu[0] * v.rx + mu[1] * v.ry + mu[2] * v.rz;
        const R ty = lj.y - li.y + mu[3] * v.rx + mu[4] * v.ry + mu[5] * v.rz;
        const R tz = lj.z - li.z + mu[6] * v.rx + mu[7] * v.ry + mu[8] * v.rz;
        const bool inR = k < n && v.d2 < cut.rcR2, inA = inR && v.d2 < cut.rcA2;
        const uint64_t mA = __ballot(inA);
        wave_fence();
        if (inA) {
          R* row = m.angr + lanes_below(mA) * AW;
          row[0] = v.rx;
          row[1] = v.ry;
          row[2] = v.rz;
          row[3] = tx;
          row[4] = ty;
          row[5] = tz;
          row[6] = (R)v.zj;
        }
        radial(inR, v, v.rx * tx + v.ry * ty + v.rz * tz);
        const int nA = __builtin_popcountll(mA);
        n_ang += nA;
        for (int a0 = 0; a0 < nA; a0 += PC) {
          const int np = nA - a0 < PC ? nA - a0 : PC;
          chunk(a0, np);
          angular(np);
        }
      }
    };

    // ---- tangent pass.  Lanes (b, k): P_b[k] = sum_{j in b} Q_k and Pd_b[k] =
    //      sum_{j in b} dQ_k (u.t); lanes (n, lm): S and its derivative along t
    walk(
        [&](bool in, const PV<R>& v, R rt) {
          // rows by species: each accumulator runs over its own
          int kr = 0, nr = 0, j0 = 0, j1 = 0;
#pragma unroll
          for (int b = 0; b < T; ++b) {
            const uint64_t mR = __ballot(in && (T == 1 || v.zj == b));
            if (T == 1 || v.zj == b) kr = nr + lanes_below(mR);
            const int nb = __builtin_popcountll(mR);
            if (lane / BR == b) {
              j0 = nr;
              j1 = nr + nb;
            }
            nr += nb;
          }
          R Q[BR], dQ[BR], ut = R(0);
          if (in) {
            const R d = sqrt_(v.d2);
            ut = rt / d;
            cheb_basis_d<BR>(d, rcR_inv, Q, dQ);
          }
          for (int r0 = 0; r0 < nr; r0 += RR) {
            wave_fence();
            if (in && kr >= r0 && kr < r0 + RR) {
              R* row = m.buf + (kr - r0) * RW;
#pragma unroll
              for (int k = 0; k < BR; ++k) {
                row[k] = Q[k];
                row[BR + k] = dQ[k] * ut;
              }
            }
            wave_fence();
            const R* q = m.buf - r0 * RW + lane % BR;
            const int i1 = j1 < r0 + RR ? j1 : r0 + RR;
#pragma unroll 4
            for (int i = j0 > r0 ? j0 : r0; i < i1; ++i) {
              P += q[i * RW];
              Pd += q[i * RW + BR];
            }
          }
        },
        [&](int np) {
          for (int it = lane; it < np * NA; it += 64) {
            const int i = it / NA, nn = it % NA;
            const R* cl = cA + ((int)zS[i] * NA + nn) * BA;
            const R* q = qS + i * QW;
            R g = R(0), gp = R(0), ck[BA];
            load_row<BA>(cl, ck);
#pragma unroll
            for (int k = 0; k < BA; ++k) {
              g = fma_(ck[k], q[k], g);
              gp = fma_(ck[k], q[BA + k], gp);
            }
            gS[i * GW + nn] = g;
            dS[i * GW + nn] = gp * uS[i];
          }
          wave_fence();
#pragma unroll 2
          for (int i = 0; i < np; ++i) {
            const R y = yS[i * YW + lm], yl = lS[i * YW + lm];
#pragma unroll
            for (int r = 0; r < NS; ++r) {
              const R g = gS[i * GW + n0 + r];
              Sa[r] = fma_(g, y, Sa[r]);
              Sb[r] = fma_(dS[i * GW + n0 + r], y, fma_(g, yl, Sb[r]));
            }
          }
        });
    wave_fence();
    if (lane < T * BR) {
      m.P[lane] = P;
      m.Pd[lane] = Pd;
    }
#pragma unroll
    for (int r = 0; r < NS; ++r)
      if (lane / K < LQ) {
        m.S_[(n0 + r) * K + lm] = Sa[r];
        m.Sd[(n0 + r) * K + lm] = Sb[r];
      }
    wave_fence();
    ahead_entry(nxt, pn);
    // ---- descriptors and their derivatives along t
    if (lane < NR) {
      R a = R(0), ad = R(0);
#pragma unroll
      for (int b = 0; b < T; ++b) {
        R ck[BR];
        load_row<BR>(cR + (b * NR + lane) * BR, ck);
#pragma unroll
        for (int k = 0; k < BR; ++k) {
          a = fma_(ck[k], m.P[b * BR + k], a);
          ad = fma_(ck[k], m.Pd[b * BR + k], ad);
        }
      }
      m.q[lane] = a;
      m.qd[lane] = ad;
    }
    if (lane < NA * L) {
      const int l = lane / NA + 1, nn = lane % NA, o = nn * K + l * l - 1;
      R a = R(0), ad = R(0);
#pragma unroll
      for (int x = 0; x < 2 * L + 1; ++x)
        if (x < 2 * l + 1) {
          a = fma_(m.S_[o + x], m.S_[o + x], a);
          ad = fma_(m.S_[o + x], m.Sd[o + x], ad);
        }
      m.q[NR + lane] = a;
      m.qd[NR + lane] = R(2.0) * ad;
      if constexpr (S::F5)
        if (l == 1) {
          m.q[S::OFF5 + nn] = a * a;
          m.qd[S::OFF5 + nn] = R(4.0) * a * ad;
        }
    }
    if constexpr (S::F4) {
      if (lane < NA) {
        R A[6], Ad[6], A2[6];
        sym_from_s2(&m.S_[lane * K + 3], A);
        sym_from_s2(&m.Sd[lane * K + 3], Ad);
        sym_sq6(A, A2);
        m.q[S::OFF4 + lane] = sym_dot(A2, A);
        m.qd[S::OFF4 + lane] = R(3.0) * sym_dot(A2, Ad);
      }
    }
    wave_fence();
    // ---- network: hidden unit `lane`, then descriptor `lane`
    {
      const R* row = W0s + (lane < H ? lane : H - 1) * WD;
      R a = b0, ad = R(0);
#pragma unroll 8
      for (int d = 0; d < D; ++d) {
        a = fma_(row[d], m.q[d], a);
        ad = fma_(row[d], m.qd[d], ad);
      }
      const R t = tanh_(a), s2 = R(1.0) - t * t, z = w1 * s2;
      const R ab = z * (eb + R(2.0) * t * ad);
      m.ab[lane] = ab;
      m.z[lane] = z;
      if (lane < H) {
        gb += ab;
        gw += eb * t - s2 * ad;
      }
      ge += eb;
      // W0: abar q^T - z qdot^T
#pragma unroll
      for (int d = 0; d < D; ++d) {
        gW[d] = fma_(ab, m.q[d], fma_(-z, m.qd[d], gW[d]));
        if (d % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // keeps the reads near their use
      }
    }
    wave_fence();
    {
      const R* col = W0s + (lane < D ? lane : D - 1);
      R qb = R(0), Fp = R(0);
#pragma unroll 10
      for (int h = 0; h < H; ++h) {
        qb = fma_(m.ab[h], col[h * WD], qb);
        Fp = fma_(m.z[h], col[h * WD], Fp);
      }
      m.qb[lane] = qb;
      m.Fp[lane] = Fp;
    }
    wave_fence();
    ahead_pos(nxt, pn);
    // c^R: qbar_R (x) P - dE/dq_R (x) P'
#pragma unroll
    for (int r = 0; r < NC; ++r) {
      const int e = lane + 64 * r < NR * T * BR ? lane + 64 * r : NR * T * BR - 1;
      const int nn = e / (T * BR), k = e % (T * BR);
      gC[r] = fma_(m.qb[nn], m.P[k], fma_(-m.Fp[nn], m.Pd[k], gC[r]));
    }
    // ---- sigma = dE/dS and Sbar = dj/dS, in place of S and Sdot
    if constexpr (S::F4) {
      if (lane < NA) {
        R A[6], Ad[6], A2[6], AAd[9], AdA[9], Ms[6], Mb[6], gs[5], gq[5];
        sym_from_s2(&m.S_[lane * K + 3], A);
        sym_from_s2(&m.Sd[lane * K + 3], Ad);
        sym_sq6(A, A2);
        sym_mul_sym(A, Ad, AAd);
        sym_mul_sym(Ad, A, AdA);
        const R fp4 = m.Fp[S::OFF4 + lane], qb4 = m.qb[S::OFF4 + lane];
        const int ix[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {0, 2}, {1, 2}};
#pragma unroll
        for (int x = 0; x < 6; ++x) {
          const R sym = AAd[3 * ix[x][0] + ix[x][1]] + AdA[3 * ix[x][0] + ix[x][1]];
          Ms[x] = R(3.0) * fp4 * A2[x];
          Mb[x] = R(3.0) * qb4 * A2[x] - R(3.0) * fp4 * sym;
        }
        chain_s2(Ms, gs);
        chain_s2(Mb, gq);
#pragma unroll
        for (int x = 0; x < 5; ++x) {
          m.g4s[lane * 5 + x] = gs[x];
          m.g4b[lane * 5 + x] = gq[x];
        }
      }
      wave_fence();
    }
    for (int a = lane; a < NA * K; a += 64) {
      const int nn = a / K, lm = a % K;
      const int l = lm < 3 ? 1 : (lm < 8 ? 2 : (lm < 15 ? 3 : 4));
      const R fp3 = m.Fp[NR + (l - 1) * NA + nn], qb3 = m.qb[NR + (l - 1) * NA + nn];
      R cs = R(2.0) * fp3, cbS = R(2.0) * qb3, cbD = -R(2.0) * fp3;
      if constexpr (S::F5) {
        if (l == 1) {
          const R fp5 = m.Fp[S::OFF5 + nn], qb5 = m.qb[S::OFF5 + nn], q1 = m.q[NR + nn], qd1 = m.qd[NR + nn];
          cs += R(4.0) * fp5 * q1;
          cbS += R(4.0) * qb5 * q1 - R(4.0) * fp5 * qd1;
          cbD += -R(4.0) * fp5 * q1;
        }
      }
      const R sv = m.S_[a], sd = m.Sd[a];
      R sg = cs * sv, sb = cbS * sv + cbD * sd;
      if constexpr (S::F4) {
        if (l == 2) {
          sg += m.g4s[nn * 5 + lm - 3];
          sb += m.g4b[nn * 5 + lm - 3];
        }
      }
      m.S_[a] = sg;
      m.Sd[a] = sb;
    }
    wave_fence();
    // ---- angular coefficients: (alpha + gamma) Q_k + beta dQ_k, with alpha =
    //      sum_lm Sbar Y, beta = -(u.t) sum_lm sigma Y, gamma = -sum_lm sigma grad Y.t
    auto coef = [&](int np) {
      for (int it = lane; it < np * NA; it += 64) {
        const int i = it / NA, nn = it % NA;
        const R* sg = m.S_ + nn * K;
        const R* sb = m.Sd + nn * K;
        R al = R(0), sy = R(0), ga = R(0);
#pragma unroll
        for (int lm = 0; lm < K; ++lm) {
          const R y = yS[i * YW + lm];
          al = fma_(sb[lm], y, al);
          sy = fma_(sg[lm], y, sy);
          ga = fma_(sg[lm], lS[i * YW + lm], ga);
        }
        gS[i * GW + nn] = al - ga;
        dS[i * GW + nn] = -uS[i] * sy;
      }
      wave_fence();
#pragma unroll 2
      for (int i = 0; i < np; ++i) {
        const int zj = __builtin_amdgcn_readfirstlane((int)zS[i]);
        R v[NG];
#pragma unroll
        for (int r = 0; r < NG; ++r) {
          const int e = lane + 64 * r < NA * BA ? lane + 64 * r : NA * BA - 1;
          const int nn = e / BA, k = e % BA;
          v[r] = fma_(gS[i * GW + nn], qS[i * QW + k], dS[i * GW + nn] * qS[i * QW + BA + k]);
        }
#pragma unroll
        for (int b = 0; b < T; ++b)
          if (T == 1 || zj == b)
#pragma unroll
            for (int r = 0; r < NG; ++r) gA[b][r] += v[r];
      }
      wave_fence();
    };
    // the pairs are still in LDS if one round and one chunk held them all
    if (n <= 64 && n_ang <= PC) {
      if (n_ang > 0) coef(n_ang);
    } else {
      walk([](bool, const PV<R>&, R) {}, coef);
    }
    wave_fence();
  }

  // ---- the block's wavefronts, in order, in float64: each puts its sums in LDS,
  //      the first layer in two halves, and every thread adds some entries
  constexpr int DH = (D + 1) / 2, NW = H * DH, NO = G::N - G::CR;
  static_assert(sizeof(R) * kTWaves * (NW > NO ? NW : NO) <= sizeof(raw), "the sums fit the wavefronts' work space");
  R* sums = reinterpret_cast<R*>(raw);
  double* out = part + (int64_t)blockIdx.x * G::N;
  auto total = [&](int i, int stride) {
    double v = (double)sums[i];
#pragma unroll
    for (int u = 1; u < kTWaves; ++u) v += (double)sums[u * stride + i];
    return v;
  };
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();
    if (lane < H) {
#pragma unroll
      for (int d = 0; d < DH; ++d)
        if (half * DH + d < D) sums[wv * NW + lane * DH + d] = gW[half * DH + d < D ? half * DH + d : 0];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NW; i += 64 * kTWaves) {
      const int d = half * DH + i % DH;
      if (d < D) out[G::W0 + i / DH * D + d] = total(i, NW);
    }
  }
  __syncthreads();
  {
    R* mine = sums + wv * NO - G::CR;
#pragma unroll
    for (int r = 0; r < NC; ++r)
      if (lane + 64 * r < NR * T * BR) mine[G::CR + lane + 64 * r] = gC[r];
#pragma unroll
    for (int b = 0; b < T; ++b)
#pragma unroll
      for (int r = 0; r < NG; ++r)
        if (lane + 64 * r < NA * BA) mine[G::CA + b * NA * BA + lane + 64 * r] = gA[b][r];
    if (lane < H) {
      mine[G::B0 + lane] = gb;
      mine[G::W1 + lane] = gw;
    }
    if (lane == 0) mine[G::B1] = ge;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NO; i += 64 * kTWaves) out[G::CR + i] = total(i, NO);
}

// The blocks' partial sums of every entry: eight runs of blocks side by side,
// combined in order.
constexpr int kFinalRuns = 8;
template <class S, class O>
__global__ __launch_bounds__(32 * kFinalRuns) void k_train_final(const int* __restrict__ base, int want,
                                                                 const double* __restrict__ part,
                                                                 O* __restrict__ grad, const int* stop) {
  const bool none = lists_void(stop);
  using G = GradEntries<S>;
  constexpr int T = S::T, NR = S::NR, BR = S::BR;
  __shared__ double sh[kFinalRuns][32];
  const int x = threadIdx.x % 32, run = threadIdx.x / 32;
  const int64_t t = (int64_t)blockIdx.x * 32 + x;
  const bool in = t < (int64_t)T * G::N;
  const int s = in ? (int)(t / G::N) : 0, e = in ? (int)(t % G::N) : 0;
  int first = 0;
  for (int z = 0; z < s; ++z) first += species_blocks(base, T, want, z);
  const int nb = in ? species_blocks(base, T, want, s) : 0;
  const int per = (nb + kFinalRuns - 1) / kFinalRuns, lo = run * per, hi = min(lo + per, nb);
  double acc = 0.0;
  const double* src = part + (int64_t)first * G::N + e;
  for (int b = lo; b < hi; b += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = b + u < hi ? src[(int64_t)(b + u) * G::N] : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) acc += v[u];
  }
  sh[run][x] = acc;
  __syncthreads();
  if (run != 0 || !in || none) return;
  for (int r = 1; r < kFinalRuns; ++r) acc += sh[r][x];
  const int64_t mlp = S::PCR + S::PCA + (int64_t)s * S::PMLP;
  int64_t dst;
  if (e < G::CR) {
    dst = mlp + e;
  } else if (e < G::CA) {
    const int r = e - G::CR, n = r / (T * BR), b = r % (T * BR) / BR, k = r % BR;
    dst = (int64_t)s * T * NR * BR + ((int64_t)b * NR + n) * BR + k;
  } else if (e < G::B0) {
    dst = S::PCR + (int64_t)s * T * S::NA * S::BA + (e - G::CA);
  } else {
    dst = mlp + S::H * S::D + (e - G::B0);
  }
  grad[dst] = (O)acc;
}

template <class S, class R>
int TrainWave<S, R>::run(hipStream_t st, const TrainIOT<R>& io, const CutoffsT<R>& cut, const R* params,
                         const int* base, double* part, R* grad) {
  const int want = train_wave_blocks<R>(io.ns);
  hipLaunchKernelGGL((k_train_wave<S, R>), dim3((unsigned)(want + S::T)), dim3(64 * kTWaves), 0, st, io, cut, params,
                     base, want, part);
  hipLaunchKernelGGL((k_train_final<S, R>), dim3((unsigned)((S::T * GradEntries<S>::N + 31) / 32)),
                     dim3(32 * kFinalRuns), 0, st, base, want, part, grad, io.stop);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template struct TrainWave<ShapeSmall, float>;
template struct TrainWave<ShapeGST, float>;
template struct TrainWave<ShapeTable2, float>;
template struct TrainWave<ShapeSmall, double>;
template struct TrainWave<ShapeGST, double>;
template struct TrainWave<ShapeTable2, double>;

}  // namespace nepmi
