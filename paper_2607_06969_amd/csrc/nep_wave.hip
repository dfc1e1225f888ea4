// nep_wave.hip -- descriptor/network and pair-force kernels with one wavefront
// per atom, for batches too small to fill the chip with one thread per atom.
//
// A thread that owns an atom walks its lists entry by entry; below some 30,000
// atoms the chip then holds less than half a wavefront per SIMD and the time is
// that of one walk.  Here the lanes of a wavefront take the pairs of one atom
// side by side, and every phase gives the lanes the work it has most of: a pair
// each for the geometry, a (pair, function) each for g_n, an accumulator each
// for the sums, a hidden unit or a descriptor each for the network.  The phases
// hand over through LDS; a wavefront needs no block-wide barrier.
//
// Every sum runs over the pairs (or d, h, n) in the order of the one-thread
// kernels, one fused multiply-add per term in one accumulator, and every value
// comes from the same helper functions, so the results agree bit for bit with
// variant 0 of k_desc and k_force, and a configuration keeps its bits whether
// it is evaluated alone or in a large batch.
#include "nep_device.hpp"
#include "nbr.hpp"

namespace nepmi {

// Order between the wavefront's LDS writes and its other lanes' reads.
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// Set bits of a ballot below this lane.
__device__ __forceinline__ int bits_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ int last_bit(uint64_t m) { return 63 - __builtin_clzll(m); }

constexpr int kPairChunk = 32;  // angular pairs held in LDS at a time
constexpr int odd(int n) { return n | 1; }  // row strides that spread a column over the banks

// Row of a derived coefficient table (16-byte aligned).
template <int B>
__device__ __forceinline__ void load_row(const float* __restrict__ src, float (&c)[B]) {
  static_assert(B % 4 == 0, "coefficient rows are read as float4");
#pragma unroll
  for (int k = 0; k < B / 4; ++k) {
    const float4 v = reinterpret_cast<const float4*>(src)[k];
    c[4 * k] = v.x;
    c[4 * k + 1] = v.y;
    c[4 * k + 2] = v.z;
    c[4 * k + 3] = v.w;
  }
}

// S_nlm accumulators of the wavefront: accumulator a = n K + lm in lane a % 64,
// register a / 64.
template <class S>
struct SumLanes {
  static constexpr int N = S::NA * S::K, R = (N + kWave - 1) / kWave;
  float v[R];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = 0.f;
  }
  // add pairs 0 .. n - 1 of the chunk in order (gS, pS: rows per pair)
  __device__ __forceinline__ void add(const float* gS, const float* pS, int n, int lane) {
    const float *g[R], *P[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int a = lane + kWave * r < N ? lane + kWave * r : N - 1;
      g[r] = gS + a / S::K;
      P[r] = pS + a % S::K;
    }
#pragma unroll 4
    for (int j = 0; j < n; ++j)
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = fmaf(g[r][j * odd(S::NA)], P[r][j * odd(S::K)], v[r]);
  }
  // apply the harmonics' constants and store [n][lm]
  __device__ __forceinline__ void store(float* sS, const float* kapS, int lane) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int a = lane + kWave * r;
      if (a < N) sS[a] = v[r] * kapS[a % S::K];
    }
  }
};

template <int L>
__device__ __forceinline__ void fill_kappa(float* kapS, int lane) {
  constexpr Kappa<L> kap;
#pragma unroll
  for (int lm = 0; lm < L * L + 2 * L; ++lm)
    if (lane == lm) kapS[lm] = kap.v[lm];
}

// ------------------------------------------------------------------ k_desc

// Latency and issue of one wavefront per atom bound it (about 930 VALU
// instructions per atom, a quarter of them on a quarter of the lanes or less,
// against 250 with one thread per atom), not the 1.3 KB it moves per atom.
// 3,686 atoms of the Ge-Sb-Te model 56 -> 15 us, 18,400 atoms 61 -> 49.
template <class S>
__global__ __launch_bounds__(kWave) void k_desc_wave(NepIO io, const float* __restrict__ params, int want_adjoint) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K, D = S::D, H = S::H;
  constexpr int RW = odd(BR + T);  // radial row: T_k, then the masked weight per species
  constexpr int PC = kPairChunk, GW = odd(NA), PW = odd(K);
  static_assert(T * BR <= kWave && D <= kWave && H <= kWave && NA * L <= kWave && NR <= kWave, "one lane each");
  constexpr int kRad = kWave * RW, kAng = PC * (GW + PW + 3);
  __shared__ ImageTable itab;
  __shared__ float buf[kRad > kAng ? kRad : kAng];  // radial rows, then the angular chunk
  __shared__ float angr[kWave * 5];                 // r_ij, |r|^2, species of the angular pairs found
  __shared__ int part_s[kWave];
  __shared__ float PT_s[T * BR], S_s[NA * K], kap_s[K];
  __shared__ __align__(16) float q_s[kWave], t_s[kWave], z_s[kWave], w_s[kWave];
  float* gS = buf;                 // [pair][n] g_n
  float* pS = gS + PC * GW;        // [pair][lm] Praw
  float* xS = pS + PC * PW;        // x, f_c / 2 and species per pair
  float* hS = xS + PC;
  float* cS = hS + PC;

  const int64_t ns = io.n_slots;
  const int64_t p = xcd_tile();
  if (p == ns) {  // the block past the last slot (there only for the flags)
    if (threadIdx.x == 0) deliver(io.mail);
    return;
  }
  const int lane = threadIdx.x;
  const int c = io.cfg_of[p];
  if (c < 0) {
    if (lane == 0) io.ccR[p] = io.ccA[p] = 0;
    return;
  }
  const float4 xi = io.pos4[p];
  const int Zs = __builtin_amdgcn_readfirstlane(__float_as_int(xi.w));
  const float* __restrict__ dco = params + S::PD;
  itab.fill();
  fill_kappa<L>(kap_s, lane);
  float Hc[9];
  load_cell(io.cfgs, c, Hc);
  const float rcR_inv = 1.0f / io.cut.rcR, rcA_inv = 1.0f / io.cut.rcA;
  const int n = io.cntR[p];
  // entries the mask's words hold (a list cut off at its capacity, which is
  // rebuilt before its results are used, may have more)
  const int kaMax = (io.capA + 63) / 64 * 64;
  lds_fence();

  // ---- filter the Verlet list into the pairs inside the two cutoffs, 64
  //      entries per round; accumulator (b, k) of lane b B_R + k sums the
  //      radial neighbours of species b in list order
  float PT = 0.f;
  SumLanes<S> sum;
  sum.zero();
  int nR = 0, nA = 0, ka0 = 0;  // pairs kept, entries of the angular part seen
  uint64_t mword = 0;           // entry mask of the angular part, 64 entries per word
  uint32_t lastR = 0, lastA = 0, lastP = 0;
  bool bad = false;
  for (int k0 = 0; k0 < n; k0 += kWave) {
    const int k = k0 + lane;
    const bool valid = k < n;
    const int64_t gi = group_index(ns, p, valid ? k : n - 1);
    const uint32_t e = io.nbrR[gi];
    const uint32_t rv = valid ? io.vrev[gi] : 0xFFFFFFFFu;
    const PairVec v = pair_vec(e, io.pos4[e & kNbrMask], xi, Hc, itab);
    const bool inR = valid && v.d2 < io.cut.rcR2;
    const bool part = rv != 0xFFFFFFFFu;
    const bool inA = inR && v.d2 < io.cut.rcA2;
    const uint64_t mR = __ballot(inR), mP = __ballot(part), mV = __ballot(inA && rv <= 0xFFFFu);
    const int kr = bits_below(mR), kp = bits_below(mP), kA = bits_below(mV);
    // within rc_angular now implies within rc_angular + skin at the last
    // build, so nA stays below capA and the reverse row exists
    const bool okA = inA && rv <= 0xFFFFu && nA + kA < io.capA;
    bad |= inA && !okA;
    const uint64_t mA = __ballot(okA);
    const uint32_t pr = (uint32_t)(ka0 + kp) | (rv << 16);
    if (inR) {
      io.cnR[group_index(ns, p, nR + kr)] = e;
      const float inv = rsqrt_hw(v.d2);
      const RadialF f = radial_f(v.d2 * inv * rcR_inv);
      float Tk[BR];
      cheb_t<BR>(f.x, Tk);
      float* row = buf + kr * RW;
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) row[kk] = Tk[kk];
#pragma unroll
      for (int b = 0; b < T; ++b) row[BR + b] = (T == 1 || v.zj == b) ? f.hf : 0.0f;
    }
    if (okA) {
      io.cnA[group_index(ns, p, nA + kA)] = e;
      io.cpA[group_index(ns, p, nA + kA)] = pr;
      float* row = angr + kA * 5;
      row[0] = v.rx;
      row[1] = v.ry;
      row[2] = v.rz;
      row[3] = v.d2;
      row[4] = __int_as_float(v.zj);
    }
    if (part) part_s[kp] = okA ? 1 : 0;
    lds_fence();
    // the mask bits of this round's entries of the angular part, appended
    const int np = __builtin_popcountll(mP);
    const uint64_t bits = __ballot(lane < np && part_s[lane] != 0);
    const int sh = ka0 & 63;
    mword |= bits << sh;
    if ((ka0 + np) >> 6 != ka0 >> 6) {
      if (lane == 0 && ka0 < kaMax) io.amask[(int64_t)(ka0 >> 6) * ns + p] = mword;
      mword = sh ? bits >> (64 - sh) : 0;
    }
    ka0 += np;
    if (mR) lastR = lane_of(e, last_bit(mR));
    if (mA) {
      lastA = lane_of(e, last_bit(mA));
      lastP = lane_of(pr, last_bit(mA));
    }
    const int cR = __builtin_popcountll(mR), cA = __builtin_popcountll(mA);
    nR += cR;
    nA += cA;
    if (lane < T * BR) {
      const float* m = buf + BR + lane / BR;
      const float* t = buf + lane % BR;
#pragma unroll 4
      for (int j = 0; j < cR; ++j) PT = fmaf(m[j * RW], t[j * RW], PT);
    }
    lds_fence();
    // the angular pairs of this round: S_nlm = sum_j g_n(r_ij) Y_lm(u_ij)
    for (int a0 = 0; a0 < cA; a0 += PC) {
      const int m = cA - a0 < PC ? cA - a0 : PC;
      if (lane < m) {
        const float* row = angr + (a0 + lane) * 5;
        const float inv = rsqrt_hw(row[3]);
        const RadialF f = radial_f(row[3] * inv * rcA_inv);
        float P[K];
        const float uy = row[1] * inv;
        raw_sph<L>(row[0] * inv, uy, row[2] * inv, dxy_sums(row[0], uy, inv), P);
#pragma unroll
        for (int lm = 0; lm < K; ++lm) pS[lane * PW + lm] = P[lm];
        xS[lane] = f.x;
        hS[lane] = f.hf;
        cS[lane] = row[4];
      }
      lds_fence();
      for (int it = lane; it < m * NA; it += kWave) {
        const int j = it / NA, nn = it % NA;
        float Tk[BA], cl[BA];
        cheb_t<BA>(xS[j], Tk);
        load_row<BA>(dco + S::PCR + (int64_t)((Zs * T + __float_as_int(cS[j])) * NA + nn) * BA, cl);
        float acc = 0.f;
#pragma unroll
        for (int kk = 0; kk < BA; ++kk) acc = fmaf(cl[kk], Tk[kk], acc);
        gS[j * GW + nn] = hS[j] * acc;
      }
      lds_fence();
      sum.add(gS, pS, m, lane);
      lds_fence();
    }
  }
  // the last, partly filled mask word and groups (they repeat the last entry)
  if (lane == 0) {
    if ((ka0 & 63) && ka0 < kaMax) io.amask[(int64_t)(ka0 >> 6) * ns + p] = mword;
    io.ccR[p] = nR;
    io.ccA[p] = nA;
  }
  if ((nR & 3) && lane < 4 - (nR & 3)) io.cnR[group_index(ns, p, nR + lane)] = lastR;
  if ((nA & 3) && lane < 4 - (nA & 3)) {
    io.cnA[group_index(ns, p, nA + lane)] = lastA;
    io.cpA[group_index(ns, p, nA + lane)] = lastP;
  }
  if (bad) atomicOr(&io.flags[kFlagAsym], 1);

  // ---- descriptors, Eq. 11, 16, 17
  if (lane < T * BR) PT_s[lane] = PT;
  sum.store(S_s, kap_s, lane);
  lds_fence();
  const float* cR = dco + (int64_t)Zs * (T * NR * BR);
  if (lane < NR) {
    float acc = 0.f;
#pragma unroll
    for (int b = 0; b < T; ++b) {
      float cl[BR];
      load_row<BR>(cR + (b * NR + lane) * BR, cl);
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) acc = fmaf(cl[kk], PT_s[b * BR + kk], acc);
    }
    q_s[lane] = acc;
  }
  if (lane < NA * L) {
    const int l = lane / NA + 1, nn = lane % NA;
    const float* Sn = S_s + nn * K + l * l - 1;
    float s = 0.f;
#pragma unroll
    for (int m = 0; m < 2 * L + 1; ++m)
      if (m < 2 * l + 1) s = fmaf(Sn[m], Sn[m], s);
    q_s[NR + lane] = s;
    if constexpr (S::F5)
      if (l == 1) q_s[S::OFF5 + nn] = s * s;
  }
  if constexpr (S::F4) {
    if (lane < NA) {
      float s2[5], A[6];
#pragma unroll
      for (int m = 0; m < 5; ++m) s2[m] = S_s[lane * K + 3 + m];
      a_from_s2(s2, A);
      q_s[S::OFF4 + lane] = tr_cube(A);
    }
  }
  lds_fence();

  // ---- network: one hidden unit, then one descriptor, per lane
  const int i = io.orig[p];
  if (io.qout && lane < D) io.qout[(int64_t)i * D + lane] = q_s[lane];
  const float* W0g = params + S::PCR + S::PCA + (int64_t)Zs * S::PMLP;
  const float* b0g = W0g + H * D;
  const float* w1g = b0g + H;
  const float* wt = params + S::PWT + (int64_t)Zs * D * kWave + lane;
  float a = lane < H ? b0g[lane] : 0.f;
#pragma unroll
  for (int d = 0; d < D; ++d) a = fmaf(wt[d * kWave], q_s[d], a);
  const float w1 = lane < H ? w1g[lane] : 0.f;
  const float t = tanh_fast(a);
  t_s[lane] = t;
  w_s[lane] = w1;
  z_s[lane] = w1 * fmaf(-t, t, 1.0f);
  lds_fence();
  float E = w1g[H];
#pragma unroll
  for (int h = 0; h < H; ++h) E = fmaf(w_s[h], t_s[h], E);
  if (lane == 0) {
    io.Ei[i] = E;
    if (io.Eproc) io.Eproc[p] = E;
  }
  if (!want_adjoint) return;
  const float* wd = W0g + (lane < D ? lane : D - 1);
  float Fp = 0.f;
#pragma unroll
  for (int h = 0; h < H; ++h) Fp = fmaf(wd[h * D], z_s[h], Fp);
  if (lane >= NR && lane < D) io.fp[(int64_t)(lane - NR) * ns + p] = Fp;
  lds_fence();
  if (lane < NR) q_s[lane] = Fp;
  lds_fence();
  // radial adjoint atil[b][k] = sum_n dE/dq_n ctil[Z_i][b][n][k]
  if (lane < T * BR) {
    const int b = lane / BR, kk = lane % BR;
    float acc = 0.f;
#pragma unroll
    for (int nn = 0; nn < NR; ++nn) acc = fmaf(q_s[nn], cR[(b * NR + nn) * BR + kk], acc);
    io.aR[((int64_t)b * ns + p) * BR + kk] = acc;
  }
}

// ----------------------------------------------------------------- k_force

// Bound as k_desc_wave.  S is recomputed: g_n is needed for the forces as well,
// so only the sums over the pairs are extra.  3,686 atoms of the Ge-Sb-Te model
// 70 -> 18 us, 18,400 atoms 79 -> 56.
template <class S>
__global__ __launch_bounds__(kWave) void k_force_wave(NepIO io, const float* __restrict__ params) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K;
  constexpr int NG = NA % 2 == 0 ? 2 : 1, NH = NA / NG;  // groups of angular functions, as variant 0
  constexpr int PC = kPairChunk, GW = odd(NA), PW = odd(K), QW = 13;
  constexpr int RW = 7;
  static_assert(BR % 4 == 0, "adjoint rows are read as float4");
  static_assert(PC * NG <= kWave, "a lane per pair and group");
  constexpr int kRad = kWave * RW, kAng = PC * (3 * GW + PW + QW + 3 * NG);
  __shared__ ImageTable itab;
  __shared__ float buf[kRad > kAng ? kRad : kAng];  // radial rows, then the angular chunk
  __shared__ float own_s[T * BR], acc_s[16], kap_s[K], S_s[NA * K], fp_s[S::NANG], psi_s[NA], s4_s[NA * 5];
  float* gS = buf;             // [pair][n] g_n
  float* dS = gS + PC * GW;    // [pair][n] g'_n
  float* zS = dS + PC * GW;    // [pair][n] sum_lm sigma_nlm Praw_lm
  float* pS = zS + PC * GW;    // [pair][lm] Praw
  float* qS = pS + PC * PW;    // [pair] u, 1/d, r, 1, x, hf, dxhf, dfc2, species
  float* fS = qS + PC * QW;    // [group][pair] dE_i/dr_ij of the group

  const int64_t ns = io.n_slots;
  const int64_t p = xcd_tile();
  const int lane = threadIdx.x;
  const int c = io.cfg_of[p];
  if (c < 0) return;
  const float4 xi = io.pos4[p];
  const int Zs = __builtin_amdgcn_readfirstlane(__float_as_int(xi.w));
  const float* __restrict__ dco = params + S::PD;
  itab.fill();
  fill_kappa<L>(kap_s, lane);
  if (lane < T * BR) own_s[lane] = io.aR[((int64_t)(lane / BR) * ns + p) * BR + lane % BR];
  if (lane < S::NANG) fp_s[lane] = io.fp[(int64_t)lane * ns + p];
  float Hc[9];
  load_cell(io.cfgs, c, Hc);
  const float rcR_inv = 1.0f / io.cut.rcR, rcA_inv = 1.0f / io.cut.rcA;
  const int nR = io.ccR[p], nA = io.ccA[p];
  lds_fence();

  // ---- radial pairs: f_ij - f_ji = (s_own + s_rev) u_ij.  Accumulators of
  //      lanes 0..2: force; 3..8: virial xx, yy, zz, xy, xz, yz.  Every term
  //      is the product of two values of the pair's row.
  const int vi = lane < 6 ? lane - 3 : (lane < 8 ? 0 : 1), vj = lane < 6 ? lane - 3 : (lane == 6 ? 1 : 2);
  const int oa = lane < 3 ? 0 : 4 + vi, ob = lane < 3 ? 1 + lane : 1 + vj;
  const float* aRz = io.aR + (int64_t)Zs * ns * BR;
  float acc = 0.f;
  for (int k0 = 0; k0 < nR; k0 += kWave) {
    const int m = nR - k0 < kWave ? nR - k0 : kWave;
    if (lane < m) {
      const uint32_t e = io.cnR[group_index(ns, p, k0 + lane)];
      const PairVec v = pair_vec(e, io.pos4[e & kNbrMask], xi, Hc, itab);
      float ar[BR];
      load_row<BR>(aRz + (int64_t)v.q * BR, ar);
      const float inv = rsqrt_hw(v.d2);
      const RadialFD f = radial_fd(v.d2 * inv * rcR_inv, rcR_inv);
      float Tk[BR], Dk[BR];
      cheb_tt<BR>(f.x, Tk, Dk);
      const float* ao = own_s + (T == 1 ? 0 : v.zj * BR);
      float to = ao[0], dn = 0.f, tr = ar[0], dr = 0.f;
#pragma unroll
      for (int kk = 1; kk < BR; ++kk) {
        to = fmaf(ao[kk], Tk[kk], to);
        dn = fmaf(ao[kk], Dk[kk], dn);
        tr = fmaf(ar[kk], Tk[kk], tr);
        dr = fmaf(ar[kk], Dk[kk], dr);
      }
      const float s_own = fmaf(f.dxhf, dn, f.dfc2 * to);
      const float s_rev = fmaf(f.dxhf, dr, f.dfc2 * tr);
      const float so = s_own * inv;
      float* row = buf + lane * RW;
      row[0] = (s_own + s_rev) * inv;
      row[1] = v.rx;
      row[2] = v.ry;
      row[3] = v.rz;
      row[4] = -(so * v.rx);
      row[5] = -(so * v.ry);
      row[6] = -(so * v.rz);
    }
    lds_fence();
    if (lane < 9) {
#pragma unroll 4
      for (int j = 0; j < m; ++j) acc = fmaf(buf[j * RW + oa], buf[j * RW + ob], acc);
    }
    lds_fence();
  }
  // from here lanes 0..2 hold the force and 3..11 the virial, row-major
  if (lane < 9) acc_s[lane] = acc;
  lds_fence();
  const int wi = (lane - 3) / 3, wj = (lane - 3) % 3;  // virial entry of lanes 3..11
  if (lane >= 3 && lane < 12) {
    const int lo = wi < wj ? wi : wj, hi = wi < wj ? wj : wi;
    acc = acc_s[lo == hi ? 3 + lo : 5 + lo + hi];  // xy, xz, yz at 6, 7, 8
  }

  // ---- angular pairs in chunks: geometry of a pair per lane, then g_n and g'_n
  //      of a (pair, function) per lane; Praw of a pair per lane apart, since
  //      the sums and the forces round dxy differently
  auto harmonics = [&](int m, bool sums) {
    if (lane < m) {
      const float* row = qS + lane * QW;
      float P[K];
      raw_sph<L>(row[0], row[1], row[2],
                 sums ? dxy_sums(row[4], row[1], row[3]) : dxy_force(row[0], row[5], row[3]), P);
#pragma unroll
      for (int lm = 0; lm < K; ++lm) pS[lane * PW + lm] = P[lm];
    }
  };
  auto chunk = [&](int a0, int m) {
    lds_fence();
    if (lane < m) {
      const uint32_t e = io.cnA[group_index(ns, p, a0 + lane)];
      const PairVec v = pair_vec(e, io.pos4[e & kNbrMask], xi, Hc, itab);
      const float inv = rsqrt_hw(v.d2);
      const float ux = v.rx * inv, uy = v.ry * inv, uz = v.rz * inv;
      const RadialFD f = radial_fd(v.d2 * inv * rcA_inv, rcA_inv);
      float* row = qS + lane * QW;
      row[0] = ux;
      row[1] = uy;
      row[2] = uz;
      row[3] = inv;
      row[4] = v.rx;
      row[5] = v.ry;
      row[6] = v.rz;
      row[7] = 1.0f;
      row[8] = f.x;
      row[9] = f.hf;
      row[10] = f.dxhf;
      row[11] = f.dfc2;
      row[12] = __int_as_float(v.zj);
    }
    lds_fence();
    for (int it = lane; it < m * NA; it += kWave) {
      const int j = it / NA, nn = it % NA;
      const float* row = qS + j * QW;
      float Tk[BA], Dk[BA], cl[BA];
      cheb_tt<BA>(row[8], Tk, Dk);
      load_row<BA>(dco + S::PCR + (int64_t)((Zs * T + __float_as_int(row[12])) * NA + nn) * BA, cl);
      float ct = cl[0], cd = 0.f;
#pragma unroll
      for (int kk = 1; kk < BA; ++kk) {
        ct = fmaf(cl[kk], Tk[kk], ct);
        cd = fmaf(cl[kk], Dk[kk], cd);
      }
      gS[j * GW + nn] = row[9] * ct;
      dS[j * GW + nn] = fmaf(row[10], cd, row[11] * ct);
    }
    lds_fence();
  };
  auto chunk_len = [&](int a0) { return nA - a0 < PC ? nA - a0 : PC; };
  if (nA > 0) {
    SumLanes<S> sum;
    sum.zero();
    for (int a0 = 0; a0 < nA; a0 += PC) {
      const int m = chunk_len(a0);
      chunk(a0, m);
      harmonics(m, true);
      lds_fence();
      sum.add(gS, pS, m, lane);
    }
    sum.store(S_s, kap_s, lane);
    lds_fence();
    // sigma = dE_i/dS in place, scaled by kappa: per function first
    if (lane < NA) {
      const float* Sn = S_s + lane * K;
      if constexpr (S::F4) {
        // d tr(A^3)/dS_n2m through A(S): 3 Fp4 A^2 contracted with dA/dS
        float s2[5], A[6], B[6];
#pragma unroll
        for (int m = 0; m < 5; ++m) s2[m] = Sn[3 + m];
        a_from_s2(s2, A);
        sym_sq(A, B);
        float s4[5];
        s4_from_sq(B, 3.0f * fp_s[S::OFF4 - NR + lane], s4);
#pragma unroll
        for (int m = 0; m < 5; ++m) s4_s[lane * 5 + m] = s4[m];
      }
      float psi1 = 2.0f * fp_s[lane];
      if constexpr (S::F5) {
        const float q1 = fmaf(Sn[2], Sn[2], fmaf(Sn[0], Sn[0], Sn[1] * Sn[1]));
        psi1 = fmaf(4.0f * q1, fp_s[S::OFF5 - NR + lane], psi1);
      }
      psi_s[lane] = psi1;
    }
    lds_fence();
    for (int a = lane; a < NA * K; a += kWave) {
      const int nn = a / K, lm = a % K;
      const int l = lm < 3 ? 1 : (lm < 8 ? 2 : (lm < 15 ? 3 : 4));
      const float psi = l == 1 ? psi_s[nn] : 2.0f * fp_s[(l - 1) * NA + nn];
      float s = S_s[a] * psi;
      if constexpr (S::F4)
        if (l == 2) s = fmaf(s4_scale(lm - 3), s4_s[nn * 5 + lm - 3], s);
      S_s[a] = s * kap_s[lm];
    }
    // pair forces of the chunk for groups h0 .. h0 + nh - 1: a (pair,
    // function) per lane for Z_n, then a (pair, group) per lane
    auto forces = [&](int m, int h0, int nh) {
      lds_fence();
      harmonics(m, false);
      lds_fence();
      for (int it = lane; it < m * NA; it += kWave) {
        const int j = it / NA, nn = it % NA;
        float zn = 0.f;
#pragma unroll
        for (int lm = 0; lm < K; ++lm) zn = fmaf(S_s[nn * K + lm], pS[j * PW + lm], zn);
        zS[j * GW + nn] = zn;
      }
      lds_fence();
      const int h = h0 + lane / PC, j = lane % PC;
      if (j < m && h < h0 + nh) {
        const float* row = qS + j * QW;
        const float ux = row[0], uy = row[1], uz = row[2], inv = row[3];
        float G[K];
#pragma unroll
        for (int lm = 0; lm < K; ++lm) G[lm] = 0.f;
        float s = 0.f;
#pragma unroll
        for (int nn = 0; nn < NH; ++nn) {
          const int n = h * NH + nn;
          const float g = gS[j * GW + n];
#pragma unroll
          for (int lm = 0; lm < K; ++lm) G[lm] = fmaf(S_s[n * K + lm], g, G[lm]);
          s = fmaf(dS[j * GW + n], zS[j * GW + n], s);
        }
        float vx, vy, vz;
        raw_sph_grad_dot<L>(ux, uy, uz, dxy_force(ux, row[5], inv), G, vx, vy, vz);
        const float uv = fmaf(ux, vx, fmaf(uy, vy, uz * vz));
        float* f = fS + 3 * (h * PC + j);
        f[0] = fmaf(s, ux, (vx - uv * ux) * inv);
        f[1] = fmaf(s, uy, (vy - uv * uy) * inv);
        f[2] = fmaf(s, uz, (vz - uv * uz) * inv);
      }
      lds_fence();
    };
    // own force and virial of group h over the chunk, in order
    const int fc = lane < 3 ? lane : wi, rc = lane < 3 ? 7 : 4 + wj;
    const float sgn = lane < 3 ? 1.0f : -1.0f;
    auto add = [&](int m, int h) {
      if (lane >= 12) return;
#pragma unroll 4
      for (int j = 0; j < m; ++j) acc = fmaf(sgn * fS[3 * (h * PC + j) + fc], qS[j * QW + rc], acc);
    };
    if (nA <= PC) {
      forces(nA, 0, NG);
#pragma unroll
      for (int h = 0; h < NG; ++h) add(nA, h);
      if (lane < nA) {
        float4 f = make_float4(fS[3 * lane], fS[3 * lane + 1], fS[3 * lane + 2], 0.f);
#pragma unroll
        for (int h = 1; h < NG; ++h) {
          const float* g = fS + 3 * (h * PC + lane);
          f = make_float4(f.x + g[0], f.y + g[1], f.z + g[2], 0.f);
        }
        io.fA[(int64_t)lane * ns + p] = f;
      }
    } else {
      for (int h = 0; h < NG; ++h)
        for (int a0 = 0; a0 < nA; a0 += PC) {
          const int m = chunk_len(a0);
          chunk(a0, m);
          forces(m, h, 1);
          add(m, h);
          if (lane < m) {
            const float* g = fS + 3 * (h * PC + lane);
            float4* slot = io.fA + (int64_t)(a0 + lane) * ns + p;
            const float4 o = h == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : *slot;
            *slot = h == 0 ? make_float4(g[0], g[1], g[2], 0.f) : make_float4(o.x + g[0], o.y + g[1], o.z + g[2], 0.f);
          }
        }
    }
  }
  float* fr = reinterpret_cast<float*>(io.frad + p);
  if (lane < 3) fr[lane] = acc;
  if (lane == 12) fr[3] = 0.f;
  if (lane >= 3 && lane < 12) io.Wi[(int64_t)io.orig[p] * 9 + lane - 3] = acc;
}

template <class S>
int WaveLaunch<S>::desc(hipStream_t st, const NepIO& io, const float* params, bool want_adjoint) {
  hipLaunchKernelGGL(k_desc_wave<S>, dim3((unsigned)io.n_slots + (io.mail.mail ? 1 : 0)), dim3(kWave), 0, st, io, params, want_adjoint ? 1 : 0);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template <class S>
int WaveLaunch<S>::force(hipStream_t st, const NepIO& io, const float* params) {
  hipLaunchKernelGGL(k_force_wave<S>, dim3((unsigned)io.n_slots), dim3(kWave), 0, st, io, params);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template struct WaveLaunch<ShapeSmall>;
template struct WaveLaunch<ShapeGST>;
template struct WaveLaunch<ShapeTable2>;

}  // namespace nepmi
