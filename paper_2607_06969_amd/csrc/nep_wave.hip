// nep_wave.hip -- descriptor/network and pair-force kernels with a group of lanes
// per atom, a whole wavefront or half of one, for batches too small to fill the
// chip with one thread per atom.
//
// A thread that owns an atom walks its lists entry by entry; below some 30,000
// atoms the chip then holds less than half a wavefront per SIMD and the time is
// that of one walk.  Here the W lanes of a group take the pairs of one atom
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
//
// The groups of a wavefront run in step: what one of them decides for itself
// (pairs kept, list lengths) lies in its lanes, and loops with an LDS hand-over
// run until the last group is done.  Its slots are of one species (see nbr.hip).
#include "nep_device.hpp"
#include "nbr.hpp"

namespace nepmi {

// A ballot over the lanes of a group, its size and this lane's rank in it.
template <int W>
struct GroupBallot {
  uint64_t m;  // of the wavefront
  __device__ __forceinline__ explicit GroupBallot(bool b) : m(__ballot(b)) {}
  // the group's part, lane 0 of the group in bit 0
  __device__ __forceinline__ uint64_t bits() const {
    if constexpr (W == kWave) return m;
    return (threadIdx.x & 32) ? (uint32_t)(m >> 32) : (uint32_t)m;
  }
  __device__ __forceinline__ int count() const {
    if constexpr (W == kWave) return __builtin_popcountll(m);
    return __builtin_popcount((uint32_t)bits());
  }
  __device__ __forceinline__ int rank() const {
    const uint32_t lo = __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u);
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), W == kWave || !(threadIdx.x & 32) ? lo : 0u);
  }
};
// The largest of the groups' values (the same in all lanes of a group), uniform.
template <int W>
__device__ __forceinline__ int over_groups(int v) {
  const int a = __builtin_amdgcn_readlane(v, 0);
  if constexpr (W == kWave) return a;
  const int b = __builtin_amdgcn_readlane(v, 32);
  return a > b ? a : b;
}

// Angular pairs of an atom held in LDS at a time.
template <int W>
constexpr int pair_chunk() {
  return W / 2;
}
constexpr int odd(int n) { return n | 1; }  // row strides that spread a column over the banks

// The harmonics' constants, for lanes to read their own.
template <int L>
static __device__ const Kappa<L> kKappa = Kappa<L>();

// Rows of the angular pairs in LDS, read as float4: g_n of a pair, and Praw_lm
// (padded to 4 floats more than a multiple of 8, which spreads 16-byte accesses
// of consecutive rows over the banks).
template <class S>
struct PairRows {
  static constexpr int GW = (S::NA + 3) / 4 * 4, PW = (S::K + 7) / 8 * 8 + 4;
  static __device__ __forceinline__ void put(float* row, const float (&P)[S::K]) {
    static_assert(S::K % 4 == 0, "rows of float4");
#pragma unroll
    for (int q = 0; q < S::K / 4; ++q)
      reinterpret_cast<float4*>(row)[q] = make_float4(P[4 * q], P[4 * q + 1], P[4 * q + 2], P[4 * q + 3]);
  }
};

// S_nlm accumulators of a group: a lane has one lm and R functions n, from n0 on.
template <class S, int W>
struct SumLanes {
  static constexpr int Q = W / S::K, R = S::NA / Q;  // lanes per lm, functions per lane
  static_assert(Q >= 1 && S::NA % Q == 0, "whole functions per lane");
  float v[R], kap;
  int lm, n0;
  bool own;  // lanes past the last accumulator repeat others'
  __device__ __forceinline__ explicit SumLanes(int l) {
    lm = l % S::K;
    own = l / S::K < Q;
    n0 = (own ? l / S::K : Q - 1) * R;
    kap = kKappa<S::L>.v[lm];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = 0.f;
  }
  // add pairs 0 .. n - 1 of the chunk in order (gS, pS: rows per pair)
  __device__ __forceinline__ void add(const float* gS, const float* pS, int n) {
    const float *g = gS + n0, *P = pS + lm;
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
      const float y = P[j * PairRows<S>::PW];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = fmaf(g[j * PairRows<S>::GW + r], y, v[r]);
    }
  }
  // apply the harmonics' constants and store [n][lm]
  __device__ __forceinline__ void store(float* sS) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] *= kap;
      if (own) sS[(n0 + r) * S::K + lm] = v[r];
    }
  }
};

// add(w_k, k) for k < N in order, w four at a time from rows of 64 lanes.  U rows
// are loaded at once (with two atoms per lane all of them would take more
// registers than four wavefronts per SIMD leave).
template <int N, int U, class F>
__device__ __forceinline__ void dot4(const float4* __restrict__ w, F&& add) {
  constexpr int Q = N / 4;
#pragma unroll U
  for (int q = 0; q < Q; ++q) {
    const float4 v = w[q * kWave];
    add(v.x, 4 * q);
    add(v.y, 4 * q + 1);
    add(v.z, 4 * q + 2);
    add(v.w, 4 * q + 3);
  }
  if constexpr (N % 4 != 0) {
    const float4 v = w[Q * kWave];
#pragma unroll
    for (int u = 0; u < N % 4; ++u) add(comp4(v, u), 4 * Q + u);
  }
}

// The atoms of a wavefront: group g of W lanes has slot p0 + g.
template <int W>
struct GroupAtom {
  int g, l;      // group, lane in it
  int64_t p, pa; // slot (may lie past the end), slot to read from (an atom's)
  bool act;      // the slot holds an atom
};
template <int W>
__device__ __forceinline__ bool group_atom(const NepIO& io, int64_t p0, bool none, GroupAtom<W>& a) {
  a.g = W == kWave ? 0 : (int)threadIdx.x / W;
  a.l = W == kWave ? (int)threadIdx.x : (int)threadIdx.x % W;
  a.p = p0 + a.g;
  a.act = a.p < io.n_slots && io.cfg_of[a.p < io.n_slots ? a.p : io.n_slots - 1] >= 0 && !none;
  const uint64_t m = __ballot(a.act);
  if (!m) return false;
  a.pa = a.act ? a.p : p0 + __builtin_ctzll(m) / W;
  return true;
}

// ------------------------------------------------------------------ k_desc

// Latency bounds it, at four wavefronts per SIMD, and issue (an atom of the
// Ge-Sb-Te model has some 29 radial and 8 angular pairs for the 32 or 64 lanes),
// not the 1.3 KB it moves per atom.  3,686 atoms of that model, one thread, 64, 32
// lanes per atom: 56, 13.2, 12.4 us; 18,400 atoms 61, 48.2, 36.8.  Left to the
// compiler, the registers of the 32-lane form allow two wavefronts: 52.
template <class S, int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_desc_wave(NepIO io, const float* __restrict__ params, int want_adjoint) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K, D = S::D, H = S::H;
  constexpr int G = kWave / W;
  constexpr int RW = odd(BR + 1);  // radial row: T_k, then f_c / 2
  constexpr int PC = pair_chunk<W>(), GW = PairRows<S>::GW, PW = PairRows<S>::PW;
  static_assert(D <= kWave && H <= kWave && NR <= W && NA <= W, "one lane each");
  constexpr int kRad = W * RW, kAng = PC * (GW + PW + 3);
  constexpr int UW = W == kWave ? 16 : 7;
  constexpr int RR = (T * BR + W - 1) / W;  // radial accumulators per lane
  static_assert(T * BR + NA * K <= kAng, "the sums take the place of the pairs");
  struct __align__(16) Atom {
    float buf[(kRad > kAng ? kRad : kAng) + 3 & ~3];  // radial rows, the angular chunk, the sums
    float angr[2 * kWave > W * 5 ? 2 * kWave : W * 5];  // r_ij, |r|^2, species of the angular pairs found;
                                                        // then tanh and z = w1 (1 - tanh^2) per hidden unit
    int part[W];
    uint32_t last[3];                      // last radial and angular entry, last reverse position
  };
  __shared__ Atom atoms[G];
  __shared__ ImageTable itab;
  __shared__ __align__(16) float q_s[G][kWave], w_s[kWave];

  const int64_t ns = io.n_slots;
  const int64_t p0 = xcd_tile() * G;
  if (p0 >= ns) {  // the block past the last slot (there only for the flags)
    if (threadIdx.x == 0) deliver(io.mail);
    return;
  }
  GroupAtom<W> at;
  if (!group_atom(io, p0, lists_void(io.stop), at)) {
    if (at.l == 0 && at.p < ns) io.ccR[at.p] = io.ccA[at.p] = 0;
    return;
  }
  const int64_t p = at.pa;
  const int lane = threadIdx.x, l = at.l;
  Atom& A = atoms[at.g];
  float* buf = A.buf;
  float* gS = buf;                 // [pair][n] g_n
  float* pS = gS + PC * GW;        // [pair][lm] Praw
  float* xS = pS + PC * PW;        // x, f_c / 2 and species per pair
  float* hS = xS + PC;
  float* cS = hS + PC;
  const float4 xi = io.pos4[p];
  const int Zs = __builtin_amdgcn_readfirstlane(__float_as_int(xi.w));
  const float* __restrict__ dco = params + S::PD;
  itab.fill();
  float Hc[9];
  load_cell(io.cfgs, io.cfg_of[p], Hc);
  const float rcR_inv = 1.0f / io.cut.rcR, rcA_inv = 1.0f / io.cut.rcA;
  const int n = at.act ? io.cntR[p] : 0;
  // entries the mask's words hold (a list cut off at its capacity, as MD may step
  // with until its chunk of steps is undone, may have more)
  const int kaMax = (io.capA + 63) / 64 * 64;
  wave_fence();

  // ---- filter the Verlet list into the pairs inside the two cutoffs, W
  //      entries per round; accumulator (b, k) = b B_R + k sums the radial
  //      neighbours of species b in list order
  float PT[RR];
#pragma unroll
  for (int r = 0; r < RR; ++r) PT[r] = 0.f;
  SumLanes<S, W> sum(l);
  int nR = 0, nA = 0, ka0 = 0;  // pairs kept, entries of the angular part seen
  uint64_t mword = 0;           // entry mask of the angular part, 64 entries per word
  bool bad = false;
  const int n_most = over_groups<W>(n);
  for (int k0 = 0; k0 < n_most; k0 += W) {
    const int k = k0 + l;
    const bool valid = k < n;
    uint32_t e = (uint32_t)p, rv = 0xFFFFFFFFu;  // past the end: the atom itself
    if (valid) {
      const int64_t gi = group_index(ns, p, k);
      e = io.nbrR[gi];
      rv = io.vrev[gi];
    }
    const PairVec v = pair_vec(e, io.pos4[e & kNbrMask], xi, Hc, itab);
    const bool inR = valid && v.d2 < io.cut.rcR2;
    const bool part = rv != 0xFFFFFFFFu;
    const bool inA = inR && v.d2 < io.cut.rcA2;
    const GroupBallot<W> mR(inR), mP(part), mV(inA && rv <= 0xFFFFu);
    const int kr = mR.rank(), kp = mP.rank(), kA = mV.rank();
    // within rc_angular now implies within rc_angular + skin at the last
    // build, so nA stays below capA and the reverse row exists
    const bool okA = inA && rv <= 0xFFFFu && nA + kA < io.capA;
    bad |= inA && !okA;
    const GroupBallot<W> mA(okA);
    const uint32_t pr = (uint32_t)(ka0 + kp) | (rv << 16);
    const int cR = mR.count(), cA = mA.count();
    // rows by species, in list order (each accumulator then runs over its own)
    int row_of = kr, first[T], count[T];
    first[0] = 0;
    count[0] = cR;
    if constexpr (T > 1) {
      int rows = 0;
#pragma unroll
      for (int b = 0; b < T; ++b) {
        const GroupBallot<W> mb(inR && v.zj == b);
        if (v.zj == b) row_of = rows + mb.rank();
        first[b] = rows;
        count[b] = mb.count();
        rows += count[b];
      }
    }
    if (inR) {
      io.cnR[group_index(ns, p, nR + kr)] = e;
      if (kr == cR - 1) A.last[0] = e;
      const float inv = rsqrt_hw(v.d2);
      const RadialF f = radial_f(v.d2 * inv * rcR_inv);
      float Tk[BR];
      cheb_t<BR>(f.x, Tk);
      float* row = buf + row_of * RW;
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) row[kk] = Tk[kk];
      row[BR] = f.hf;
    }
    if (okA) {
      io.cnA[group_index(ns, p, nA + kA)] = e;
      io.cpA[group_index(ns, p, nA + kA)] = pr;
      if (kA == cA - 1) {
        A.last[1] = e;
        A.last[2] = pr;
      }
      float* row = A.angr + kA * 5;
      row[0] = v.rx;
      row[1] = v.ry;
      row[2] = v.rz;
      row[3] = v.d2;
      row[4] = __int_as_float(v.zj);
    }
    if (part) A.part[kp] = okA ? 1 : 0;
    wave_fence();
    // the mask bits of this round's entries of the angular part, appended
    const int np = mP.count();
    const uint64_t bits = GroupBallot<W>(l < np && A.part[l] != 0).bits();
    const int sh = ka0 & 63;
    mword |= bits << sh;
    if ((ka0 + np) >> 6 != ka0 >> 6) {
      if (l == 0 && ka0 < kaMax) io.amask[(int64_t)(ka0 >> 6) * ns + p] = mword;
      mword = sh ? bits >> (64 - sh) : 0;
    }
    ka0 += np;
    nR += cR;
    nA += cA;
#pragma unroll
    for (int r = 0; r < RR; ++r) {
      const int a = l + W * r, b = a / BR;
      int j0 = 0, nj = 0;
#pragma unroll
      for (int x = 0; x < T; ++x)
        if (b == x) {
          j0 = first[x];
          nj = count[x];
        }
      const float* row = buf + j0 * RW;
#pragma unroll 4
      for (int j = 0; j < nj; ++j) PT[r] = fmaf(row[j * RW + BR], row[j * RW + a % BR], PT[r]);
    }
    wave_fence();
    // the angular pairs of this round: S_nlm = sum_j g_n(r_ij) Y_lm(u_ij)
    const int most = over_groups<W>(cA);
    for (int a0 = 0; a0 < most; a0 += PC) {
      const int m = cA - a0 < PC ? cA - a0 : PC;
      if (l < m) {
        const float* row = A.angr + (a0 + l) * 5;
        const float inv = rsqrt_hw(row[3]);
        const RadialF f = radial_f(row[3] * inv * rcA_inv);
        float P[K];
        const float uy = row[1] * inv;
        raw_sph<L>(row[0] * inv, uy, row[2] * inv, dxy_sums(row[0], uy, inv), P);
        PairRows<S>::put(pS + l * PW, P);
        xS[l] = f.x;
        hS[l] = f.hf;
        cS[l] = row[4];
      }
      wave_fence();
      for (int it = l; it < m * NA; it += W) {
        const int j = it / NA, nn = it % NA;
        float Tk[BA], cl[BA];
        cheb_t<BA>(xS[j], Tk);
        load_row<BA>(dco + S::PCR + (int64_t)((Zs * T + __float_as_int(cS[j])) * NA + nn) * BA, cl);
        float acc = 0.f;
#pragma unroll
        for (int kk = 0; kk < BA; ++kk) acc = fmaf(cl[kk], Tk[kk], acc);
        gS[j * GW + nn] = hS[j] * acc;
      }
      wave_fence();
      sum.add(gS, pS, m);
      wave_fence();
    }
  }
  // the last, partly filled mask word and groups (they repeat the last entry)
  if (l == 0) {
    if ((ka0 & 63) && ka0 < kaMax) io.amask[(int64_t)(ka0 >> 6) * ns + p] = mword;
    if (at.p < ns) {
      io.ccR[at.p] = nR;
      io.ccA[at.p] = nA;
    }
  }
  if ((nR & 3) && l < 4 - (nR & 3)) io.cnR[group_index(ns, p, nR + l)] = A.last[0];
  if ((nA & 3) && l < 4 - (nA & 3)) {
    io.cnA[group_index(ns, p, nA + l)] = A.last[1];
    io.cpA[group_index(ns, p, nA + l)] = A.last[2];
  }
  if (bad) atomicOr(&io.flags[kFlagLate], 1);

  // ---- descriptors, Eq. 11, 16, 17
  float* PT_s = buf;            // [b][k]
  float* S_s = buf + T * BR;    // [n][lm]
  float* q = q_s[at.g];
#pragma unroll
  for (int r = 0; r < RR; ++r)
    if (l + W * r < T * BR) PT_s[l + W * r] = PT[r];
  sum.store(S_s);
  wave_fence();
  const float* cR = dco + (int64_t)Zs * (T * NR * BR);
  if (l < NR) {
    float acc = 0.f;
#pragma unroll
    for (int b = 0; b < T; ++b) {
      float cl[BR];
      load_row<BR>(cR + (b * NR + l) * BR, cl);
#pragma unroll
      for (int kk = 0; kk < BR; ++kk) acc = fmaf(cl[kk], PT_s[b * BR + kk], acc);
    }
    q[l] = acc;
  }
  for (int it = l; it < NA * L; it += W) {
    const int ll = it / NA + 1, nn = it % NA;
    const float* Sn = S_s + nn * K + ll * ll - 1;
    float s = 0.f;
#pragma unroll
    for (int m = 0; m < 2 * L + 1; ++m)
      if (m < 2 * ll + 1) s = fmaf(Sn[m], Sn[m], s);
    q[NR + it] = s;
    if constexpr (S::F5)
      if (ll == 1) q[S::OFF5 + nn] = s * s;
  }
  if constexpr (S::F4) {
    if (l < NA) {
      float s2[5], B[6];
#pragma unroll
      for (int m = 0; m < 5; ++m) s2[m] = S_s[l * K + 3 + m];
      a_from_s2(s2, B);
      q[S::OFF4 + l] = tr_cube(B);
    }
  }
  wave_fence();

  // ---- network: one hidden unit, then one descriptor, of every atom per lane
  const int i = io.orig[p];
  if (io.qout) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int ig = __builtin_amdgcn_readlane(at.act ? i : -1, g * W);
      if (ig >= 0 && lane < D) io.qout[(int64_t)ig * D + lane] = q_s[g][lane];
    }
  }
  const float* W0g = params + S::PCR + S::PCA + (int64_t)Zs * S::PMLP;
  const float* b0g = W0g + H * D;
  const float* w1g = b0g + H;
  // both layers' weights of this lane four at a time: W0[lane][.], W0[.][lane]
  const float4* wt = reinterpret_cast<const float4*>(params + S::PWT) + (int64_t)Zs * (S::WQ * kWave) + lane;
  float a[G];
  a[0] = lane < H ? b0g[lane] : 0.f;
#pragma unroll
  for (int g = 1; g < G; ++g) a[g] = a[0];
  dot4<D, UW>(wt, [&](float w, int d) {
#pragma unroll
    for (int g = 0; g < G; ++g) a[g] = fmaf(w, q_s[g][d], a[g]);
  });
  const float w1 = lane < H ? w1g[lane] : 0.f;
  w_s[lane] = w1;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float t = tanh_fast(a[g]);
    atoms[g].angr[lane] = t;
    atoms[g].angr[kWave + lane] = w1 * fmaf(-t, t, 1.0f);
  }
  wave_fence();
  float E = w1g[H];
#pragma unroll 25
  for (int h = 0; h < H; ++h) E = fmaf(w_s[h], A.angr[h], E);
  if (l == 0 && at.act) {
    io.Ei[i] = E;
    if (io.Eproc) io.Eproc[p] = E;
  }
  if (!want_adjoint) return;
  wt += (D + 3) / 4 * kWave;
  float Fp[G];
#pragma unroll
  for (int g = 0; g < G; ++g) Fp[g] = 0.f;
  dot4<H, UW>(wt, [&](float w, int h) {
#pragma unroll
    for (int g = 0; g < G; ++g) Fp[g] = fmaf(w, atoms[g].angr[kWave + h], Fp[g]);
  });
  wave_fence();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    if (lane >= NR && lane < D && p0 + g < ns) io.fp[(int64_t)(lane - NR) * ns + p0 + g] = Fp[g];
    if (lane < NR) q_s[g][lane] = Fp[g];
  }
  wave_fence();
  // radial adjoint atil[b][k] = sum_n dE/dq_n ctil[Z_i][b][n][k]
  for (int it = l; it < T * BR; it += W) {
    const int b = it / BR, kk = it % BR;
    float acc = 0.f;
#pragma unroll
    for (int nn = 0; nn < NR; ++nn) acc = fmaf(q[nn], cR[(b * NR + nn) * BR + kk], acc);
    if (at.act) io.aR[((int64_t)b * ns + p) * BR + kk] = acc;
  }
}

// ----------------------------------------------------------------- k_force

// Bound as k_desc_wave.  S is recomputed: g_n is needed for the forces as well,
// so only the sums over the pairs are extra.  3,686 atoms of the Ge-Sb-Te model,
// one thread, 64, 32 lanes per atom: 70, 17.3, 11.5 us; 18,400 atoms 79, 56.6,
// 36.8.
template <class S, int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_force_wave(NepIO io, const float* __restrict__ params) {
  constexpr int T = S::T, NR = S::NR, NA = S::NA, BR = S::BR, BA = S::BA, L = S::L, K = S::K;
  constexpr int G = kWave / W;
  constexpr int NG = NA % 2 == 0 ? 2 : 1, NH = NA / NG;  // groups of angular functions, as variant 0
  constexpr int PC = pair_chunk<W>(), GW = PairRows<S>::GW, PW = PairRows<S>::PW, QW = 13, ZW = odd(NA);
  constexpr int RW = 7;
  static_assert(BR % 4 == 0, "adjoint rows are read as float4");
  static_assert(PC * NG <= W && 3 * NG <= PW && 13 <= W && NA <= W, "a lane per pair and group");
  constexpr int kRad = W * RW, kAng = PC * (GW + 2 * ZW + PW + QW);
  static_assert(kRad + T * BR + 16 <= kAng && 6 * NA <= PC * PW, "shared room");
  struct __align__(16) Atom {
    float buf[(kRad > kAng ? kRad : kAng) + 3 & ~3];  // radial rows, then the angular chunk
    float S_[NA * K], fp[S::NANG];
  };
  __shared__ Atom atoms[G];
  __shared__ ImageTable itab;

  const int64_t ns = io.n_slots;
  GroupAtom<W> at;
  const bool none = lists_void(io.stop);
  if (!group_atom(io, xcd_tile() * G, false, at)) return;
  const int64_t p = at.pa;
  const int l = at.l;
  Atom& A = atoms[at.g];
  float* buf = A.buf;
  float *S_s = A.S_, *fp_s = A.fp;
  float *own_s = buf + kRad, *acc_s = own_s + T * BR;  // of the radial pairs
  float* gS = buf;             // [pair][n] g_n
  float* pS = gS + PC * GW;    // [pair][lm] Praw
  float* dS = pS + PC * PW;    // [pair][n] g'_n
  float* zS = dS + PC * ZW;    // [pair][n] sum_lm sigma_nlm Praw_lm
  float* qS = zS + PC * ZW;    // [pair] u, 1/d, r, 1, x, hf, dxhf, dfc2, species
  float* fS = pS;              // [group][pair] dE_i/dr_ij of the group (Praw is spent by then)
  float *psi_s = pS, *s4_s = psi_s + NA;  // of the sums (between two uses of Praw)
  const float4 xi = io.pos4[p];
  const int Zs = __builtin_amdgcn_readfirstlane(__float_as_int(xi.w));
  const float* __restrict__ dco = params + S::PD;
  itab.fill();
  for (int it = l; it < T * BR; it += W) own_s[it] = io.aR[((int64_t)(it / BR) * ns + p) * BR + it % BR];
  for (int it = l; it < S::NANG; it += W) fp_s[it] = io.fp[(int64_t)it * ns + p];
  float Hc[9];
  load_cell(io.cfgs, io.cfg_of[p], Hc);
  const float rcR_inv = 1.0f / io.cut.rcR, rcA_inv = 1.0f / io.cut.rcA;
  const int nR = at.act ? io.ccR[p] : 0, nA = at.act ? io.ccA[p] : 0;
  wave_fence();

  // ---- radial pairs: f_ij - f_ji = (s_own + s_rev) u_ij.  Accumulators of
  //      lanes 0..2: force; 3..8: virial xx, yy, zz, xy, xz, yz.  Every term
  //      is the product of two values of the pair's row.
  const int vi = l < 6 ? l - 3 : (l < 8 ? 0 : 1), vj = l < 6 ? l - 3 : (l == 6 ? 1 : 2);
  const int oa = l < 3 ? 0 : 4 + vi, ob = l < 3 ? 1 + l : 1 + vj;
  const float* aRz = io.aR + (int64_t)Zs * ns * BR;
  float acc = 0.f;
  const int nR_most = over_groups<W>(nR);
  for (int k0 = 0; k0 < nR_most; k0 += W) {
    const int m = nR - k0 < W ? nR - k0 : W;
    if (l < m) {
      const uint32_t e = io.cnR[group_index(ns, p, k0 + l)];
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
      float* row = buf + l * RW;
      row[0] = (s_own + s_rev) * inv;
      row[1] = v.rx;
      row[2] = v.ry;
      row[3] = v.rz;
      row[4] = -(so * v.rx);
      row[5] = -(so * v.ry);
      row[6] = -(so * v.rz);
    }
    wave_fence();
    if (l < 9) {
#pragma unroll 4
      for (int j = 0; j < m; ++j) acc = fmaf(buf[j * RW + oa], buf[j * RW + ob], acc);
    }
    wave_fence();
  }
  // from here lanes 0..2 hold the force and 3..11 the virial, row-major
  if (l < 9) acc_s[l] = acc;
  wave_fence();
  const int wi = (l - 3) / 3, wj = (l - 3) % 3;  // virial entry of lanes 3..11
  if (l >= 3 && l < 12) {
    const int lo = wi < wj ? wi : wj, hi = wi < wj ? wj : wi;
    acc = acc_s[lo == hi ? 3 + lo : 5 + lo + hi];  // xy, xz, yz at 6, 7, 8
  }

  // ---- angular pairs in chunks: geometry of a pair per lane, then g_n and g'_n
  //      of a (pair, function) per lane; Praw of a pair per lane apart, since
  //      the sums and the forces round dxy differently
  auto harmonics = [&](int m, bool sums) {
    if (l < m) {
      const float* row = qS + l * QW;
      float P[K];
      raw_sph<L>(row[0], row[1], row[2],
                 sums ? dxy_sums(row[4], row[1], row[3]) : dxy_force(row[0], row[5], row[3]), P);
      PairRows<S>::put(pS + l * PW, P);
    }
  };
  auto chunk = [&](int a0, int m) {
    wave_fence();
    if (l < m) {
      const uint32_t e = io.cnA[group_index(ns, p, a0 + l)];
      const PairVec v = pair_vec(e, io.pos4[e & kNbrMask], xi, Hc, itab);
      const float inv = rsqrt_hw(v.d2);
      const float ux = v.rx * inv, uy = v.ry * inv, uz = v.rz * inv;
      const RadialFD f = radial_fd(v.d2 * inv * rcA_inv, rcA_inv);
      float* row = qS + l * QW;
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
    wave_fence();
    for (int it = l; it < m * NA; it += W) {
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
      dS[j * ZW + nn] = fmaf(row[10], cd, row[11] * ct);
    }
    wave_fence();
  };
  auto chunk_len = [&](int a0) { return nA - a0 < PC ? nA - a0 : PC; };
  const int nA_most = over_groups<W>(nA);
  if (nA_most > 0) {
    SumLanes<S, W> sum(l);
    for (int a0 = 0; a0 < nA_most; a0 += PC) {
      const int m = chunk_len(a0);
      chunk(a0, m);
      harmonics(m, true);
      wave_fence();
      sum.add(gS, pS, m);
    }
    sum.store(S_s);
    wave_fence();
    // sigma = dE_i/dS in place, scaled by kappa: per function first
    if (l < NA) {
      const float* Sn = S_s + l * K;
      if constexpr (S::F4) {
        // d tr(A^3)/dS_n2m through A(S): 3 Fp4 A^2 contracted with dA/dS
        float s2[5], M[6], B[6];
#pragma unroll
        for (int m = 0; m < 5; ++m) s2[m] = Sn[3 + m];
        a_from_s2(s2, M);
        sym_sq(M, B);
        float s4[5];
        s4_from_sq(B, 3.0f * fp_s[S::OFF4 - NR + l], s4);
#pragma unroll
        for (int m = 0; m < 5; ++m) s4_s[l * 5 + m] = s4[m];
      }
      float psi1 = 2.0f * fp_s[l];
      if constexpr (S::F5) {
        const float q1 = fmaf(Sn[2], Sn[2], fmaf(Sn[0], Sn[0], Sn[1] * Sn[1]));
        psi1 = fmaf(4.0f * q1, fp_s[S::OFF5 - NR + l], psi1);
      }
      psi_s[l] = psi1;
    }
    wave_fence();
    if (sum.own) {
      const int lm = sum.lm, ll = lm < 3 ? 1 : (lm < 8 ? 2 : (lm < 15 ? 3 : 4));
#pragma unroll
      for (int r = 0; r < SumLanes<S, W>::R; ++r) {
        const int nn = sum.n0 + r;
        const float psi = ll == 1 ? psi_s[nn] : 2.0f * fp_s[(ll - 1) * NA + nn];
        float s = sum.v[r] * psi;
        if constexpr (S::F4)
          if (ll == 2) s = fmaf(s4_scale(lm - 3), s4_s[nn * 5 + lm - 3], s);
        S_s[nn * K + lm] = s * sum.kap;
      }
    }
    // pair forces of the chunk for groups h0 .. h0 + nh - 1: a (pair,
    // function) per lane for Z_n, then a (pair, group) per lane
    auto forces = [&](int m, int h0, int nh) {
      wave_fence();
      harmonics(m, false);
      wave_fence();
      for (int it = l; it < m * NA; it += W) {
        const int j = it / NA, nn = it % NA;
        float zn = 0.f;
#pragma unroll
        for (int lm = 0; lm < K; ++lm) zn = fmaf(S_s[nn * K + lm], pS[j * PW + lm], zn);
        zS[j * ZW + nn] = zn;
      }
      wave_fence();
      const int h = h0 + l / PC, j = l % PC;
      if (j < m && h < h0 + nh) {
        const float* row = qS + j * QW;
        const float ux = row[0], uy = row[1], uz = row[2], inv = row[3];
        float Gm[K];
#pragma unroll
        for (int lm = 0; lm < K; ++lm) Gm[lm] = 0.f;
        float s = 0.f;
#pragma unroll
        for (int nn = 0; nn < NH; ++nn) {
          const int n = h * NH + nn;
          const float g = gS[j * GW + n];
#pragma unroll
          for (int lm = 0; lm < K; ++lm) Gm[lm] = fmaf(S_s[n * K + lm], g, Gm[lm]);
          s = fmaf(dS[j * ZW + n], zS[j * ZW + n], s);
        }
        float vx, vy, vz;
        raw_sph_grad_dot<L>(ux, uy, uz, dxy_force(ux, row[5], inv), Gm, vx, vy, vz);
        const float uv = fmaf(ux, vx, fmaf(uy, vy, uz * vz));
        float* f = fS + 3 * (h * PC + j);
        f[0] = fmaf(s, ux, (vx - uv * ux) * inv);
        f[1] = fmaf(s, uy, (vy - uv * uy) * inv);
        f[2] = fmaf(s, uz, (vz - uv * uz) * inv);
      }
      wave_fence();
    };
    // own force and virial of group h over the chunk, in order
    const int fc = l < 3 ? l : wi, rc = l < 3 ? 7 : 4 + wj;
    const float sgn = l < 3 ? 1.0f : -1.0f;
    auto add = [&](int m, int h) {
      if (l >= 12) return;
#pragma unroll 4
      for (int j = 0; j < m; ++j) acc = fmaf(sgn * fS[3 * (h * PC + j) + fc], qS[j * QW + rc], acc);
    };
    if (nA_most <= PC) {
      forces(nA, 0, NG);
#pragma unroll
      for (int h = 0; h < NG; ++h) add(nA, h);
      if (l < nA) {
        float4 f = make_float4(fS[3 * l], fS[3 * l + 1], fS[3 * l + 2], 0.f);
#pragma unroll
        for (int h = 1; h < NG; ++h) {
          const float* g = fS + 3 * (h * PC + l);
          f = make_float4(f.x + g[0], f.y + g[1], f.z + g[2], 0.f);
        }
        io.fA[(int64_t)l * ns + p] = f;
      }
    } else {
      for (int h = 0; h < NG; ++h)
        for (int a0 = 0; a0 < nA_most; a0 += PC) {
          const int m = chunk_len(a0);
          chunk(a0, m);
          forces(m, h, 1);
          add(m, h);
          if (l < m) {
            const float* g = fS + 3 * (h * PC + l);
            float4* slot = io.fA + (int64_t)(a0 + l) * ns + p;
            const float4 o = h == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : *slot;
            *slot = h == 0 ? make_float4(g[0], g[1], g[2], 0.f) : make_float4(o.x + g[0], o.y + g[1], o.z + g[2], 0.f);
          }
        }
    }
  }
  if (!at.act) return;
  float* fr = reinterpret_cast<float*>(io.frad + p);
  if (l < 3) fr[l] = acc;
  if (l == 12) fr[3] = 0.f;
  if (l >= 3 && l < 12 && !none) io.Wi[(int64_t)io.orig[p] * 9 + l - 3] = acc;
}

// Lanes per atom: half a wavefront if it holds the angular pairs of nearly every
// atom in one chunk (16 pairs, at most 11 on average), else a whole one: beyond a
// chunk the forces take the pairs chunk by chunk and group by group.  The Ge-Sb-Te
// model has 8 at the density of its solids (18,400 atoms, k_desc + k_force: 105 us
// with 64 lanes, 74 with 32), the model of Table 2 has 16.
static bool half_wave(const NepIO& io) { return io.pairsA <= 11.0f; }

template <class S, int W>
static void launch_desc_wave(hipStream_t st, const NepIO& io, const float* params, bool want_adjoint) {
  constexpr int G = kWave / W;
  const unsigned tiles = (unsigned)((io.n_slots + G - 1) / G);
  hipLaunchKernelGGL((k_desc_wave<S, W>), dim3(tiles + (io.mail.mail ? 1 : 0)), dim3(kWave), 0, st, io, params,
                     want_adjoint ? 1 : 0);
}

template <class S, int W>
static void launch_force_wave(hipStream_t st, const NepIO& io, const float* params) {
  constexpr int G = kWave / W;
  hipLaunchKernelGGL((k_force_wave<S, W>), dim3((unsigned)((io.n_slots + G - 1) / G)), dim3(kWave), 0, st, io, params);
}

template <class S>
int WaveLaunch<S>::desc(hipStream_t st, const NepIO& io, const float* params, bool want_adjoint) {
  (half_wave(io) ? launch_desc_wave<S, 32> : launch_desc_wave<S, kWave>)(st, io, params, want_adjoint);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template <class S>
int WaveLaunch<S>::force(hipStream_t st, const NepIO& io, const float* params) {
  (half_wave(io) ? launch_force_wave<S, 32> : launch_force_wave<S, kWave>)(st, io, params);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

template struct WaveLaunch<ShapeSmall>;
template struct WaveLaunch<ShapeGST>;
template struct WaveLaunch<ShapeTable2>;

}  // namespace nepmi
