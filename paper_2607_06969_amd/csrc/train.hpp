// train.hpp -- training kernels: loss seeds and the parameter gradient.
#pragma once

#include "reduce.hpp"

namespace nepmi {

// Blocks per species of the gradient sums over atoms (a fixed number: the
// summation order, hence every bit of the gradient, does not depend on the
// launch).  The partial-sum buffer holds T * kRBlocks * (largest sum) doubles.
// On the 256-cell batch: 64 blocks 2.27 ms per loss and gradient, 128 1.96,
// 256 1.88, 512 2.06.
constexpr int kRBlocks = 256;

// Per-slot training state; every array is column-major [dim][ns].  R is the
// arithmetic precision (float, or double for the float64 variant).
template <class R>
struct TrainIOT {
  int64_t ns;
  const Vec4<R>* pos4;
  const int* cfg_of;
  const int* orig;
  const CfgDev* cfgs;
  const uint32_t* nbrR;
  const int* cntR;
  const uint32_t* nbrA;
  const int* cntA;
  Vec4<R>* lam4;       // [ns] dL/dF in slot order
  const double* mu;    // [n_cfg][9] dL/dV
  const double* ebar;  // [n_cfg] dL/dE
  R* Sst;              // [NA*K] S, then sigma = dE/dS
  R* Sdt;              // [NA*K] Sdot, then Sbar = dj/dS
  R* q;                // [D]
  R* qd;               // [D]
  R* Pb;               // [T*BR] sum_j Q_k per neighbour species
  R* Pdn;              // [T*BR] -sum_j dQ_k (u.t)
  R* abar;             // [H]
  R* zneg;             // [H] -w1 (1 - h^2)
  R* gw1;              // [H] dj/dw1
  R* eat;              // [1] ebar of the atom's configuration
  R* qbR;              // [NR] dj/dq (radial)
  R* FpR;              // [NR] dE/dq (radial)
  R* GA;               // [T*NA*BA] angular coefficient gradient of the atom
  R* FpA;              // [D] dE/dq (rows NR..D-1 used), network pass -> sigma pass
  R* qbA;              // [D] dj/dq (rows NR..D-1 used), network pass -> sigma pass
  R* Ei;               // [N] site energies, caller order (float64 variant only; may be null)
  const int* stop;     // see lists_void
};
using TrainIO = TrainIOT<float>;

struct TrainSeedArgs {
  const RedItem* items;
  int n_items;
  const int* item_start;
  int n_cfg;
  int form;
  double w[3];
  double inv_3ntot;
  const int64_t* off;
  const float* F;
  const float* Fref;
  const double* E;
  const double* Eref;
  const double* V;
  const double* Vref;
  const int* slot_of;
  int64_t n_slots;
  float4* lam4;  // [n_slots] (padding slots are not written)
  double* ebar;
  double* mu;
  double* partF;  // [n_items]
  const int* stop;  // see lists_void
  int* done;      // items summed so far: 0 between launches
  double* loss;
};

// Inputs of the float64 variant: positions in caller order, float64 (the
// neighbour lists are built from their float32 rounding; every pair is then
// tested and evaluated in float64).
struct F64Args {
  const int64_t* atom_off;  // device [n_cfg + 1]
  int n_cfg;
  const double* pos;        // device [N][3]
  const double* params;     // device [P], the parameter layout of the model
  double4* pos4;            // work: [ns] positions in slot order
  double* Wi;               // work: [N][9] per-atom virial, caller order
  const uint32_t* vrev;     // reverse index of the Verlet list (grouped as the list)
  const uint32_t* nbrTA;    // angular part (rc_angular + skin) of each list, row-major, rows of rowTA
  int rowTA;
  const int* cntAV;         // [ns] entries in that part
  double4* fA;              // work: [capA][ns] dE_i/dr_ij of the angular part of i's list, by position
  double* aR;               // work: [T][ns][BR] radial adjoint rows
};

template <class S>
struct TrainLaunch {
  static int seeds(hipStream_t st, const TrainSeedArgs& a);
  static int backward(hipStream_t st, TrainIO io, const Cutoffs& cut, const float* params, const float* lam,
                      const int* base, double* part, double* grad64, float* grad, const MailArgs& mail);
  // float64 variant: forces, site energies (io.Ei) and per-atom virials
  // (a.Wi), all in caller order; the caller sums them per configuration (wave: with
  // a wavefront per atom, otherwise in passes that need the passes' buffers) ...
  static int forward64(hipStream_t st, TrainIOT<double> io, const CutoffsT<double>& cut, const F64Args& a,
                       double* forces, bool wave);
  // ... and the parameter gradient of ebar.E + lambda.F + mu:V
  static int backward64(hipStream_t st, TrainIOT<double> io, const CutoffsT<double>& cut, const F64Args& a,
                        const double* lam, const int* base, double* part, double* grad, bool wave);
};

// The parameter gradient in one pass over the atoms (train_wave.hip), for io with
// pos4, cfg_of, cfgs, lam4, mu, ebar and the list nbrR, cntR (every pair within
// the radial cutoff, more allowed).  part holds train_wave_part(...) doubles.
//
// It serves batches of up to kTrainWaveSlots slots in float32 and train_wave64(...)
// in float64; larger ones take the passes of train.hip, which
// hold an atom per lane and so keep more atoms in flight (lists and gradient, one
// pass against passes, us.  float32, Ge-Sb-Te model: 677 atoms 38 and 162, 9,285
// atoms 120 and 190, 19,800 atoms 213 and 250, 39,402 atoms 370 and 348; model of
// Table 2: 19,800 atoms 250 and 259, 27,173 atoms 351 and 335.  float64: 2,555
// atoms 142 and 408, 46,872 atoms 1000 and 1128, Table 2 1230 and 1318, 74,000
// atoms 1910 and 1718).
constexpr int64_t kTrainWaveSlots = 24576;
// In float64 up to 49,152 slots, but 20,480 where an atom has more angular pairs
// than one chunk holds and few others (molecules): it then walks its list twice,
// and a short radial list is soon done by one lane.  Whole call, one pass and
// passes, Table 2 model, open cells of 20 atoms: 18,000 atoms 573 and 549 us, 24,000
// 702 and 621, 36,000 945 and 824; its solids (angular lists of 20, radial ones of
// 56 at most): 42,000 atoms 1105 and 1185.
inline bool few_beyond_angular(int longestR, int longestA) { return longestA > 16 && longestR < 32; }
inline bool train_wave64(int64_t ns, int longestR, int longestA) {
  return ns <= (few_beyond_angular(longestR, longestA) ? 20480 : 49152);
}
// Blocks: an atom per wavefront while the chip holds them all, then what it
// holds in one round (two blocks per compute unit in float32, one in float64).
template <class R>
inline int train_wave_blocks(int64_t ns) {
  const int64_t few = (ns + 3) / 4, holds = sizeof(R) == 4 ? 512 : 256;
  return (int)(few < holds ? few : holds);
}
template <class R>
inline size_t train_wave_part(int64_t ns, int n_species, size_t entries) {
  return (size_t)(train_wave_blocks<R>(ns) + n_species) * entries;
}
template <class S, class R>
struct TrainWave {
  static int run(hipStream_t st, const TrainIOT<R>& io, const CutoffsT<R>& cut, const R* params, const int* base,
                 double* part, R* grad);
};

// The float64 evaluation with one wavefront per atom (nep_wave64.hip), for io with
// pos4, cfg_of, orig, cfgs, the list and Ei.  It serves batches as wave64(...)
// says; larger ones take the passes of train.hip with a thread per
// atom (whole evaluation, passes and one wavefront per atom, us: Ge-Sb-Te model
// 2,555 atoms 350 and 125, 19,812 atoms 488 and 307, 39,402 atoms 595 and 511,
// 58,570 atoms 700 and 692, 151,707 atoms 1354 and 1549; model of Table 2 2,555
// atoms 478 and 147, 39,402 atoms 783 and 684, 58,570 atoms 899 and 930; its open
// cells of 20 atoms: 30,000 atoms 613 and 600, 36,000 665 and 685, 44,000 723 and
// 797).
inline bool wave64(int64_t ns, int longestR, int longestA) {
  return ns <= (few_beyond_angular(longestR, longestA) ? 32768 : 49152);
}
template <class S>
struct Wave64 {
  static int forward(hipStream_t st, const TrainIOT<double>& io, const CutoffsT<double>& cut, const F64Args& a,
                     double* forces);
};

// float64 helpers: stage positions in slot order, round positions to float32
// (for the neighbour lists), fill a float64 array.
int launch_stage64(hipStream_t st, const TrainIOT<double>& io, const F64Args& a, const float4* pos4f);
int launch_round_pos(hipStream_t st, int64_t n, const double* a, float* b);
int launch_fill64(hipStream_t st, int64_t n, double v, double* a);

}  // namespace nepmi
