// nep_kernels.hpp -- NEP evaluation kernels for gfx950, templated on the shape.
//
// One thread evaluates one atom slot (a wavefront or half of one in small
// batches, see nep_wave.hip); every wavefront holds one species (see
// nbr.hip), so species-pair coefficients c[Z_i][.] and the network weights of
// Z_i are read through the scalar unit.  Coefficients that depend on the
// neighbour's species are read from LDS.  The kernels use a derived copy of
// the Chebyshev coefficients stored after the parameters (k_derive), in which
// the "+1" of Q_k = (T_k + 1) f_c / 2 is folded into column 0.
//
//   k_desc   filters the Verlet list into compact lists of the pairs inside
//            the radial and angular cutoffs (accumulating the radial sums on
//            the way), then computes the descriptors (Eq. 11, 16, 17 and the
//            4-/5-body invariants), the network (Sec. 2.3), site energy E_i,
//            and the adjoints the force kernel needs: dE_i/dq for the angular
//            descriptors, and atil_i[b][k] = sum_n dE_i/dq_n ctil[Z_i][b][n][k]
//            for the radial ones.
//   k_force  pair forces dE_i/dr_ij and the per-atom virial (Eq. 3, Eq. 4).
//            Radial pairs gather the neighbour's atil_j[Z_i] and add both
//            directions at once; for angular pairs, dE_i/dr_ij is added to
//            i's own force and kept in i's compact slot (no atomics).  S_i is
//            recomputed rather than stored.
//   k_gather F_i = own part - sum_j dE_j/dr_ji over i's angular pairs (Eq. 3),
//            finding i's slot in j's compact list from the reverse index
//            built with the lists and j's entry mask.
#pragma once

#include "reduce.hpp"

namespace nepmi {

struct NepIO {
  int64_t n_slots;
  int capR;              // rows of the Verlet list and of the pair buffer
  int capA;              // rows of the compact angular list
  const float4* pos4;
  const int* cfg_of;
  const int* orig;
  const CfgDev* cfgs;
  const uint32_t* nbrR;  // Verlet list (rc_radial + skin), in groups of four entries
  const int* cntR;
  const uint32_t* vrev;  // position of i in the angular part (rc_angular + skin) of j's Verlet list,
                         // 0xFFFFFFFF outside that part; grouped as nbrR
  uint32_t* cnR;         // compact list: pairs within rc_radial (written by k_desc)
  int* ccR;
  uint32_t* cnA;         // compact list: pairs within rc_angular (written by k_desc)
  uint32_t* cpA;         // own angular-part position | reverse position << 16, grouped as cnA
  int* ccA;
  int* flags;
  const int* stop;       // see lists_void
  Cutoffs cut;
  float* fp;     // [NANG][n_slots]  dE_i/dq (angular descriptors)
  float* aR;     // [T][n_slots][BR] radial adjoint, part b = atil_i[b][.]
  float* Ei;     // [N] caller order (site energies)
  float* qout;   // [N][D] caller order, optional
  float4* frad;  // [n_slots] own force part (radial pairs both ways, angular dE_i/dr_ij)
  float4* fA;    // [capA][n_slots] angular pair forces dE_i/dr_ij in i's compact slots
  uint64_t* amask; // [ceil(capA/64)][n_slots] entries of the angular part of i's Verlet list that are
                   // in its compact angular list
  float* Wi;     // [N][9] caller order, per-atom virial
  float* Fuser;  // [N][3] caller order, optional
  float4* Fproc; // [n_slots], optional
  float* Eproc;  // [n_slots] site energies in slot order, optional
  MailArgs mail; // list flags for k_desc to deliver, if any
  float pairsA = 0.f;  // angular pairs of an atom at the mean density of the fullest configuration
};

constexpr int kDescVariants = 10;  // compiled variants of k_desc (4..7: network in its own kernel;
                                   // 8, 9: variant 0 in blocks of 128 and 512 threads)
constexpr int kForceVariants = 6;  // compiled variants of k_force (4, 5: variant 0 in blocks of 128, 512)
constexpr int kGatherVariants = 4; // k_gather in blocks of 256, 128, 512, 1024 threads

// Constants of an MD step.
constexpr int kMaxSpecies = 8;
struct MdConst {
  float acc[kMaxSpecies];   // dt/2 * kAccUnit / m_s   (half kick per unit force)
  float kin[kMaxSpecies];   // m_s / (2 kAccUnit)       (eV per (A/fs)^2)
  float dt;
  float half_skin2;         // (skin/2)^2
};

// The second half kick of an MD step, and the step's bookkeeping.
struct KickArgs {
  MdConst mc;
  const float4* pos4 = nullptr;
  float4* vel4 = nullptr;         // [n_slots]
  float* Ki = nullptr;            // [N] caller order, kinetic energies
  int* flags = nullptr;           // of the neighbour lists
  long long* counters = nullptr;  // steps, rebuilds
};

template <class S>
struct Launch {
  static int desc(hipStream_t st, const NepIO& io, const float* params, bool want_adjoint, int variant);
  static int force(hipStream_t st, const NepIO& io, const float* params, int variant);
  // with the sums of an evaluation (may be null), or the half kick that
  // follows the forces of an MD step (may be null), in the same launch
  static int gather(hipStream_t st, const NepIO& io, int variant, const SumArgs<float>* sums, const KickArgs* kick);
  // Copies the P parameters and writes the derived tables after them (the
  // parameter buffer holds PALL floats).
  static int derive(hipStream_t st, const float* given, float* params);
};

// Variant 0 of k_desc and k_force with a group of lanes per atom, bit for bit the
// same results (nep_wave.hip), for batches that fit kWaveSlots slots.
// With one thread per atom these kernels take the time of one walk up to about
// 65,000 atoms (one wavefront per SIMD); with a group the time grows with the
// atoms.  k_desc + k_force + k_gather, thread -> group (us): Ge-Sb-Te model
// 9,285 atoms 146 -> 54, 19,812 147 -> 85, 34,707 164 -> 135, 46,872 166 -> 174;
// Table 2 model 9,285 atoms 182 -> 65, 34,707 203 -> 187, 46,872 210 -> 242.
// k_desc alone: 34,707 atoms 64 -> 51 and 78 -> 70, 46,872 68 -> 66 and 80 -> 91.
constexpr int64_t kWaveSlots = 36864;
template <class S>
struct WaveLaunch {
  static int desc(hipStream_t st, const NepIO& io, const float* params, bool want_adjoint);
  static int force(hipStream_t st, const NepIO& io, const float* params);
};

}  // namespace nepmi
