// nbr.hpp -- device buffers and the neighbour-list pipeline (host side).
#pragma once

#include <vector>

#include "common.hpp"

namespace nepmi {

// Slots of the device flag word array.  The first four make the lists void (see
// lists_void) and are final when the lists are built.
enum {
  kFlagOverflow = 0,   // a list exceeded its capacity
  kFlagNaN = 1,        // non-finite input position
  kFlagBadSpecies = 2, // species out of range
  kFlagAsym = 3,       // a pair found from one side only by the list build
  kFlagMaxR = 4,       // largest radial list length seen
  kFlagMaxA = 5,       // largest angular list length seen
  kFlagRebuild = 6,    // MD: rebuild the lists in this step
  kFlagLate = 7,       // a pair that an evaluation found from one side only
  kFlagNone = 12,      // four words that stay zero
  kFlagCount = 16
};

// Whether the lists are void: the call that built them is going to build them
// again or to end in an error.  Of the work launched on lists whose flags the host
// has not read yet, the descriptor kernel then leaves every atom without pairs, and
// the kernels behind it run on that but write no output, so that such a call leaves
// its outputs as they were (`stop`: the flags, or the words at kFlagNone where the
// lists are known to be good).  All but the descriptor kernel look at what they
// loaded only where they write (a wait for it up front cost each some 0.2 us).
__device__ __forceinline__ bool lists_void(const int* stop) {
  const int4 f = *reinterpret_cast<const int4*>(stop);
  return (f.x | f.y | f.z | f.w) != 0;
}

// Most species of a model: the list build holds a slot range per species of every
// neighbouring bin.
constexpr int kListSpecies = 4;

// Largest Verlet list length: positions are kept in 16 bits.
constexpr int kMaxListRows = 65535;

// A fixed block of device memory handed out front to back (a bump
// allocator).  Buffers bound to an arena take their memory from it instead of
// hipMalloc, and never free it; the owner resets `used` to reuse the block.
struct Arena {
  char* base = nullptr;
  size_t cap = 0;
  size_t used = 0;
};

// Device allocation that grows on demand (contents are not preserved).  With
// an arena, growing takes a new region of the arena (NEPMI_INVALID_ARG when
// the arena is exhausted) and nothing is ever freed.
struct DevBuf {
  void* p = nullptr;
  size_t bytes = 0;
  Arena* arena = nullptr;
  template <class T>
  T* ptr() const {
    return static_cast<T*>(p);
  }
  int ensure(size_t n);
  void release();
  ~DevBuf() { release(); }
  DevBuf() = default;
  DevBuf(const DevBuf&) = delete;
  DevBuf& operator=(const DevBuf&) = delete;
};

// A handle's block of pinned host memory: the list flags on their way to the
// host (the first kPinMail bytes), then tables on their way to the GPU.  Blocks
// come from a pool that grows by a chunk when more handles live than ever before
// and keeps its memory until the process ends: a call never allocates or frees
// host memory, and host memory that a kernel has read is never unmapped.  A
// handle gives its block back when nothing on the GPU uses it any more (every
// call that ends in an error has waited for its stream, see settle).
constexpr size_t kPinBytes = (size_t)128 << 10, kPinMail = 128;
struct PinBlock {
  char* p = nullptr;
  int take();  // from the pool, unless one is held
  ~PinBlock();
  PinBlock() = default;
  PinBlock(const PinBlock&) = delete;
  PinBlock& operator=(const PinBlock&) = delete;
};

struct UploadArgs {
  static constexpr int kMost = 5;  // tables
  struct {
    const uint4* src;
    uint4* dst;
    int64_t n;
  } seg[kMost];
  int n_seg;
  int* clear;
  int n_clear;
  int64_t words;  // 16-byte words of all tables
};

// Host tables on their way to device buffers: copied into the handle's pinned
// block, then moved by one kernel (a copy call for each table costs the host some
// 10 us and the stream 5).  The block is free again once the stream has passed the
// kernel; the owner waits for that before the next upload.  Tables that exceed
// the block (some 500 configurations) are copied by the runtime instead.
struct Uploader {
  struct Table {
    const void* src;
    DevBuf* dst;
    size_t bytes;
  };
  char* pin = nullptr;  // the handle's block
  std::vector<Table> tables;
  // dst receives the bytes (and is sized for them)
  int add(const void* src, size_t bytes, DevBuf& dst);
  // The upload of the added tables, clearing n_clear ints at clear: for a kernel
  // on st that does it (upload_part), and launched by itself.
  int plan(hipStream_t st, int* clear, int n_clear, UploadArgs& out);
  int run(hipStream_t st, int* clear, int n_clear);
};

// The list flags on their way to the host: the kernel that gets these writes
// them into pinned memory, then a one behind them (a zero before).
struct MailArgs {
  const int* flags = nullptr;
  int* mail = nullptr;  // null: nothing to deliver
};
__device__ __forceinline__ void deliver(const MailArgs& m) {
  for (int k = 0; k < kFlagCount; ++k) m.mail[k] = m.flags[k];
  __threadfence_system();
  __hip_atomic_store(&m.mail[kFlagCount], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// State that a rebuild moves from caller order into the new slot order along
// with the positions (MD: float64 positions, velocities, and the positions the
// new lists are built from, as the drift reference).  Used when xd is not null.
struct SlotCarry {
  const double* xd_user = nullptr;  // [N][3] float64 positions, caller order
  const float4* x_user = nullptr;   // [N] the float32 positions the build staged
  const float4* v_user = nullptr;   // [N] velocities
  double* xd = nullptr;             // [n_slots][3]
  float4* vel4 = nullptr;           // [n_slots] (zero in padding slots)
  float4* ref4 = nullptr;           // [n_slots]
};

// State in the present slot order (MD) that a rebuild takes its atoms from: it
// goes back to caller order, positions wrapped, before it is sorted.  Used when
// xd is not null.
struct SlotSource {
  const int* cfg_of = nullptr;      // [n_slots]
  const int* orig = nullptr;        // [n_slots]
  const double* xd = nullptr;       // [n_slots][3]
  const float4* vel4 = nullptr;     // [n_slots]
  double* xd_user = nullptr;        // [N][3], caller order
  float4* x_user = nullptr;         // [N] float32 positions
  float4* v_user = nullptr;         // [N]
};

// Neighbour lists of one batch of configurations, in processing order.
struct NbrPipeline {
  int64_t N = 0;        // atoms
  int n_cfg = 0;
  int n_species = 0;
  int64_t n_slots = 0;  // N + n_species * wavefront (upper bound of used slots)
  int total_bins = 0;   // bins of every configuration in whole 4 x 4 x 4 tiles
  int real_bins = 0;    // those inside the cells
  int bin_atoms = 0;    // atoms per bin of the fullest configuration (mean over its bins, rounded up)
  double density = 0.0; // atoms per volume of the densest configuration
  int capR = 0, capA = 0;
  int longestR = 0, longestA = 0;  // longest lists that the last flags read told of (0: none read yet)
  float rclR2 = 0.f, rclA2 = 0.f;
  float far0 = 0.f;     // beyond it from a bin's atoms, no candidate is a neighbour (see k_build_lists)
  double skin = 0.0;
  std::vector<CfgDev> host_cfgs;
  std::vector<int64_t> host_off;

  DevBuf cfgs, atom_off_dev;
  DevBuf key, cnt, start, cursor, tile_sums, base, perm, pos_tmp, cfg_tmp;
  DevBuf pos4, cfg_of, orig, slot_of;
  DevBuf nbrR, cntR;             // Verlet list (rc_radial + skin)
  DevBuf cntAV;                  // entries within rc_angular + skin (the angular part of the list)
  DevBuf nbrTA;                  // the angular part of each list, row-major, rows of rowTA entries (reverse search)
  DevBuf angm;                   // uint32: bit k % 32 of word k / 32 ([word][slot]): entry k is in the angular part
  int rowTA = 0;
  int clear_keys = 0;            // key counts (cnt) known to be zero between sorts
  DevBuf vrev;                   // reverse index of the Verlet list (see k_reverse)
  DevBuf cnbrR, ccntR, cnbrA, ccntA, cposA;  // per-evaluation compact lists (rc_radial, rc_angular),
                                             // in groups of four entries (see list_groups)
  DevBuf flags;
  Uploader up;
  bool unsent = false;  // a kernel launched on the lists is to deliver the flags (post)
  // Work in the pinned block of a handle from now on.
  void use_pinned(const PinBlock& b) { up.pin = b.p; }
  int* mail() const { return reinterpret_cast<int*>(up.pin); }

  // Host-side setup of a batch: validates the cells, computes bins, sizes
  // buffers and adds the configuration tables to `up`.  pbc: host int32[3
  // n_cfg] (1 periodic, 0 not, per lattice vector) or null (all periodic).
  // Returns NEPMI_* codes.
  int setup(int n_cfg, const int64_t* atom_off, const double* cells, const int32_t* pbc, int n_species, double rcR,
            double rcA, double skin);
  // Sizes the lists for capR x capA entries per slot.
  int ensure_lists(int capR_, int capA_);
  // Take every device buffer from `a` from now on (releases what is held; the
  // next setup sizes the lists afresh).
  void use_arena(Arena* a);
  // Stage, bin and sort (pos: N x pos_stride floats).  gate: optional device
  // flag; every kernel returns at once when *gate == 0.  carry: state moved
  // into slot order with the positions (optional).  src: take the atoms from
  // this state instead of pos (optional).  upload: to be done first (optional).
  int launch_sort(hipStream_t st, const float* pos, int pos_stride, const int32_t* species, int n_species,
                  const int* gate, const SlotCarry* carry = nullptr, const SlotSource* src = nullptr,
                  const UploadArgs* upload = nullptr);
  int launch_lists(hipStream_t st, int n_species, const int* gate);
  // Full build, in two parts so that work on the lists can be launched between
  // them: build_start launches the upload, sort and lists; build_end waits for
  // the flags, reports what the build found wrong, and builds lists that were
  // too short again with a larger capacity (regrown: work launched on the first
  // ones, which kept within the capacity, is void).  post: the first kernel
  // launched on the lists delivers the flags (post()), as one of its own costs
  // the 4.5 us of any kernel behind another; otherwise build_start launches it.
  int build_start(hipStream_t st, const float* pos, const int32_t* species, bool post);
  MailArgs post() const;
  // atoms within rc of a point at that density
  float pairs_within(double rc) const { return (float)(density * 4.18879020478639 * rc * rc * rc); }
  int build_end(hipStream_t st, bool& regrown);
  int check_flags(hipStream_t st, int* host_flags);
};

// Wrap r into the cell along its periodic directions in float64, and round it
// to f; if the rounding lands outside the cell (a last-ulp case at a face),
// wrap the rounded value once more.  Non-periodic directions are left alone.
static __device__ __forceinline__ void wrap_periodic(const CfgDev& C, double r[3], float f[3]) {
  for (int pass = 0; pass < 2; ++pass) {
    double m[3];
    for (int a = 0; a < 3; ++a) {
      const double s = r[0] * C.Hinv[a] + r[1] * C.Hinv[3 + a] + r[2] * C.Hinv[6 + a];
      m[a] = (C.periodic >> a) & 1 ? floor(s) : 0.0;
    }
    for (int a = 0; a < 3; ++a) r[a] -= m[0] * C.Hd[a] + m[1] * C.Hd[3 + a] + m[2] * C.Hd[6 + a];
    for (int a = 0; a < 3; ++a) f[a] = (float)r[a];
    // the float32 copy must also lie in the cell (as the staging kernel sees it)
    bool inside = true;
    for (int a = 0; a < 3; ++a) {
      const double s = (double)f[0] * C.Hinv[a] + (double)f[1] * C.Hinv[3 + a] + (double)f[2] * C.Hinv[6 + a];
      if ((C.periodic >> a) & 1 && floor(s) != 0.0) inside = false;
    }
    if (inside) break;
    for (int a = 0; a < 3; ++a) r[a] = (double)f[a];
  }
}

// Fill an int array with a value on the stream (graph-safe, no memset node).
void fill_int(hipStream_t st, int* p, int64_t n, int v, const int* gate);

}  // namespace nepmi
