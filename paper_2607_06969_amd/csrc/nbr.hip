// nbr.hip -- cell-list binning, processing order and Verlet neighbour lists.
//
// The paper builds neighbour lists on the fly with linear complexity before
// every evaluation (Sec. 3.4, Sec. 3.5).  Here that is a counting sort of the
// atoms into cell bins, done on the GPU, followed by a 27-bin stencil search.
//
// Processing order.  Atoms are renumbered into "slots" sorted by
// (species, global bin, caller index).  Each species group starts at a
// multiple of the wavefront size, so every wavefront of the evaluation
// kernels holds atoms of a single species and reads that species'
// coefficients and network weights through the scalar unit.  Padding slots
// carry orig = -1.
//
// Neighbour entries are 32-bit: slot index (27 bits) | image code (5 bits),
// code = (w0+1)*9 + (w1+1)*3 + (w2+1) for the lattice shift w in {-1,0,1}^3.
// Lists are stored in groups of four entries, group g of slot p as one 16-byte
// word at [g * n_slots + p] (group_index).  The Verlet list holds pairs within
// rc_radial + skin; at every evaluation the descriptor kernel filters it into
// compact lists of the pairs within rc_radial and within rc_angular, which all
// later kernels iterate.
#include "nbr.hpp"

#include <algorithm>
#include <cstring>
#include <mutex>

namespace nepmi {

constexpr int kScanBlock = 1024;
// Largest sort that one block does whole, and most keys that one block scans
// (see k_sort_small, k_scan_one).
constexpr int kSmallAtoms = 4096, kSmallKeys = 8192;
// Upload that such a sort takes along, in 16-byte words: one per thread (3,686
// atoms: sort 15.4 us behind an upload of 4.1, 18.3 with it and a launch less).
constexpr int kSmallUpload = 1024;
constexpr int kOneScan = 1 << 15, kOneScanGated = 1 << 20;

// ------------------------------------------------------------------ staging

// Global sort key of a cell bin.  Bins are numbered in 4 x 4 x 4 tiles (tile
// row-major, then row-major inside the tile), so that a contiguous range of
// slots covers a compact region of space: the atoms a GPU die processes at
// the same time, and their neighbours, then fit its L2 better than with
// row-major slabs.  Each configuration owns ceil(nb/4)^3 * 64 keys.
__device__ __forceinline__ int bin_key(const CfgDev& C, int b0, int b1, int b2) {
  const int nt1 = (C.nb[1] + 3) >> 2, nt2 = (C.nb[2] + 3) >> 2;
  const int t = ((b0 >> 2) * nt1 + (b1 >> 2)) * nt2 + (b2 >> 2);
  return C.bin_off + (t << 6) + (((b0 & 3) << 4) | ((b1 & 3) << 2) | (b2 & 3));
}

// Sort key of an atom at (x, y, w) of species z, and its position wrapped into
// the cell.
__device__ __forceinline__ int stage_atom(const CfgDev& C, int z, int total_bins, float x, float y, float w,
                                          float (&o)[3]) {
  int b[3];
  double m[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double s = (double)x * C.Hinv[a] + (double)y * C.Hinv[3 + a] + (double)w * C.Hinv[6 + a];
    // along a non-periodic direction the atom is not wrapped, and one outside
    // the cell goes to the nearest bin: its neighbours within the list cutoff
    // lie in that bin or beyond the face as well (bins are wider than the
    // cutoff), so the stencil still finds every pair
    m[a] = (C.periodic >> a) & 1 ? floor(s) : 0.0;
    const double t = (s - m[a]) * C.nb[a];
    b[a] = t < 0.0 ? 0 : (t >= (double)C.nb[a] ? C.nb[a] - 1 : (int)t);
  }
  o[0] = x;
  o[1] = y;
  o[2] = w;
  if (m[0] != 0.0 || m[1] != 0.0 || m[2] != 0.0) {
    // wrap by whole lattice vectors (float64, then rounded once)
#pragma unroll
    for (int a = 0; a < 3; ++a)
      o[a] = (float)((double)o[a] - m[0] * C.Hd[a] - m[1] * C.Hd[3 + a] - m[2] * C.Hd[6 + a]);
  }
  return z * total_bins + bin_key(C, b[0], b[1], b[2]);
}

// Thread t of `step` of an upload.
__device__ __forceinline__ void upload_part(const UploadArgs& a, int64_t t, int64_t step) {
  if (t < a.n_clear) a.clear[t] = 0;
#pragma unroll
  for (int s = 0; s < UploadArgs::kMost; ++s)
    if (s < a.n_seg)
      for (int64_t i = t; i < a.seg[s].n; i += step) a.seg[s].dst[i] = a.seg[s].src[i];
}

// Where the atoms to sort come from and what the sort works on.
struct SortArgs {
  int64_t N, n_slots;
  int n_cfg, n_species, total_bins;
  const int64_t* atom_off;
  const CfgDev* cfgs;
  const float* pos;          // caller order, pos_stride floats per atom (unused with src.xd)
  int pos_stride;
  const int32_t* species;    // caller order
  SlotSource src;            // MD state in the present slot order (src.xd null: none)
  SlotCarry carry;
  // work
  float4* pos_tmp;
  int *cfg_tmp, *key, *cnt, *start, *cursor, *perm;
  // results
  float4* pos4;
  int *base, *cfg_of, *orig, *slot_of, *cntR, *cntAV, *flags;
};

// An atom on its way to its slot.
struct Staged {
  int key;         // sort key, -1 if the atom is refused (the flags say why)
  int i, c;        // caller index, configuration
  float4 x;        // wrapped position and species
  float4 xu, v;    // MD state: float32 position the build stages, velocity
  double r[3];     // MD state: float64 position
};

// Stage caller atom i of configuration c at (x, y, w).
__device__ __forceinline__ void stage_one(const SortArgs& a, Staged& s, float x, float y, float w) {
  const int z = a.species[s.i];
  s.key = -1;
  if (z < 0 || z >= a.n_species) {
    atomicOr(&a.flags[kFlagBadSpecies], 1);
  } else if (!(isfinite(x) && isfinite(y) && isfinite(w))) {
    atomicOr(&a.flags[kFlagNaN], 1);
  } else {
    float o[3];
    s.key = stage_atom(a.cfgs[s.c], z, a.total_bins, x, y, w, o);
    s.x = make_float4(o[0], o[1], o[2], __int_as_float(z));
  }
}

// Configuration of caller atom i: the last c with off[c] <= i.
template <class P>
__device__ __forceinline__ int config_of(P off, int n_cfg, int64_t i) {
  int lo = 0, hi = n_cfg;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// Stage slot p of the MD state, its position wrapped into the cell in float64
// (so that the float32 copy needs no further wrapping); false for padding.
__device__ __forceinline__ bool stage_slot(const SortArgs& a, Staged& s, int64_t p) {
  s.key = -1;
  s.c = a.src.cfg_of[p];
  if (s.c < 0) return false;
  s.i = a.src.orig[p];
  s.v = a.src.vel4[p];
  float f[3];
#pragma unroll
  for (int x = 0; x < 3; ++x) s.r[x] = a.src.xd[3 * p + x];
  wrap_periodic(a.cfgs[s.c], s.r, f);
  s.xu = make_float4(f[0], f[1], f[2], 0.f);
  stage_one(a, s, f[0], f[1], f[2]);
  return true;
}

// Stage the atom of each thread: a caller atom, or a slot of the MD state, whose
// state goes back to caller order.
template <bool SLOTS>
__global__ void k_stage(SortArgs a, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (SLOTS ? a.n_slots : a.N)) return;
  Staged s;
  if constexpr (SLOTS) {
    if (!stage_slot(a, s, t)) return;
#pragma unroll
    for (int x = 0; x < 3; ++x) a.src.xd_user[3 * (int64_t)s.i + x] = s.r[x];
    a.src.x_user[s.i] = s.xu;
    a.src.v_user[s.i] = s.v;
  } else {
    s.i = (int)t;
    s.c = config_of(a.atom_off, a.n_cfg, t);
    const float* x = a.pos + t * a.pos_stride;
    stage_one(a, s, x[0], x[1], x[2]);
  }
  a.key[s.i] = s.key;
  if (s.key < 0) return;
  a.pos_tmp[s.i] = s.x;
  a.cfg_tmp[s.i] = s.c;
  atomicAdd(&a.cnt[s.key], 1);
}

// Put an atom into slot p.  With carry.xd set, the carried state moves into the
// slot as well: the staging wraps again only in a last-ulp case at a cell face,
// and that shift (zero otherwise) is carried into the float64 position.
__device__ __forceinline__ void put_slot(const SortArgs& a, int64_t p, const Staged& s) {
  a.pos4[p] = s.x;
  a.cfg_of[p] = s.c;
  a.orig[p] = s.i;
  if (a.slot_of) a.slot_of[s.i] = (int)p;
  if (a.carry.xd) {
    double* o = a.carry.xd + 3 * p;
    o[0] = s.r[0] + ((double)s.x.x - (double)s.xu.x);
    o[1] = s.r[1] + ((double)s.x.y - (double)s.xu.y);
    o[2] = s.r[2] + ((double)s.x.z - (double)s.xu.z);
    a.carry.vel4[p] = s.v;
    a.carry.ref4[p] = s.x;
  }
}

// The carried state of caller atom i.
__device__ __forceinline__ void load_carry(const SortArgs& a, Staged& s) {
  if (!a.carry.xd) return;
#pragma unroll
  for (int x = 0; x < 3; ++x) s.r[x] = a.carry.xd_user[3 * (int64_t)s.i + x];
  s.xu = a.carry.x_user[s.i];
  s.v = a.carry.v_user[s.i];
}

// Padding slots get orig = -1, their group's species and empty lists (the list
// build visits atoms only).
__device__ __forceinline__ void pad_slot(const SortArgs& a, int64_t p, int z) {
  if (a.carry.xd) a.carry.vel4[p] = make_float4(0.f, 0.f, 0.f, 0.f);
  a.pos4[p] = make_float4(0.f, 0.f, 0.f, __int_as_float(z));
  a.cfg_of[p] = -1;
  a.orig[p] = -1;
  a.cntR[p] = 0;
  a.cntAV[p] = 0;
}

// ------------------------------------------------------------ exclusive scan

constexpr int kScanItems = 4;
constexpr int kScanTile = kScanBlock * kScanItems;

// Inclusive scan over a block of kScanBlock threads (wavefront scans, then the
// wavefront totals); sh holds one int per wavefront.  Ends with a barrier.
__device__ __forceinline__ int block_inclusive(int v, int* sh, int& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63) sh[wv] = v;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kScanBlock / 64; ++w) {
    before += w < wv ? sh[w] : 0;
    total += sh[w];
  }
  __syncthreads();
  return v + before;
}

// out[0..M] = exclusive prefix sum of in[0..M-1] (out[M] = total), tile level.
__global__ __launch_bounds__(kScanBlock) void k_scan_tiles(const int* __restrict__ in, int M, int* __restrict__ out,
                                                           int* __restrict__ tile_sums, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  __shared__ int sh[kScanBlock / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int v[kScanItems], s = 0;
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = (base + j < M) ? in[base + j] : 0;
    s += v[j];
  }
  int total;
  int ex = block_inclusive(s, sh, total) - s;
  for (int j = 0; j < kScanItems; ++j) {
    if (base + j < M) out[base + j] = ex;
    ex += v[j];
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// Scan of the tile sums (one block; n_tiles <= kScanTile) and the final
// total, then the processing order's species bases: base[z] = first slot of
// species z, each species' group padded to the wavefront size.  out holds the
// tile-local prefixes of k_scan_tiles; the global prefix of key k is
// out[k] + (scanned tile sum of k's tile).
__global__ __launch_bounds__(kScanBlock) void k_scan_sums(int* __restrict__ tile_sums, int n_tiles,
                                                          int* __restrict__ out, int M, int total_bins,
                                                          int n_species, int* __restrict__ species_base,
                                                          const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  __shared__ int sh[kScanBlock / 64];
  __shared__ int tile_ex[kScanTile];
  const int b0 = threadIdx.x * kScanItems;
  int v[kScanItems], s = 0;
  for (int j = 0; j < kScanItems; ++j) {
    v[j] = (b0 + j < n_tiles) ? tile_sums[b0 + j] : 0;
    s += v[j];
  }
  int total;
  int ex = block_inclusive(s, sh, total) - s;
  for (int j = 0; j < kScanItems; ++j) {
    if (b0 + j < n_tiles) {
      tile_sums[b0 + j] = ex;
      tile_ex[b0 + j] = ex;
    }
    ex += v[j];
  }
  if (threadIdx.x == 0) out[M] = total;
  __syncthreads();
  if (threadIdx.x != 0) return;
  int acc = 0, lo = 0;  // lo: global prefix at z * total_bins
  for (int z = 0; z < n_species; ++z) {
    const int k = (z + 1) * total_bins;
    const int hi = k < M ? out[k] + tile_ex[k / kScanTile] : total;
    species_base[z] = acc;
    acc += (hi - lo + kWave - 1) / kWave * kWave;
    lo = hi;
  }
  species_base[n_species] = acc;
}

// Global prefixes, also copied into the scatter cursors; the counts are cleared
// for the next sort.
__global__ void k_scan_add(int* __restrict__ out, int M, const int* __restrict__ tile_sums,
                           int* __restrict__ cursor, int* __restrict__ cnt, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < M) {
    const int v = out[i] + tile_sums[i / kScanTile];
    out[i] = v;
    cursor[i] = v;
    cnt[i] = 0;
  }
}

// Species bases from the number of atoms before each species: base[z] = first
// slot of species z, each group padded to the wavefront size.
__device__ __forceinline__ void species_bases(int n_species, const int* lo, int total, int* base) {
  int acc = 0;
  for (int z = 0; z < n_species; ++z) {
    const int n = (z + 1 < n_species ? lo[z + 1] : total) - lo[z];
    base[z] = acc;
    acc += (n + kWave - 1) / kWave * kWave;
  }
  base[n_species] = acc;
}

// The whole scan by one block: prefixes, cursors, cleared counts, species
// bases.  One kernel instead of three for the small sorts, where a launch costs
// more than the scan, and for the gated sorts of MD, where every kernel costs
// 4.5 us in every step and the sort runs once in some 40 (255 thousand keys
// there at 900,000 atoms).  12,288 keys: 12.5 us in three kernels, 5.8 in one;
// 49,152 keys: 14.8 and 15.1.
__global__ __launch_bounds__(kScanBlock) void k_scan_one(SortArgs a, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  constexpr int Q = 2;  // int4 per thread and round
  __shared__ int sh[kScanBlock / 64];
  __shared__ int lo_s[kListSpecies];
  const int M = a.n_species * a.total_bins;  // a multiple of 64 (bins come in tiles of 64)
  int4* cnt = reinterpret_cast<int4*>(a.cnt);
  int4* start = reinterpret_cast<int4*>(a.start);
  int4* cursor = reinterpret_cast<int4*>(a.cursor);
  const int M4 = M / 4, wave0 = (int)(threadIdx.x & ~63u) * Q + (int)(threadIdx.x & 63u);
  int run = 0;
  int4 v[Q];
  // a wavefront takes 64 Q consecutive int4, lane by lane
  auto load = [&](int b) {
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = b + 64 * q < M4 ? cnt[b + 64 * q] : make_int4(0, 0, 0, 0);
  };
  load(wave0);
  for (int b0 = 0; b0 < M4; b0 += kScanBlock * Q) {
    const int b = b0 + wave0;
    int4 c[Q];
    int before = 0;  // keys of this wavefront's earlier int4 rows
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int s = v[q].x + v[q].y + v[q].z + v[q].w;
      int inc = s;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
      }
      const int ex = before + inc - s;
      c[q] = make_int4(ex, ex + v[q].x, ex + v[q].x + v[q].y, ex + v[q].x + v[q].y + v[q].z);
      before += __shfl(inc, 63, 64);
    }
    load(b + kScanBlock * Q);  // the next round's counts, ahead of the barriers
    if (lane == 0) sh[wv] = before;
    __syncthreads();
    int off = run;
#pragma unroll
    for (int w = 0; w < kScanBlock / 64; ++w) {
      off += w < wv ? sh[w] : 0;
      run += sh[w];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (b + 64 * q < M4) {
        const int4 o = make_int4(c[q].x + off, c[q].y + off, c[q].z + off, c[q].w + off);
        start[b + 64 * q] = o;
        cursor[b + 64 * q] = o;
        cnt[b + 64 * q] = make_int4(0, 0, 0, 0);
      }
  }
  __syncthreads();
  if ((int)threadIdx.x < a.n_species) lo_s[threadIdx.x] = a.start[threadIdx.x * a.total_bins];
  __syncthreads();
  if (threadIdx.x == 0) {
    a.start[M] = run;
    species_bases(a.n_species, lo_s, run, a.base);
  }
}

// ------------------------------------------------------- processing order

// Slots of the atoms of each key, in the order an atomic decides; k_fill_slots
// makes it the caller's order.
__global__ void k_scatter(SortArgs a, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.N) return;
  const int k = a.key[i];
  if (k < 0) return;
  const int z = k / a.total_bins;
  // cursor[k] starts at start[k]: the returned value is start[k] + rank in key
  const int r = atomicAdd(&a.cursor[k], 1);
  a.perm[a.base[z] + (r - a.start[z * a.total_bins])] = (int)i;
}

// Fill the slot arrays.  The thread of scattered atom i counts the atoms of its
// key with a smaller caller index: its place in the key (an insertion sort of
// each key by one thread took 7 to 41 us, its swaps one after another).
__global__ void k_fill_slots(SortArgs a, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.n_slots) return;
  int z = -1;
  for (int t = 0; t < a.n_species; ++t)
    if (p >= a.base[t] && p < a.base[t + 1]) z = t;
  if (z >= 0) {
    const int s0 = a.start[z * a.total_bins];
    if (p - a.base[z] < a.start[(z + 1) * a.total_bins] - s0) {
      const int i = a.perm[p];
      const int k = a.key[i];
      const int q0 = a.base[z] + (a.start[k] - s0), n = a.start[k + 1] - a.start[k];
      int rank = 0;
      for (int q = 0; q < n; q += 4) {  // four loads at a time (clamped into the key)
        int v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = a.perm[q0 + (q + u < n ? q + u : n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) rank += q + u < n && v[u] < i ? 1 : 0;
      }
      Staged s;
      s.i = i;
      s.c = a.cfg_tmp[i];
      s.x = a.pos_tmp[i];
      load_carry(a, s);
      put_slot(a, q0 + rank, s);
      return;
    }
  }
  pad_slot(a, p, z < 0 ? 0 : z);
}

// The whole sort by one block, the counts and the order in LDS and the atoms in
// registers: one kernel instead of four for batches of a few thousand atoms,
// where launches are most of the cost.  A gated sort then
// costs an MD step one idle kernel instead of eight (4.5 us each).  3,686 atoms:
// 37 us in seven kernels, 16 in one.
template <bool SLOTS>
__global__ __launch_bounds__(kScanBlock) void k_sort_small(SortArgs a, const int* __restrict__ gate,
                                                           UploadArgs up) {
  if (gate && *gate == 0) return;
  constexpr int IT = kSmallAtoms / kScanBlock;
  constexpr int kOff = 512;         // configurations whose offsets fit LDS
  __shared__ int cur[kSmallKeys];   // counts, then (scanned) next free place, then end of every key
  __shared__ int perm[kSmallAtoms];
  __shared__ int off_s[SLOTS ? 1 : kOff];
  __shared__ int sh[kScanBlock / 64];
  __shared__ int lo_s[kListSpecies], base_s[kListSpecies + 1];
  const int t = threadIdx.x, M = a.n_species * a.total_bins;
  if constexpr (!SLOTS) {
    upload_part(up, t, kScanBlock);
    __syncthreads();
  }
  for (int k = t; k < M; k += kScanBlock) cur[k] = 0;
  const bool in_lds = a.n_cfg <= kOff;
  if (!SLOTS && in_lds)
    for (int c = t; c < a.n_cfg; c += kScanBlock) off_s[c] = (int)a.atom_off[c];
  __syncthreads();
  Staged s[IT];
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int j = t + u * kScanBlock;
    s[u].key = -1;
    if (j < (int)(SLOTS ? a.n_slots : a.N)) {
      if constexpr (SLOTS) {
        stage_slot(a, s[u], j);
      } else {
        s[u].i = j;
        s[u].c = in_lds ? config_of(off_s, a.n_cfg, j) : config_of(a.atom_off, a.n_cfg, j);
        const float* x = a.pos + (int64_t)j * a.pos_stride;
        stage_one(a, s[u], x[0], x[1], x[2]);
        load_carry(a, s[u]);
      }
      if (s[u].key >= 0) atomicAdd(&cur[s[u].key], 1);
    }
  }
  __syncthreads();
  int run = 0;
  for (int b0 = 0; b0 < M; b0 += kScanBlock) {
    const int k = b0 + t;
    const int n = k < M ? cur[k] : 0;
    int total;
    const int ex = run + block_inclusive(n, sh, total) - n;
    if (k < M) {
      cur[k] = ex;
      a.start[k] = ex;
    }
    run += total;
  }
  __syncthreads();
  if (t < a.n_species) lo_s[t] = cur[t * a.total_bins];
  __syncthreads();
  if (t == 0) {
    a.start[M] = run;
    species_bases(a.n_species, lo_s, run, base_s);
    for (int z = 0; z <= a.n_species; ++z) a.base[z] = base_s[z];
  }
#pragma unroll
  for (int u = 0; u < IT; ++u)
    if (s[u].key >= 0) perm[atomicAdd(&cur[s[u].key], 1)] = s[u].i;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < IT; ++u) {
    const int k = s[u].key;
    if (k < 0) continue;
    const int z = k / a.total_bins;
    const int q0 = k > 0 ? cur[k - 1] : 0, q1 = cur[k];
    int rank = 0;
    for (int q = q0; q < q1; ++q) rank += perm[q] < s[u].i ? 1 : 0;
    a.key[s[u].i] = k;
    put_slot(a, base_s[z] + (q0 - lo_s[z]) + rank, s[u]);
  }
  for (int z = 0; z < a.n_species; ++z) {
    const int n = (z + 1 < a.n_species ? lo_s[z + 1] : run) - lo_s[z];
    for (int p = base_s[z] + n + t; p < base_s[z + 1]; p += kScanBlock) pad_slot(a, p, z);
  }
  for (int64_t p = base_s[a.n_species] + t; p < a.n_slots; p += kScanBlock) pad_slot(a, p, 0);
}

// --------------------------------------------------------- Verlet lists

// Smallest and largest value over the wavefront (DPP butterfly towards lane 63;
// lanes without a source keep their own value, which changes neither).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  const int i = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane63(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_min(float v) {
  v = fminf(v, dpp_move<0x111>(v));  // row_shr 1, 2, 4, 8
  v = fminf(v, dpp_move<0x112>(v));
  v = fminf(v, dpp_move<0x114>(v));
  v = fminf(v, dpp_move<0x118>(v));
  v = fminf(v, dpp_move<0x142>(v));  // row_bcast 15, 31
  v = fminf(v, dpp_move<0x143>(v));
  return lane63(v);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_move<0x111>(v));
  v = fmaxf(v, dpp_move<0x112>(v));
  v = fmaxf(v, dpp_move<0x114>(v));
  v = fmaxf(v, dpp_move<0x118>(v));
  v = fmaxf(v, dpp_move<0x142>(v));
  v = fmaxf(v, dpp_move<0x143>(v));
  return lane63(v);
}

// Verlet lists, one home bin per wavefront: the atoms of a bin share their
// candidates (the atoms of the 27 stencil bins with their periodic images).
// The wavefront collects those once, in list order, drops the ones beyond the
// list cutoff from the box of the bin's atoms, and then takes the atoms in
// turn, 64 candidates per round, one per lane.  Kept entries are compacted by
// ballot into a stage in LDS and leave it together.
//
// The list comes out in slot order: slots are ordered by (species, bin key),
// so the stencil bins are visited per species in ascending bin key.
// Neighbouring atoms then tend to have their k-th neighbours in the same
// cache lines.  Each bin is packed with its image code (bin key << 5 | code:
// unique, so the order is total; bin keys are below 2^27).  Along a
// non-periodic direction a stencil bin beyond the cell has no atoms (no
// images): it is skipped.
//
// The entries within rc_angular + skin (the angular part of the list, which
// the reverse index searches) are also kept in their own row-major list, and
// marked in a bit mask over the list (bit k % 32 of word k / 32: entry k is in
// that part).
//
// Grid (bins, parts): part y of a bin takes its atoms y, y + parts, ...; a
// batch of few bins takes several parts, so that a wavefront has a few atoms
// whatever the bin holds.  With SPARSE a wavefront per slot instead: the one of
// every share-th atom of a bin takes that atom and the share - 1 after it, the
// others end at once (see launch_lists).
//
// What bounds it: with one atom per thread and a scan of the 27 bins each, the
// bins of a wavefront's lanes differ in occupancy (45 % of the lanes in use),
// every candidate is a gather of its own, and a small batch leaves all but a
// few SIMDs idle.  Sharing a bin's candidates removes the gathers and fills the
// lanes; what remains is issue: about 520 VALU instructions to set a bin up and
// 97 per atom.  One thread per atom -> one bin per wavefront (us): 900,000
// atoms 610 -> 346, 64 cells of 64..512 atoms 189 -> 35, 3,686 atoms 160 -> 20,
// 64 atoms 77 -> 9.
// Longest lists of a wavefront to the flags (one lane).
__device__ __forceinline__ void note_lengths(int maxR, int maxA, int capR, int capA, int* __restrict__ flags) {
  if ((threadIdx.x & (kWave - 1)) != 0) return;
  // read first, past the L2 of this XCD: few wavefronts raise a value, and atomics
  // on one address run one after another (lists of 900 open cells of 20 atoms that
  // all exceed the capacity: 280 us with an atomic per wavefront, 50 so)
  auto raise = [&](int f, int v) {
    if (v > __hip_atomic_load(&flags[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&flags[f], v);
  };
  raise(kFlagMaxR, maxR);
  raise(kFlagMaxA, maxA);
  raise(kFlagOverflow, maxR > capR || maxA > capA ? 1 : 0);
}

// Bin o of the 27 around bin (b0, b1, b2), packed with its image code; `none` if
// there is nothing (beyond the cell along a non-periodic direction).
__device__ __forceinline__ uint32_t stencil_bin(const CfgDev& C, int b0, int b1, int b2, int o, uint32_t none) {
  int t0 = b0 + o / 9 - 1, t1 = b1 + (o / 3) % 3 - 1, t2 = b2 + o % 3 - 1;
  const int w0 = t0 < 0 ? -1 : (t0 >= C.nb[0] ? 1 : 0);
  const int w1 = t1 < 0 ? -1 : (t1 >= C.nb[1] ? 1 : 0);
  const int w2 = t2 < 0 ? -1 : (t2 >= C.nb[2] ? 1 : 0);
  if ((w0 && !(C.periodic & 1)) || (w1 && !(C.periodic & 2)) || (w2 && !(C.periodic & 4))) return none;
  t0 -= w0 * C.nb[0];
  t1 -= w1 * C.nb[1];
  t2 -= w2 * C.nb[2];
  return ((uint32_t)bin_key(C, t0, t1, t2) << 5) | (uint32_t)((w0 + 1) * 9 + (w1 + 1) * 3 + (w2 + 1));
}

// The bin of a key (see bin_key).
__device__ __forceinline__ void bin_of_key(const CfgDev& C, int k, int& b0, int& b1, int& b2) {
  const int rel = k - C.bin_off, tl = rel >> 6;
  const int nt1 = (C.nb[1] + 3) >> 2, nt2 = (C.nb[2] + 3) >> 2;
  b0 = ((tl / (nt1 * nt2)) << 2) | ((rel >> 4) & 3);
  b1 = (((tl / nt2) % nt1) << 2) | ((rel >> 2) & 3);
  b2 = ((tl % nt2) << 2) | (rel & 3);
}

constexpr int kListRanges = 27 * kListSpecies;  // (species, stencil bin) slot ranges
constexpr int kListCandMin = 512, kListCandMax = 2048;  // candidates listed in LDS (CAND); longer lists are searched
constexpr int kListRegs = 3;                    // rounds of candidates held in registers
constexpr int kListWaves = 1024;                // wavefronts a small batch is split into
constexpr unsigned kListGated = 16384;          // most blocks of a gated launch
constexpr int64_t kListThread = 49152;          // slots from which sparse batches take a thread per atom
template <int CAND, bool SPARSE>
__global__ __launch_bounds__(kWave) void k_build_lists(int64_t n_slots, int n_species, int total_bins, int share,
                                                       const CfgDev* __restrict__ cfgs,
                                                       const float4* __restrict__ pos4, const int* __restrict__ cfg_of,
                                                       const int* __restrict__ orig, const int* __restrict__ key,
                                                       const int* __restrict__ start, const int* __restrict__ base,
                                                       float rclR2, float rclA2, float far0, int capR, int capA,
                                                       int rowTA,
                                                       uint32_t* __restrict__ nbrR, uint32_t* __restrict__ nbrTA,
                                                       uint32_t* __restrict__ angm, int* __restrict__ cntR,
                                                       int* __restrict__ cntAV, int* __restrict__ flags,
                                                       const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  constexpr uint32_t kNoBin = 0xFFFFFFFFu;
  __shared__ uint32_t bin_s[27];
  __shared__ float4 shift_s[27];
  __shared__ int pre_s[kListRanges + 1];
  __shared__ uint32_t first_s[kListRanges];
  __shared__ uint32_t cand_s[CAND];
  __shared__ uint2 st[2 * kWave];  // kept entries waiting for a full round: (entry, |r|^2)
  const int lane = threadIdx.x;
  const int nr = 27 * n_species;
  const int capG = 4 * list_groups(capR);   // entries the groups can hold
  const int capGA = 4 * list_groups(capA);
  const int64_t group_off = group_index(n_slots, 0, lane);
  int zoff[kListSpecies];  // slot of key k of species z: zoff[z] + start[k]
#pragma unroll
  for (int z = 0; z < kListSpecies; ++z) zoff[z] = z < n_species ? base[z] - start[z * total_bins] : 0;
  int maxR = 0, maxA = 0;
  // every XCD takes one contiguous range of bins, or of slots (see xcd_tile)
  const int units = SPARSE ? (int)n_slots : total_bins;
  const int per = (units + (int)kXcds - 1) / (int)kXcds;
  const int b_lo = (int)(blockIdx.x % kXcds) * per;
  const int b_hi = b_lo + per < units ? b_lo + per : units;
  for (int unit = b_lo + (int)(blockIdx.x / kXcds); unit < b_hi; unit += (int)(gridDim.x / kXcds)) {
    int hb = unit, uz = 0;  // the home bin, and with SPARSE the species of the slot
    if constexpr (SPARSE) {
      if (cfg_of[unit] < 0) continue;
      const int k = key[orig[unit]];
      uz = k / total_bins;
      hb = k - uz * total_bins;
    }
    // the bin's atoms: slots hq[z] .. hq[z] + hn[z] - 1 (most padding bins are empty)
    int hq[kListSpecies], hn[kListSpecies], nh = 0;
#pragma unroll
    for (int z = 0; z < kListSpecies; ++z) {
      hq[z] = hn[z] = 0;
      if (z < n_species) {
        const int k = z * total_bins + hb;
        hq[z] = zoff[z] + start[k];
        hn[z] = start[k + 1] - start[k];
      }
      nh += hn[z];
    }
    // the atoms of the bin that this wavefront takes: h0, h0 + step, ... < h1
    int h0 = (int)blockIdx.y, h1 = nh;
    const int step = SPARSE ? 1 : (int)gridDim.y;
    if constexpr (SPARSE) {
      h0 = unit;
#pragma unroll
      for (int z = 0; z < kListSpecies; ++z) h0 += z < uz ? hn[z] : z == uz ? -hq[z] : 0;
      if (h0 % share != 0) continue;
      h1 = h0 + share < nh ? h0 + share : nh;
    }
    if (h0 >= h1) continue;
    // slot of home atom h (clamped to the last)
    auto home = [&](int h) {
      h = h < nh ? h : nh - 1;
      int p = 0, acc = 0;
#pragma unroll
      for (int z = 0; z < kListSpecies; ++z) {
        if (h >= acc && h < acc + hn[z]) p = hq[z] + h - acc;
        acc += hn[z];
      }
      return p;
    };
    int hp = home(lane);  // one home atom per lane
    float4 hx = pos4[hp];
    float lox = hx.x, loy = hx.y, loz = hx.z, hix = hx.x, hiy = hx.y, hiz = hx.z;
    for (int q0 = kWave; q0 < nh; q0 += kWave) {
      const float4 x = pos4[home(q0 + lane)];
      lox = fminf(lox, x.x);
      loy = fminf(loy, x.y);
      loz = fminf(loz, x.z);
      hix = fmaxf(hix, x.x);
      hiy = fmaxf(hiy, x.y);
      hiz = fmaxf(hiz, x.z);
    }
    const CfgDev& C = cfgs[cfg_of[__builtin_amdgcn_readfirstlane(hp)]];
    __syncthreads();  // the previous bin's tables are no longer read
    uint32_t v = kNoBin;
    if (lane < 27) {
      int c0, c1, c2;
      bin_of_key(C, hb, c0, c1, c2);
      v = stencil_bin(C, c0, c1, c2, lane, kNoBin);
      float sx, sy, sz;
      image_shift(C.H, (uint32_t)lane, sx, sy, sz);
      shift_s[lane] = make_float4(sx, sy, sz, 0.f);
    }
    // rank of every bin among the 27; skipped ones at the end
    const uint64_t none = __ballot(lane < 27 && v == kNoBin);
    int rank = 0;
#pragma unroll
    for (int o = 0; o < 27; ++o) rank += (uint32_t)__builtin_amdgcn_readlane(v, o) < v ? 1 : 0;
    if (v == kNoBin) rank += lanes_below(none);
    if (lane < 27) bin_s[rank] = v;
    wave_fence();
    // the slot ranges in list order and the running number of candidates
    int total = 0;
    for (int r0 = 0; r0 < nr; r0 += kWave) {
      const int r = r0 + lane;
      int n = 0;
      uint32_t first = 0;
      if (r < nr) {
        const int z = r / 27;
        const uint32_t b = bin_s[r - 27 * z];
        if (b != kNoBin) {
          const int k = z * total_bins + (int)(b >> 5);
          const int s = start[k];
          n = start[k + 1] - s;
          int zo = zoff[0];
#pragma unroll
          for (int u = 1; u < kListSpecies; ++u) zo = z == u ? zoff[u] : zo;
          first = (uint32_t)(zo + s) | ((b & 31u) << kNbrShift);
        }
      }
      int s = n;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int u = __shfl_up(s, o, kWave);
        if (lane >= o) s += u;
      }
      const int c0 = total + s - n;  // first candidate of this range
      if (r < nr) {
        pre_s[r] = c0;
        first_s[r] = first;
      }
      for (int j = 0; j < n && c0 + j < CAND; ++j) cand_s[c0 + j] = first + (uint32_t)j;
      total += __builtin_amdgcn_readlane(s, kWave - 1);
    }
    if (lane == 0) pre_s[nr] = total;
    wave_fence();
    const bool listed = total <= CAND;
    if (listed) {
      // drop the candidates farther than the list cutoff from the box of the
      // home atoms, keeping the order.  The margin (that of the lattice vectors is in
      // far0) is far above what the roundings of position plus shift here and of the
      // pair vector can differ by: at most an ulp (2^-23) of the coordinates and of
      // the lattice vectors per component (a cell of 1e5 A: 0.02 A).
      lox = wave_min(lox);
      loy = wave_min(loy);
      loz = wave_min(loz);
      hix = wave_max(hix);
      hiy = wave_max(hiy);
      hiz = wave_max(hiz);
      const float reach = fmaxf(fmaxf(fmaxf(fabsf(lox), fabsf(hix)), fmaxf(fabsf(loy), fabsf(hiy))),
                                fmaxf(fabsf(loz), fabsf(hiz)));
      const float far = fmaf(reach, 4e-7f, far0);
      const float far2 = far * far;
      int out = 0;
      for (int c0 = 0; c0 < total; c0 += kWave) {
        const int c = c0 + lane;
        const uint32_t e = cand_s[c < total ? c : total - 1];
        const float4 x = pos4[e & kNbrMask];
        const float4 s = shift_s[e >> kNbrShift];
        const float px = x.x + s.x, py = x.y + s.y, pz = x.z + s.z;
        // distance to the box (the point minus its nearest point in it)
        const float dx = px - __builtin_amdgcn_fmed3f(px, lox, hix);
        const float dy = py - __builtin_amdgcn_fmed3f(py, loy, hiy);
        const float dz = pz - __builtin_amdgcn_fmed3f(pz, loz, hiz);
        const bool keep = c < total && pair_d2(dx, dy, dz) < far2;
        const uint64_t m = __ballot(keep);
        wave_fence();
        if (keep) cand_s[out + lanes_below(m)] = e;
        out += __builtin_popcountll(m);
        wave_fence();
      }
      total = out;
    }
    // entry of candidate c (slot | image code)
    auto cand = [&](int c) -> uint32_t {
      if (listed) return cand_s[c];
      int lo = 0, hi = nr;  // last range with pre_s[lo] <= c
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pre_s[mid] <= c) lo = mid; else hi = mid;
      }
      return first_s[lo] + (uint32_t)(c - pre_s[lo]);
    };
    // the first rounds of candidates, held through all atoms of the bin (a
    // lane without one holds a point that no distance test accepts)
    uint32_t ce[kListRegs];
    float4 cx[kListRegs], cs[kListRegs];
#pragma unroll
    for (int u = 0; u < kListRegs; ++u) {
      const int c = kWave * u + lane;
      ce[u] = cand(c < total ? c : total - 1);
      cx[u] = pos4[ce[u] & kNbrMask];
      cs[u] = shift_s[ce[u] >> kNbrShift];
      if (c >= total) cx[u].x = __builtin_inff();
    }
    for (int h = h0; h < h1; h += step) {
      if (nh > kWave && (h == h0 || (h & (kWave - 1)) < step)) {  // the next 64 home atoms
        hp = home((h & ~(kWave - 1)) + lane);
        hx = pos4[hp];
      }
      const int hl = h & (kWave - 1);
      const int64_t p = __builtin_amdgcn_readlane(hp, hl);
      const float xi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hx.x), hl));
      const float yi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hx.y), hl));
      const float zi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hx.z), hl));
      const uint32_t self = (uint32_t)p | (13u << kNbrShift);
      int kR = 0, kA = 0, ns = 0;  // entries out, angular entries out, entries staged
      uint32_t last_a = 0;
      // the first n staged entries leave as groups and mask words (kR is a
      // multiple of 64 before every call)
      auto emit = [&](int n) {
        wave_fence();
        const uint2 w = st[lane < n ? lane : n - 1];
        const bool ang = lane < n && __uint_as_float(w.y) < rclA2;
        // the last group repeats the last entry
        uint32_t* col = nbrR + 4 * ((int64_t)(kR >> 2) * n_slots + p);
        if (lane < ((n + 3) & ~3) && kR + lane < capG) col[group_off] = w.x;
        const uint64_t am = __ballot(ang);
        if (lane < 2 && 32 * lane < n && kR + 32 * lane < capG)
          angm[(int64_t)((kR >> 5) + lane) * n_slots + p] = (uint32_t)(am >> (32 * lane));
        const int ka = kA + lanes_below(am);
        if (ang && ka < capGA) (nbrTA + p * rowTA)[ka] = w.x;
        if (am) last_a = __builtin_amdgcn_readlane(w.x, 63 - __builtin_clzll(am));
        kA += __builtin_popcountll(am);
        kR += n;
      };
      auto round = [&](uint32_t e, const float4& x, const float4& s) {
        const float rx = (x.x - xi) + s.x, ry = (x.y - yi) + s.y, rz = (x.z - zi) + s.z;
        const float d2 = pair_d2(rx, ry, rz);
        const bool in = d2 < rclR2 && e != self;
        const uint64_t m = __ballot(in);
        if (in) st[ns + lanes_below(m)] = make_uint2(e, __float_as_uint(d2));
        ns += __builtin_popcountll(m);
      };
      auto flush = [&] {
        if (ns < kWave) return;
        emit(kWave);
        const uint2 w = st[kWave + lane];
        wave_fence();
        st[lane] = w;
        ns -= kWave;
      };
#pragma unroll
      for (int u = 0; u < kListRegs; ++u)
        if (kWave * u < total) {
          round(ce[u], cx[u], cs[u]);
          if (u > 0) flush();  // (the first round stages 64 at most)
        }
      for (int c0 = kWave * kListRegs; c0 < total; c0 += kWave) {
        const int c = c0 + lane;
        const uint32_t e = cand(c < total ? c : total - 1);
        float4 x = pos4[e & kNbrMask];
        if (c >= total) x.x = __builtin_inff();
        round(e, x, shift_s[e >> kNbrShift]);
        flush();
      }
      if (ns > 0) emit(ns);
      if ((kA & 3) && kA < capGA && lane < 4 - (kA & 3)) (nbrTA + p * rowTA)[kA + lane] = last_a;
      if (lane == 0) {
        cntR[p] = kR < capR ? kR : capR;
        cntAV[p] = kA < capA ? kA : capA;
      }
      // the angular pairs within rc_angular at any step between rebuilds are
      // among those within rc_angular + skin now, so kA bounds the per-step
      // angular list
      maxR = kR > maxR ? kR : maxR;
      maxA = kA > maxA ? kA : maxA;
      wave_fence();
    }
  }
  note_lengths(maxR, maxA, capR, capA, flags);
}

// The same lists with a thread per atom, for large batches of mostly empty bins: a
// wavefront for each bin's few atoms spends its 520 instructions of set-up on
// them, a thread walks its 27 bins for some 10 candidates.  300,000 atoms in a
// 1,000 A cell, descriptors of the Ge-Sb-Te model: 857 us with a wavefront per
// occupied bin, 449 so; see launch_lists for where the line lies.
//
// The sorted bins wait in the thread's LDS column.  Entries and mask bits shift in
// from the top, so a full group or word holds them in list order; the store
// pointers advance one column at a time.
__global__ __launch_bounds__(256) void k_build_lists_thread(
    int64_t n_slots, int n_species, int total_bins, const CfgDev* __restrict__ cfgs, const float4* __restrict__ pos4,
    const int* __restrict__ cfg_of, const int* __restrict__ orig, const int* __restrict__ key,
    const int* __restrict__ start, const int* __restrict__ base, float rclR2, float rclA2, int capR, int capA,
    int rowTA, uint32_t* __restrict__ nbrR, uint32_t* __restrict__ nbrTA, uint32_t* __restrict__ angm,
    int* __restrict__ cntR, int* __restrict__ cntAV, int* __restrict__ flags, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  constexpr uint32_t kNoBin = 0xFFFFFFFFu;
  __shared__ uint32_t sorted_bins[27 * 256];
  const int64_t p = xcd_tile() * 256 + threadIdx.x;
  const int c = p < n_slots ? cfg_of[p] : -1;
  int kR = 0, kA = 0;
  if (c >= 0) {
    const CfgDev& C = cfgs[c];
    const float4 xi = pos4[p];
    int b0, b1, b2;
    bin_of_key(C, key[orig[p]] % total_bins, b0, b1, b2);
    uint32_t sb[27];
#pragma unroll
    for (int o = 0; o < 27; ++o) sb[o] = stencil_bin(C, b0, b1, b2, o, kNoBin);
#pragma unroll
    for (int i = 1; i < 27; ++i)
#pragma unroll
      for (int j = i; j > 0; --j) {
        const uint32_t lo = sb[j - 1] < sb[j] ? sb[j - 1] : sb[j];
        const uint32_t hi = sb[j - 1] < sb[j] ? sb[j] : sb[j - 1];
        sb[j - 1] = lo;
        sb[j] = hi;
      }
#pragma unroll
    for (int o = 0; o < 27; ++o) sorted_bins[o * 256 + threadIdx.x] = sb[o];
    const int capG = 4 * list_groups(capR);   // entries the groups can hold
    const int capGA = 4 * list_groups(capA);
    uint4 grp = make_uint4(0u, 0u, 0u, 0u), gra = grp;
    uint32_t mword = 0;
    uint4* colG = reinterpret_cast<uint4*>(nbrR) + p;           // next group
    uint4* rowA = reinterpret_cast<uint4*>(nbrTA + p * rowTA);  // angular part
    uint32_t* colM = angm + p;                                  // next mask word
    for (int z = 0; z < n_species; ++z) {
      for (int o = 0; o < 27; ++o) {
        const uint32_t sbo = sorted_bins[o * 256 + threadIdx.x];
        if (sbo == kNoBin) break;
        const uint32_t code = sbo & 31u;
        float sx, sy, sz;
        image_shift(C.H, code, sx, sy, sz);
        const int k = z * total_bins + (int)(sbo >> 5);
        const int q0 = base[z] + start[k] - start[z * total_bins];
        const int q1 = q0 + start[k + 1] - start[k];
        // four candidates per round, loaded together (clamped into the bin)
        for (int q4 = q0; q4 < q1; q4 += 4) {
          float4 xs[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) xs[u] = pos4[q4 + u < q1 ? q4 + u : q1 - 1];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int q = q4 + u;
            if (q >= q1 || (q == (int)p && code == 13u)) continue;
            const float rx = (xs[u].x - xi.x) + sx, ry = (xs[u].y - xi.y) + sy, rz = (xs[u].z - xi.z) + sz;
            const float d2 = pair_d2(rx, ry, rz);
            if (!(d2 < rclR2)) continue;
            const uint32_t e = (uint32_t)q | (code << kNbrShift);
            grp = make_uint4(grp.y, grp.z, grp.w, e);
            mword = (mword >> 1) | (d2 < rclA2 ? 0x80000000u : 0u);
            ++kR;
            if ((kR & 3) == 0 && kR <= capG) {
              *colG = grp;
              colG += n_slots;
            }
            if ((kR & 31) == 0 && kR <= capG) {
              *colM = mword;
              colM += n_slots;
            }
            if (d2 < rclA2) {
              gra = make_uint4(gra.y, gra.z, gra.w, e);
              ++kA;
              if ((kA & 3) == 0 && kA <= capGA) rowA[(kA >> 2) - 1] = gra;
            }
          }
        }
      }
    }
    // the last, partly filled groups (their r entries sit in the top r
    // components: moved down to the front) and mask word
    auto front = [](uint4 g, int r) {
      return r == 1 ? make_uint4(g.w, g.w, g.w, g.w) : r == 2 ? make_uint4(g.z, g.w, g.w, g.w)
                                                             : make_uint4(g.y, g.z, g.w, g.w);
    };
    if ((kR & 3) && kR < capG) *colG = front(grp, kR & 3);
    if ((kR & 31) && (kR & ~31) < capG) *colM = mword >> (32 - (kR & 31));
    if ((kA & 3) && kA < capGA) rowA[kA >> 2] = front(gra, kA & 3);
    cntR[p] = kR < capR ? kR : capR;
    cntAV[p] = kA < capA ? kA : capA;
  }
  note_lengths((int)wave_max((float)kR), (int)wave_max((float)kA), capR, capA, flags);
}

// Reverse index: for every entry k of i's Verlet list whose pair is within
// rc_angular + skin (the angular part of the list), the position of i in the
// angular part of the list of the neighbour j (the entry with i's slot and the
// opposite image code), else 0xFFFFFFFF; 0xFFFFFFFE marks an angular entry
// whose partner was not found, which also raises the asymmetry flag.  The
// pair-force buffer is indexed through these positions, so that each step's
// gather reads without searching.  The angular entries are known from the
// bit mask k_build_lists leaves, and the search reads the angular part of j's
// list only (about a third of the list).
//
// Eight lanes per atom take its angular entries side by side, so the lanes search
// (a thread that owned four entries of a list found one angular among them, and
// compared for all); the results of 64 list entries at a time are put together
// in LDS and leave as whole groups.  Bound by the compares and the latency of
// entry, list length and row.  900,000 atoms 190 -> 132 us, 18,400 atoms 12.6 ->
// 7.9, 3,686 atoms 9.8 -> 5.9.
constexpr int kRevLanes = 8, kRevAtoms = 256 / kRevLanes, kRevSpan = 64;
// Blocks beyond which a gated launch has a block take several tiles: blocks cost
// time even when the gate sends them home at once.
constexpr unsigned kRevGated = 2048;

// Position of the r-th set bit of x (r < popcount).
__device__ __forceinline__ int nth_bit(uint32_t x, int r) {
  int k = 0;
#pragma unroll
  for (int s = 16; s > 0; s >>= 1) {
    const int c = __builtin_popcount(x & ((1u << s) - 1u));
    const bool up = r >= c;
    r -= up ? c : 0;
    x >>= up ? s : 0;
    k += up ? s : 0;
  }
  return k;
}

__global__ __launch_bounds__(256) void k_reverse(int64_t n_slots, const int* __restrict__ cfg_of,
                                                 const uint32_t* __restrict__ nbrR, const uint32_t* __restrict__ nbrTA,
                                                 int rowTA, const uint32_t* __restrict__ angm,
                                                 const int* __restrict__ cntR, const int* __restrict__ cntAV,
                                                 uint32_t* __restrict__ vrev, int* __restrict__ flags,
                                                 const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  __shared__ __align__(16) uint32_t res[kRevAtoms][kRevSpan + 4];
  __shared__ int n_s[kRevAtoms];
  const int t8 = threadIdx.x % kRevLanes, at = threadIdx.x / kRevLanes;
  const int64_t tiles = (n_slots + kRevAtoms - 1) / kRevAtoms;
  bool missing = false;
  for (int64_t tile = xcd_tile(); tile < tiles; tile += gridDim.x) {
    const int64_t p = tile * kRevAtoms + at;
    const int n = p < n_slots && cfg_of[p] >= 0 ? cntR[p] : 0;
    if (t8 == 0) n_s[at] = n;
    for (int k0 = 0; __syncthreads_or(k0 < n); k0 += kRevSpan) {
      for (int x = threadIdx.x; x < kRevAtoms * kRevSpan / 4; x += 256)
        *reinterpret_cast<uint4*>(&res[x % kRevAtoms][x / kRevAtoms * 4]) = make_uint4(~0u, ~0u, ~0u, ~0u);
      // the angular entries among the 64: bits of two words
      const int left = n - k0;
      uint32_t w0 = left > 0 ? angm[(int64_t)(k0 >> 5) * n_slots + p] : 0u;
      uint32_t w1 = left > 32 ? angm[(int64_t)((k0 >> 5) + 1) * n_slots + p] : 0u;
      if (left < 32) w0 &= (1u << (left > 0 ? left : 0)) - 1u;
      else if (left < 64) w1 &= (1u << (left - 32)) - 1u;
      const int c0 = __builtin_popcount(w0), cnt = c0 + __builtin_popcount(w1);
      __syncthreads();
      for (int a = t8; a < cnt; a += kRevLanes) {
        const int k = a < c0 ? nth_bit(w0, a) : 32 + nth_bit(w1, a - c0);
        const uint32_t e = nbrR[group_index(n_slots, p, k0 + k)];
        const int nq = cntAV[e & kNbrMask];
        const uint32_t want = (uint32_t)p | ((26u - (e >> kNbrShift)) << kNbrShift);
        // the angular part of the neighbour's list, row-major, rows padded to a
        // multiple of 4 entries so that the 16-byte reads stay inside the row;
        // entries at or past nq are ignored.  Sixteen entries are read at once.
        const uint4* row = reinterpret_cast<const uint4*>(nbrTA + (int64_t)(e & kNbrMask) * rowTA);
        uint32_t r = 0xFFFFFFFEu;
        for (int j0 = 0; j0 < nq && r == 0xFFFFFFFEu; j0 += 16) {
          uint4 x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = j0 + 4 * u < nq ? row[(j0 >> 2) + u] : make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
          for (int u = 3; u >= 0; --u) {
            const int j = j0 + 4 * u;
            if (x[u].w == want && j + 3 < nq) r = (uint32_t)(j + 3);
            if (x[u].z == want && j + 2 < nq) r = (uint32_t)(j + 2);
            if (x[u].y == want && j + 1 < nq) r = (uint32_t)(j + 1);
            if (x[u].x == want && j < nq) r = (uint32_t)j;
          }
        }
        missing |= r == 0xFFFFFFFEu;
        res[at][k] = r;
      }
      __syncthreads();
      for (int x = threadIdx.x; x < kRevAtoms * kRevSpan / 4; x += 256) {
        const int i = x % kRevAtoms, g = x / kRevAtoms;
        if (k0 + 4 * g < n_s[i])
          reinterpret_cast<uint4*>(vrev)[(int64_t)(k0 / 4 + g) * n_slots + tile * kRevAtoms + i] =
              *reinterpret_cast<const uint4*>(&res[i][4 * g]);
      }
    }
  }
  if (missing) atomicOr(&flags[kFlagAsym], 1);
}

// ---------------------------------------------------------------- host side

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

__global__ void k_fill_int(int* __restrict__ p, int64_t n, int v, const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

void fill_int(hipStream_t st, int* p, int64_t n, int v, const int* gate) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_int, dim3(nblk(n, 256)), dim3(256), 0, st, p, n, v, gate);
}

int DevBuf::ensure(size_t n) {
  if (n <= bytes && p) return NEPMI_OK;
  if (arena) {
    const size_t want = ((n < 256 ? 256 : n) + 255) / 256 * 256;
    if (arena->used + want > arena->cap) {
      set_error("the batch needs more than the " + std::to_string(arena->cap >> 20) +
                " MiB of the allocation-free workspace");
      return NEPMI_INVALID_ARG;
    }
    p = arena->base + arena->used;
    arena->used += want;
    bytes = want;
    return NEPMI_OK;
  }
  release();
  const size_t want = n < 256 ? 256 : n;
  NEPMI_HIP(hipMalloc(&p, want));
  bytes = want;
  return NEPMI_OK;
}

void DevBuf::release() {
  if (p && !arena) (void)hipFree(p);
  p = nullptr;
  bytes = 0;
}

static void cell_geometry(const double* H, double w[3], double Hi[9], double& det) {
  const double *a = H, *b = H + 3, *c = H + 6;
  const double bc[3] = {b[1] * c[2] - b[2] * c[1], b[2] * c[0] - b[0] * c[2], b[0] * c[1] - b[1] * c[0]};
  const double ca[3] = {c[1] * a[2] - c[2] * a[1], c[2] * a[0] - c[0] * a[2], c[0] * a[1] - c[1] * a[0]};
  const double ab[3] = {a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]};
  det = a[0] * bc[0] + a[1] * bc[1] + a[2] * bc[2];
  const double V = fabs(det);
  w[0] = V / sqrt(bc[0] * bc[0] + bc[1] * bc[1] + bc[2] * bc[2]);
  w[1] = V / sqrt(ca[0] * ca[0] + ca[1] * ca[1] + ca[2] * ca[2]);
  w[2] = V / sqrt(ab[0] * ab[0] + ab[1] * ab[1] + ab[2] * ab[2]);
  // rows of Hinv^T are bc, ca, ab divided by det: fractional s_a = x . (col a of Hinv)
  for (int x = 0; x < 3; ++x) {
    Hi[3 * x + 0] = bc[x] / det;
    Hi[3 * x + 1] = ca[x] / det;
    Hi[3 * x + 2] = ab[x] / det;
  }
}

// Free blocks of the pool.
struct PinFree {
  PinFree* next;
};
static std::mutex g_pin_mutex;
static PinFree* g_pin_free = nullptr;

int PinBlock::take() {
  if (p) return NEPMI_OK;
  std::lock_guard<std::mutex> lock(g_pin_mutex);
  if (!g_pin_free) {
    constexpr int kBlocks = 16;  // per chunk
    void* chunk = nullptr;
    NEPMI_HIP(hipHostMalloc(&chunk, kBlocks * kPinBytes,
                            hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent));
    for (int k = 0; k < kBlocks; ++k) {
      PinFree* b = reinterpret_cast<PinFree*>(static_cast<char*>(chunk) + k * kPinBytes);
      b->next = g_pin_free;
      g_pin_free = b;
    }
  }
  p = reinterpret_cast<char*>(g_pin_free);
  g_pin_free = g_pin_free->next;
  return NEPMI_OK;
}

PinBlock::~PinBlock() {
  if (!p) return;
  std::lock_guard<std::mutex> lock(g_pin_mutex);
  PinFree* b = reinterpret_cast<PinFree*>(p);
  b->next = g_pin_free;
  g_pin_free = b;
}

__global__ void k_upload(UploadArgs a) {
  upload_part(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

int Uploader::add(const void* src, size_t bytes, DevBuf& dst) {
  if (tables.size() >= (size_t)UploadArgs::kMost) {
    set_error("too many tables in one upload");
    return NEPMI_INVALID_ARG;
  }
  const int rc = dst.ensure((bytes + 15) / 16 * 16);
  if (rc) return rc;
  tables.push_back({src, &dst, bytes});
  return NEPMI_OK;
}

int Uploader::plan(hipStream_t st, int* clear, int n_clear, UploadArgs& a) {
  size_t total = 0;
  for (const Table& t : tables) total += (t.bytes + 15) / 16 * 16;
  a = UploadArgs{};
  a.clear = clear;
  a.n_clear = n_clear;
  if (total > kPinBytes - kPinMail) {
    for (const Table& t : tables) NEPMI_HIP(hipMemcpyAsync(t.dst->p, t.src, t.bytes, hipMemcpyHostToDevice, st));
    tables.clear();
    return NEPMI_OK;
  }
  char* h = pin + kPinMail;
  for (const Table& t : tables) {
    const size_t n = (t.bytes + 15) / 16;
    memcpy(h, t.src, t.bytes);
    a.seg[a.n_seg].src = reinterpret_cast<const uint4*>(h);
    a.seg[a.n_seg].dst = t.dst->ptr<uint4>();
    a.seg[a.n_seg].n = (int64_t)n;
    ++a.n_seg;
    h += 16 * n;
  }
  tables.clear();
  a.words = (int64_t)(total / 16);
  return NEPMI_OK;
}

static int launch_upload(hipStream_t st, const UploadArgs& a) {
  const int64_t want = (a.words + 255) / 256;
  const unsigned blocks = (unsigned)(want < 1 ? 1 : (want > 256 ? 256 : want));
  hipLaunchKernelGGL(k_upload, dim3(blocks), dim3(256), 0, st, a);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

int Uploader::run(hipStream_t st, int* clear, int n_clear) {
  UploadArgs a;
  const int rc = plan(st, clear, n_clear, a);
  return rc ? rc : launch_upload(st, a);
}

int NbrPipeline::setup(int n_cfg_, const int64_t* atom_off, const double* cells, const int32_t* pbc, int n_species_,
                       double rcR, double rcA, double skin_) {
  if (n_cfg_ < 1 || !atom_off || !cells) {
    set_error("n_cfg must be >= 1 and atom_off, cells non-null");
    return NEPMI_INVALID_ARG;
  }
  if (atom_off[0] != 0) {
    set_error("atom_off[0] must be 0");
    return NEPMI_INVALID_ARG;
  }
  for (int c = 0; c < n_cfg_; ++c)
    if (atom_off[c + 1] < atom_off[c]) {
      set_error("atom_off must be non-decreasing");
      return NEPMI_INVALID_ARG;
    }
  const int64_t N_ = atom_off[n_cfg_];
  if (N_ < 1) {
    set_error("the batch holds no atoms");
    return NEPMI_INVALID_ARG;
  }
  if (N_ > (int64_t)kMaxAtoms - 64 * n_species_) {
    set_error("too many atoms for 27-bit neighbour indices");
    return NEPMI_INVALID_ARG;
  }
  const double rcl = rcR + skin_;
  std::vector<CfgDev> hc((size_t)n_cfg_);
  int64_t bins = 0, real = 0, most = 0;
  double densest = 0.0, longest = 0.0;
  for (int c = 0; c < n_cfg_; ++c) {
    CfgDev& C = hc[(size_t)c];
    const double* H = cells + 9 * (size_t)c;
    double w[3], det;
    cell_geometry(H, w, C.Hinv, det);
    if (!(fabs(det) > 0.0) || !std::isfinite(det)) {
      set_error("singular or non-finite cell");
      return NEPMI_INVALID_ARG;
    }
    C.periodic = 0;
    for (int a = 0; a < 3; ++a) {
      const int32_t pa = pbc ? pbc[3 * (size_t)c + a] : 1;
      if (pa != 0 && pa != 1) {
        set_error("pbc entries must be 0 or 1");
        return NEPMI_INVALID_ARG;
      }
      C.periodic |= pa << a;
      // only a periodic direction needs the width: no pair may meet two
      // images of one atom
      if (pa && w[a] < 2.0 * rcl) {
        set_error("cell width " + std::to_string(w[a]) + " of configuration " + std::to_string(c) +
                  " is below 2 * (rc_radial + skin) = " + std::to_string(2.0 * rcl));
        return NEPMI_CELL_TOO_SMALL;
      }
      // bins a little wider than the list cutoff, so that a position rounded
      // differently by 1e-3 A cannot move a neighbour out of the 27-bin stencil
      int nb = (int)floor(w[a] / (rcl * (1.0 + 1e-6) + 1e-3));
      C.nb[a] = nb < 1 ? 1 : (nb > 1024 ? 1024 : nb);
    }
    for (int x = 0; x < 9; ++x) {
      C.Hd[x] = H[x];
      C.H[x] = (float)H[x];
      longest = std::max(longest, fabs(H[x]));
    }
    C.bin_off = (int)bins;
    C.atom_off = atom_off[c];
    C.n_atoms = (int)(atom_off[c + 1] - atom_off[c]);
    const int64_t nb = (int64_t)C.nb[0] * C.nb[1] * C.nb[2];
    real += nb;
    most = std::max(most, (C.n_atoms + nb - 1) / nb);
    densest = std::max(densest, (double)C.n_atoms / fabs(det));
    bins += (int64_t)((C.nb[0] + 3) / 4) * ((C.nb[1] + 3) / 4) * ((C.nb[2] + 3) / 4) * 64;
  }
  // bin keys below 2^27: the list build packs a key and a 5-bit image code
  // into 32 bits
  if (bins >= (int64_t)1 << 27 || bins * n_species_ > (int64_t)1 << 30) {
    set_error("too many cell bins");
    return NEPMI_INVALID_ARG;
  }
  N = N_;
  n_cfg = n_cfg_;
  n_species = n_species_;
  n_slots = N + (int64_t)kWave * n_species_;
  total_bins = (int)bins;
  real_bins = (int)real;
  bin_atoms = (int)most;
  density = densest;
  skin = skin_;
  const float rlR = (float)(rcR + skin_), rlA = (float)(rcA + skin_);
  rclR2 = rlR * rlR;
  rclA2 = rlA * rlA;
  far0 = (float)(1.0005 * rlR + 5e-4 + 3.0 * 4e-7 * longest);
  host_cfgs = hc;
  host_off.assign(atom_off, atom_off + n_cfg_ + 1);
  const int64_t M = (int64_t)n_species_ * bins;
  const int64_t n_tiles = (M + kScanTile - 1) / kScanTile;
  if (n_tiles > kScanTile) {
    set_error("too many sort keys");
    return NEPMI_INVALID_ARG;
  }
  int rc;
  const size_t Na = (size_t)(N > 0 ? N : 1);
  if (cnt.bytes < 4 * (size_t)(M + 1)) clear_keys = 0;  // the counts get new memory
  // uploaded from the members
  up.tables.clear();
  if ((rc = up.add(host_cfgs.data(), sizeof(CfgDev) * (size_t)n_cfg_, cfgs)) ||
      (rc = up.add(host_off.data(), 8 * (size_t)(n_cfg_ + 1), atom_off_dev)) ||
      (rc = key.ensure(4 * Na)) || (rc = cnt.ensure(4 * (size_t)(M + 1))) || (rc = start.ensure(4 * (size_t)(M + 1))) ||
      (rc = cursor.ensure(4 * (size_t)(M + 1))) || (rc = tile_sums.ensure(4 * (size_t)(n_tiles + 1))) ||
      (rc = base.ensure(4 * (size_t)(n_species_ + 1))) || (rc = perm.ensure(4 * (size_t)n_slots)) ||
      (rc = pos_tmp.ensure(16 * Na)) || (rc = cfg_tmp.ensure(4 * Na)) || (rc = pos4.ensure(16 * (size_t)n_slots)) ||
      (rc = cfg_of.ensure(4 * (size_t)n_slots)) || (rc = orig.ensure(4 * (size_t)n_slots)) ||
      (rc = slot_of.ensure(4 * Na)) ||
      (rc = cntR.ensure(4 * (size_t)n_slots)) || (rc = cntAV.ensure(4 * (size_t)n_slots)) ||
      (rc = ccntR.ensure(4 * (size_t)n_slots)) ||
      (rc = ccntA.ensure(4 * (size_t)n_slots)) ||
      (rc = flags.ensure(4 * kFlagCount)))
    return rc;
  if (capR == 0) {
    // initial capacity from the densest configuration
    const double vR = 4.18879020478639 * rlR * rlR * rlR, vA = 4.18879020478639 * rlA * rlA * rlA;
    capR = (int)(1.5 * density * vR) + 16;
    capA = (int)(1.5 * density * vA) + 16;
  }
  return ensure_lists(capR, capA);
}

void NbrPipeline::use_arena(Arena* a) {
  DevBuf* all[] = {&cfgs, &atom_off_dev, &key, &cnt, &start, &cursor, &tile_sums, &base, &perm, &pos_tmp,
                   &cfg_tmp, &pos4, &cfg_of, &orig, &slot_of, &nbrR, &cntR, &cntAV, &nbrTA, &angm, &vrev,
                   &cnbrR, &ccntR, &cnbrA, &ccntA, &cposA, &flags};
  for (DevBuf* b : all) {
    b->release();
    b->arena = a;
  }
  capR = capA = 0;
  clear_keys = 0;
}

int NbrPipeline::ensure_lists(int capR_, int capA_) {
  if (capR_ > kMaxListRows) {
    // list positions are stored in 16 bits (reverse index, pair buffer rows)
    set_error("more than " + std::to_string(kMaxListRows) + " neighbours within rc_radial + skin");
    return NEPMI_NEIGHBOR_OVERFLOW;
  }
  capR = capR_;
  capA = capA_;
  int rc;
  const size_t ns = (size_t)n_slots;
  rowTA = 4 * list_groups(capA_);
  // the Verlet list, its reverse index and the compact lists are stored in
  // groups of four entries (see list_groups); the angular part of the Verlet
  // list, row-major, in rows of rowTA entries
  if ((rc = nbrR.ensure(16 * (size_t)list_groups(capR) * ns)) || (rc = nbrTA.ensure(4 * (size_t)rowTA * ns)) ||
      (rc = angm.ensure(4 * (size_t)((4 * list_groups(capR) + 31) / 32) * ns)) ||
      (rc = vrev.ensure(16 * (size_t)list_groups(capR) * ns)) ||
      (rc = cnbrR.ensure(16 * (size_t)list_groups(capR) * ns)) ||
      (rc = cnbrA.ensure(16 * (size_t)list_groups(capA) * ns)) ||
      (rc = cposA.ensure(16 * (size_t)list_groups(capA) * ns)))
    return rc;
  return NEPMI_OK;
}

// What the flags say of the input.
static int flag_errors(const int* hf) {
  if (hf[kFlagNaN]) {
    set_error("non-finite position");
    return NEPMI_NAN_DETECTED;
  }
  if (hf[kFlagBadSpecies]) {
    set_error("species index out of range");
    return NEPMI_INVALID_ARG;
  }
  return NEPMI_OK;
}

int NbrPipeline::check_flags(hipStream_t st, int* hf) {
  NEPMI_HIP(hipMemcpyAsync(hf, flags.p, sizeof(int) * kFlagCount, hipMemcpyDeviceToHost, st));
  NEPMI_HIP(hipStreamSynchronize(st));
  longestR = hf[kFlagMaxR];
  longestA = hf[kFlagMaxA];
  return flag_errors(hf);
}

__global__ void k_mail_flags(MailArgs m) { deliver(m); }

static void mail_flags(hipStream_t st, const MailArgs& m) {
  hipLaunchKernelGGL(k_mail_flags, dim3(1), dim3(1), 0, st, m);
}

MailArgs NbrPipeline::post() const {
  MailArgs m;
  if (!unsent) return m;
  m.flags = flags.ptr<int>();
  m.mail = mail();
  return m;
}

int NbrPipeline::build_start(hipStream_t st, const float* pos, const int32_t* species, bool post_later) {
  static_assert(sizeof(int) * (kFlagCount + 1) <= kPinMail, "the flags fit their part of the block");
  int rc;
  UploadArgs u;
  __atomic_store_n(&mail()[kFlagCount], 0, __ATOMIC_RELEASE);
  if ((rc = up.plan(st, flags.ptr<int>(), kFlagCount, u)) ||
      (rc = launch_sort(st, pos, 3, species, n_species, nullptr, nullptr, nullptr, &u)) ||
      (rc = launch_lists(st, n_species, nullptr)))
    return rc;
  unsent = true;
  if (!post_later) mail_flags(st, post());
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

// Wait until the stream has delivered the flags.  The host
// watches the pinned word (a synchronisation of the stream would also wait for
// the work launched behind the lists); every so often it asks the stream, which
// ends the wait if the stream has failed or finished.
static int await_mail(hipStream_t st, const int* mail) {
  for (unsigned n = 1; !__atomic_load_n(&mail[kFlagCount], __ATOMIC_ACQUIRE); ++n) {
    if (n % 16384) {
      __builtin_ia32_pause();
      continue;
    }
    const hipError_t e = hipStreamQuery(st);
    if (e == hipErrorNotReady) {
      (void)hipGetLastError();
      continue;
    }
    if (e != hipSuccess) return hip_fail(e, "hipStreamQuery (neighbour lists)");
    if (__atomic_load_n(&mail[kFlagCount], __ATOMIC_ACQUIRE)) break;
    set_error("the neighbour build ended without its flags");
    return NEPMI_HIP_ERROR;
  }
  return NEPMI_OK;
}

int NbrPipeline::build_end(hipStream_t st, bool& regrown) {
  regrown = false;
  unsent = false;  // delivered by what has been launched
  int* m = mail();
  for (int attempt = 0; attempt < 2; ++attempt) {
    int rc = await_mail(st, m);
    if (rc) return rc;
    int hf[kFlagCount];
    memcpy(hf, m, sizeof hf);
    if ((rc = flag_errors(hf))) return rc;
    longestR = hf[kFlagMaxR];
    longestA = hf[kFlagMaxA];
    if (!hf[kFlagOverflow]) {
      if (hf[kFlagAsym]) {
        set_error("neighbour list is not symmetric");
        return NEPMI_INVALID_ARG;
      }
      return NEPMI_OK;
    }
    if (attempt) break;
    // grow to the largest list seen plus a margin and rebuild the lists
    regrown = true;
    if ((rc = ensure_lists(hf[kFlagMaxR] + 8, hf[kFlagMaxA] + 8))) return rc;
    fill_int(st, flags.ptr<int>(), kFlagCount, 0, nullptr);
    if ((rc = launch_lists(st, n_species, nullptr))) return rc;
    __atomic_store_n(&m[kFlagCount], 0, __ATOMIC_RELEASE);
    unsent = true;
    mail_flags(st, post());
    unsent = false;
    NEPMI_HIP(hipGetLastError());
  }
  set_error("neighbour capacity overflow after regrow");
  return NEPMI_NEIGHBOR_OVERFLOW;
}

int NbrPipeline::launch_sort(hipStream_t st, const float* pos, int pos_stride, const int32_t* species, int n_species,
                             const int* gate, const SlotCarry* carry, const SlotSource* src,
                             const UploadArgs* upload) {
  const int M = n_species * total_bins;
  SortArgs a{};
  a.N = N;
  a.n_slots = n_slots;
  a.n_cfg = n_cfg;
  a.n_species = n_species;
  a.total_bins = total_bins;
  a.atom_off = atom_off_dev.ptr<int64_t>();
  a.cfgs = cfgs.ptr<CfgDev>();
  a.pos = pos;
  a.pos_stride = pos_stride;
  a.species = species;
  if (src) a.src = *src;
  if (carry) a.carry = *carry;
  a.pos_tmp = pos_tmp.ptr<float4>();
  a.cfg_tmp = cfg_tmp.ptr<int>();
  a.key = key.ptr<int>();
  a.cnt = cnt.ptr<int>();
  a.start = start.ptr<int>();
  a.cursor = cursor.ptr<int>();
  a.perm = perm.ptr<int>();
  a.pos4 = pos4.ptr<float4>();
  a.base = base.ptr<int>();
  a.cfg_of = cfg_of.ptr<int>();
  a.orig = orig.ptr<int>();
  a.slot_of = slot_of.ptr<int>();
  a.cntR = cntR.ptr<int>();
  a.cntAV = cntAV.ptr<int>();
  a.flags = flags.ptr<int>();
  const bool small = n_slots <= kSmallAtoms && M <= kSmallKeys;
  // the one block of a small sort takes a small upload along
  const bool along = small && !src && upload && upload->words <= kSmallUpload;
  if (upload && !along) {
    const int rc = launch_upload(st, *upload);
    if (rc) return rc;
  }
  if (small) {
    if (src)
      hipLaunchKernelGGL(k_sort_small<true>, dim3(1), dim3(kScanBlock), 0, st, a, gate, UploadArgs{});
    else
      hipLaunchKernelGGL(k_sort_small<false>, dim3(1), dim3(kScanBlock), 0, st, a, gate,
                         along ? *upload : UploadArgs{});
    NEPMI_HIP(hipGetLastError());
    return NEPMI_OK;
  }
  // the counts are clear: every sort leaves them so (new memory is cleared here)
  if (clear_keys < M) {
    fill_int(st, a.cnt, M, 0, nullptr);
    clear_keys = M;
  }
  if (src)
    hipLaunchKernelGGL(k_stage<true>, dim3(nblk(n_slots, 256)), dim3(256), 0, st, a, gate);
  else
    hipLaunchKernelGGL(k_stage<false>, dim3(nblk(N, 256)), dim3(256), 0, st, a, gate);
  if (M <= (gate ? kOneScanGated : kOneScan)) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanBlock), 0, st, a, gate);
  } else {
    const int n_tiles = (M + kScanTile - 1) / kScanTile;
    hipLaunchKernelGGL(k_scan_tiles, dim3(n_tiles), dim3(kScanBlock), 0, st, a.cnt, M, a.start, tile_sums.ptr<int>(),
                       gate);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanBlock), 0, st, tile_sums.ptr<int>(), n_tiles, a.start, M,
                       total_bins, n_species, a.base, gate);
    hipLaunchKernelGGL(k_scan_add, dim3(nblk(M, 256)), dim3(256), 0, st, a.start, M, tile_sums.ptr<int>(), a.cursor,
                       a.cnt, gate);
  }
  hipLaunchKernelGGL(k_scatter, dim3(nblk(N, 256)), dim3(256), 0, st, a, gate);
  hipLaunchKernelGGL(k_fill_slots, dim3(nblk(n_slots, 256)), dim3(256), 0, st, a, gate);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

int NbrPipeline::launch_lists(hipStream_t st, int n_species, const int* gate) {
  // Candidates of a bin's atoms, from the mean over all bins and, as a hint (the
  // lists are the same either way), from the longest list read last: 27 bins at the
  // density of the atoms that have it.
  const int mean = 27 * bin_atoms, dense = 7 * longestR;
  // Where most bins are empty (a cluster or a gas in a wide cell, many small cells)
  // or the full ones hold far more than the mean, a wavefront per slot, of which
  // those of every share-th atom of a bin work, with the larger candidate table;
  // from kListThread slots on a thread per atom, and sooner.
  // Descriptors of the Ge-Sb-Te model (us), wavefront per bin, per slot, thread per
  // atom: 1,000 atoms in 1,000 A 1450, 150, -; a cluster of 27,000 atoms 1.9 A
  // apart in 600 A 1050, 340, -, in 200 A 824, 323, -; a cluster of 2,197 atoms 2.9 A
  // apart in 100 A (1.7 bins per slot) 110, 125, -; 30,000 atoms spread over 600 A
  // 410, 190, -; 50,000 over 300 A -, 222, 195; 64,000 over 350 A -, 256, 200; a
  // cluster of 64,000 in 600 A 545, 287, 313; 100,000 spread over 300 A (1.4 bins per
  // slot) 293, 344, 230; 300,000 over 1,000 A 1760, 857, 449.
  const bool many = n_slots >= kListThread;
  const bool sparse = total_bins > (many ? 1 : 4) * n_slots || (dense > kListCandMin && dense > 2 * mean);
  if (sparse && many) {
    hipLaunchKernelGGL(k_build_lists_thread, dim3(nblk(n_slots, 256)), dim3(256), 0, st, n_slots, n_species, total_bins,
                       cfgs.ptr<CfgDev>(), pos4.ptr<float4>(), cfg_of.ptr<int>(), orig.ptr<int>(), key.ptr<int>(),
                       start.ptr<int>(), base.ptr<int>(), rclR2, rclA2, capR, capA, rowTA, nbrR.ptr<uint32_t>(),
                       nbrTA.ptr<uint32_t>(), angm.ptr<uint32_t>(), cntR.ptr<int>(), cntAV.ptr<int>(),
                       flags.ptr<int>(), gate);
  } else {
    const int share = (int)std::max<int64_t>(1, N / kListWaves);
    // parts: enough that about one wavefront per SIMD is at work
    const unsigned parts = sparse ? 1u : (unsigned)std::min(bin_atoms, std::max(1, kListWaves / real_bins));
    // without a gate, a block per bin (at 900k atoms 346 us, 371 in 16384 blocks
    // and 437 in 8192: most of a block's bins are alike, but the empty ones and
    // the fuller ones are not spread evenly); with one, fewer blocks, since
    // blocks cost time even when the gate sends them home at once
    const unsigned want = ((unsigned)(sparse ? n_slots : total_bins) + kXcds - 1) / kXcds * kXcds;
    const unsigned blocks = gate && want > kListGated ? kListGated : want;
    // the larger candidate table takes LDS that the smaller one leaves to more
    // wavefronts (lists of 900,000 atoms 361 and 493 us); a third is left for bins
    // fuller than the mean, and a handle's first lists take it in any case: beyond
    // the table every candidate of every atom is searched for (27,000 atoms 1.9 A
    // apart, half of a 150 A cell: 507 us searched, 193 listed, with a thread per atom 329)
    const auto kernel = sparse ? k_build_lists<kListCandMax, true>
                        : longestR > 0 && mean * 4 / 3 <= kListCandMin ? k_build_lists<kListCandMin, false>
                                                                       : k_build_lists<kListCandMax, false>;
    hipLaunchKernelGGL(kernel, dim3(blocks, parts), dim3(kWave), 0, st, n_slots, n_species, total_bins, share,
                       cfgs.ptr<CfgDev>(), pos4.ptr<float4>(), cfg_of.ptr<int>(), orig.ptr<int>(), key.ptr<int>(),
                       start.ptr<int>(), base.ptr<int>(), rclR2, rclA2, far0, capR, capA, rowTA, nbrR.ptr<uint32_t>(),
                       nbrTA.ptr<uint32_t>(), angm.ptr<uint32_t>(), cntR.ptr<int>(), cntAV.ptr<int>(),
                       flags.ptr<int>(), gate);
  }
  const unsigned rev_tiles = (nblk(n_slots, kRevAtoms) + kXcds - 1) / kXcds * kXcds;
  const unsigned rev_blocks = gate && rev_tiles > kRevGated ? kRevGated : rev_tiles;
  hipLaunchKernelGGL(k_reverse, dim3(rev_blocks), dim3(256), 0, st, n_slots, cfg_of.ptr<int>(),
                     nbrR.ptr<uint32_t>(), nbrTA.ptr<uint32_t>(), rowTA, angm.ptr<uint32_t>(), cntR.ptr<int>(),
                     cntAV.ptr<int>(), vrev.ptr<uint32_t>(), flags.ptr<int>(), gate);
  NEPMI_HIP(hipGetLastError());
  return NEPMI_OK;
}

}  // namespace nepmi
