// le_internal.h -- device-side layout shared by the host runtime and the
// kernels of the Lees-Edwards library (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "le.h"

namespace le {

constexpr int kBlock = 256;        // threads per block of the streaming per-particle kernels
// Particles per tile of the list search and of the force kernel with the LDS
// halo (Dev::tile), and per block of the pair kernels without it (kTile).  Small
// systems take small tiles, as many more blocks: 1000 particles are 8 tiles of
// 128, on 8 of 256 CUs.
constexpr int kTile = 128, kTileSmall = 32;
constexpr int kSearchThreads = 512;
// Tile configurations: positions a tile may stage (LDS slot HALO: far
// sentinel), threads per block of the force kernel (shared among the tile's particles),
// whether a batch spreads its blocks over the XCDs.  Sparse systems stage and
// list far fewer partners than dense ones, so they take a smaller halo (more blocks
// per CU) and fewer threads per particle.
struct TileDense { static constexpr int HALO = 2048, kForceThreads = 512; static constexpr bool kSpread = true; };
struct TileSparse { static constexpr int HALO = 1024, kForceThreads = 256; static constexpr bool kSpread = false; };
// without a force-time halo: the dense list search (two blocks per CU beside the
// table of entries it keeps), and the blocks of the force kernel
struct TileDenseGlobal { static constexpr int HALO = 2048; };
struct TileNone { static constexpr int HALO = 0, kForceThreads = kTile; static constexpr bool kSpread = false; };
enum { kTilesDense = 0, kTilesSparse = 1 };
constexpr int kPlainBatch = 8;     // padding of the lists of LDS indices (one 16-byte block)
constexpr int kOtherBatch = 4;     // padding of the lists of global slots
constexpr int kStressComps = 12;   // 6 kinetic + 6 virial partial sums per block
constexpr int kSlots = 64;         // words (one per 128-byte line) a block maximum is spread over
constexpr int kLineInts = 32;      // 32-bit words per 128-byte line
constexpr int kLineU64 = 16;       // 64-bit words per 128-byte line
constexpr int kSortParticles = 512;  // particles per block of the scan-and-permute pass (on average)
// particles up to which a step rebuilds in one launch, and sorts in one, and the blocks
// such a launch may have (see launch_rebuild)
constexpr int kOneLaunch = 20000, kSortOneLaunch = 65536, kWaitBlocks = 512;
constexpr int kBinBlock = 2 * kBlock;  // particles per block of the binning pass (two per thread)

// Mutable per-simulation scalars that live on the device so that a step
// never needs the host: step counter, offset, rebuild bookkeeping.  Two
// copies alternate: the kernel that advances the step reads one and writes
// the other (every block reads, one block writes), so no block ever sees a
// half-updated state; the host passes the current copy to each launch.
struct alignas(64) Ctrl {
  int64_t step;          // index n of the current state
  int64_t rebuild_step;  // step of the last neighbour-list build (m)
  int64_t n_rebuilds;
  double Delta;          // offset of step n, in [0, L_x)
  double Delta_ref;      // offset at the last build
  double drift;          // sum over steps since the build of dt * max |peculiar velocity|
  int32_t pos_cur;       // which position buffer holds the current positions
  int32_t aux_cur;       // which velocity/force/tag buffer is current
  int32_t rebuild;       // kRebuild*: the lists are (being) rebuilt for this state
  int32_t wraps;         // whole L_x folds of the offset since the build
};

enum { kRebuildDue = 1, kRebuildForced = 2 };

// Counts of kernels in one launch: places given out, blocks done of the binning and of
// the scan-and-permute pass, and blocks of the search that have waited.
enum { kPlace = 0, kBinned = 1, kSorted = 2, kWaited = 3, kJoined = 4 };
constexpr int kJoinedLine = 32;    // 64-bit words between the counts (blocks that wait poll one of them)

// Sticky status and telemetry shared by both control copies.
struct alignas(64) Flags {
  int32_t status;        // LE_OK or the first LE_E_* code latched by a kernel
  // largest neighbour count of the last build: max over kSlots words, one per
  // 128-byte line (block b updates word b mod kSlots)
  int32_t max_nb_slot[kSlots * kLineInts];
};

// One 32-byte gather of a DPD partner.
struct alignas(32) VtRec { double x, y, z; int32_t tag, pad; };

// Everything a kernel needs, passed by value.
struct Dev {
  // geometry and physics
  double Lx, Ly, Lz;
  double inv_lx, inv_ly, inv_lz;   // cells per unit length (n_a / L_a)
  double lx;                       // cell length along x
  double shear_rate, sv;           // gamma_dot and gamma_dot * L_y
  // velocity storage (LE_VEL_*): the peculiar velocity is c = u - c_sr (y - L_y/2) e_x,
  // the drift moves x by dt (u_x + drift_sr (y - L_y/2)), a face crossing jumps
  // u_x by -k_y jump_sv.  Lab storage: (gamma_dot, 0, gamma_dot L_y); peculiar
  // storage: (0, gamma_dot, 0).
  double c_sr, drift_sr, jump_sv;
  double dt, h;                    // time step and dt / (2 m)
  double gamma_m;                  // gamma * m
  double pref;                     // sqrt(24 gamma m kT / dt)
  double dpd_gamma, dpd_pref;      // DPD: gamma and sqrt(24 gamma kT / dt)
  double dpd_rc2, dpd_inv_rc;      // DPD: r_c^2 and 1 / r_c of the weight omega
  double mass;
  double eps24, sig2;              // 24 eps, sigma^2
  double lj_c;                     // 48 eps / sigma^2
  double rc2, rlist, rlist2;       // cutoff^2, list radius, list radius^2
  double fene_k, fene_r02;
  double angle_k;                  // cosine angle term of the chains (0: none)
  double force_cap;                // > 0: pair-force magnitude cap (warm-up of overlapping starts)
  double inv_vol;
  int32_t nx, ny, nz, ncell;
  int32_t n, np;                   // particles, padded stride (np > n: slot n is a far-away sentinel)
  int32_t cap, units;              // capacity of a particle's list: entries (a multiple of 16) of either
                                   // kind, and units of 16 bytes (see nl)
  int32_t by_sh, bz_sh;            // log2 of the rows of a beam along y and z (see cell_slot)
  int32_t tile, tile_sh, halo_cap; // particles per tile and their log2, positions it may stage
  int32_t chain_len;
  int32_t n_bonded;                 // n_chains * chain_len (tags >= n_bonded are free)
  int32_t precision;
  int32_t staged;                  // 1: partners in the tile's LDS halo; 0: all from global memory
  int32_t tiles;                   // tile configuration (kTiles*)
  // FP32 pre-test of the list build: r^2 (float) below nb_lo - nb_rel S is
  // certainly inside r_list^2, at or above nb_hi + nb_rel S certainly outside (S:
  // the squared extent of the pair's coordinates, see neighbors_body); in
  // between the plain FP64 displacement decides.
  float nb_lo, nb_hi, nb_rel, rlist_f;
  uint32_t seed_lo, seed_hi;
  uint32_t dpd_key_hi;             // seed_hi ^ 0x44504421: key word of the DPD pair noise
  int32_t thermostat;              // LE_THERMO_*
  int32_t nblocks;                 // blocks of the force kernel (ntiles, or one per kTile particles without the halo)
  // buffers (device)
  double* pos[2];                  // double4 [np] each (x, y, z, wrap counts along y and z)
  double* vel[2];                  // [3][np]
  double* frc[2];                  // [3][np] total force of the current step
  VtRec* vt;                       // DPD only: [np] velocity and tag of the current slots,
                                   // packed before each force evaluation (one gather per partner)
  int32_t* tag[2];                 // slot -> tag
  int32_t* slot_of_tag;            // tag -> slot
  int32_t bcap;                    // bucket capacity per cell
  int2* bucket;                    // [ncell][bcap] (tag, slot) of the particles binned into each
                                   // cell, in arrival order
  int32_t* cell_count;             // [ncell]
  int32_t* cell_start;             // [ncell + 1]
  // Neighbour lists: `units` units of 16 bytes per particle, unit u of particles
  // i, i + 1, ... contiguous (u np + i).
  //   partners found in the tile's staged halo, from unit 0 up: LDS indices, 8 (16-bit)
  //     per unit (halo layout), or slots in global memory in the low kSlotBits bits with
  //     the image code (pack_img) above them, 4 per unit (global layout)
  //   partners of rows that did not fit, from the last unit down: slots and codes
  uint4* nl;
  int32_t* n_plain;                // [np] entries from the front, a multiple of 8 (halo layout) or 4
  int32_t* n_og;                   // [np] entries from the back, a multiple of 4
  // [ntiles][halo_cap] slot and image code (og_entry) of each LDS position.  Shares its memory with
  // the buckets, which only hold values from the binning to the end of the sort.
  uint32_t* halo;
  int32_t* tile_nstage;            // [ntiles] staged positions per tile
  int32_t ntiles;
  int32_t* bond;                   // [2][np] slot of the chain neighbour below/above, -1 if none
  double* partials;                // [nblocks][kStressComps]
  double* obs_part;                // [ceil(n / kBlock)][3 * LE_MAX_BINS + 4] observable partials
  Ctrl* ctrl;                      // current control copy (see Ctrl)
  Ctrl* ctrl_other;                // the other control copy (written by a batched rebuild test)
  // running max of |c|^2 of the last drift (bits of doubles >= 0) in kSlots
  // words of kLineU64 stride; two arrays alternate with the control copies
  unsigned long long* vmax;
  unsigned long long* vmax_other;  // the speed-bound slots paired with ctrl_other
  unsigned long long* scan_status; // [sp_blocks] look-back words of the cell scan
  unsigned long long* joined;      // [kJoined] counts of kernels in one launch (zero between rebuilds)
  int32_t sp_cells, sp_blocks;     // cells per block of the scan-and-permute pass, and its blocks
  Flags* flags;
};

// Descriptor table of a batched launch: simulation k owns the blocks
// [start[k], start[k+1]) of the grid and reads its descriptor (a Dev kept in
// its own workspace, one per control copy) through dev[k].  Passed by value.
constexpr int kMaxBatch = 64;
struct Batch {
  int32_t nsims;
  int32_t start[kMaxBatch + 1];
  const Dev* dev[kMaxBatch];
};
struct BatchOut {
  double* ptr[kMaxBatch];  // per-simulation output (the stress sample of this step)
};

// Entries of the lists of global slots: slot | code << kSlotBits (codes use 7 bits).
constexpr int kSlotBits = 24;
constexpr uint32_t kSlotMask = (1u << kSlotBits) - 1u;
__host__ __device__ inline uint32_t og_entry(uint32_t slot, uint8_t code) {
  return slot | ((uint32_t)code << kSlotBits);
}

// Image code of an imaged neighbour: sx in [-3, 3], sy and sz in [-1, 1].
__host__ __device__ inline uint8_t pack_img(int sx, int sy, int sz) {
  return (uint8_t)((sx + 3) | ((sy + 1) << 3) | ((sz + 1) << 5));
}
__host__ __device__ inline void unpack_img(uint8_t c, int& sx, int& sy, int& sz) {
  sx = (int)(c & 7) - 3;
  sy = (int)((c >> 3) & 3) - 1;
  sz = (int)((c >> 5) & 3) - 1;
}

// Launchers (le_kernels.hip).  Each enqueues on `stream` and returns the
// hipError_t of the launch.
enum ForceMode { kForcesOnly = 0, kStepFused = 1, kStepLast = 2, kInitForce = 3, kDpdForce = 4 };

// launch_rebuild reads control copy d.ctrl and writes `next`, which the
// following launches must then be given.  control: advance the step first
// (after a drift); force: rebuild whatever the criterion says.
hipError_t launch_rebuild(const Dev& d, Ctrl* next, unsigned long long* next_vmax, hipStream_t s,
                          bool force, bool control);
hipError_t launch_kick_drift(const Dev& d, hipStream_t s);
// DPD steps: the force kernel (kDpdForce) only writes the total force; this
// kernel then applies the second half-kick (and, unless last, the next
// half-kick and drift), with kinetic stress partials when sample is set.
hipError_t launch_integrate(const Dev& d, hipStream_t s, bool last, bool sample);
hipError_t launch_force(const Dev& d, hipStream_t s, ForceMode mode, bool sample, double* f_out,
                        double* sample_out, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_stress_final(const Dev& d, hipStream_t s, double* out6, bool virial_only);
hipError_t launch_observables(const Dev& d, hipStream_t s, int nbins, double* out);
hipError_t launch_unwrapped(const Dev& d, hipStream_t s, double* out);
hipError_t launch_msd(const Dev& d, hipStream_t s, const double* ref, double* out2);
hipError_t launch_ctrl_copy(const Ctrl* src, Ctrl* dst, const unsigned long long* vsrc,
                            unsigned long long* vdst, hipStream_t s);
hipError_t launch_state_out(const Dev& d, hipStream_t s, double* x, double* u, int32_t* cell_of,
                            int32_t* order);
hipError_t launch_pairs_out(const Dev& d, hipStream_t s, int64_t* pairs, int64_t cap,
                            unsigned long long* counter);
hipError_t launch_load_state(const Dev& d, hipStream_t s, const double* x0, const double* u0,
                             const double* f0, int64_t step0, double Delta0);
hipError_t launch_status_out(const Dev& d, hipStream_t s, int32_t* out);

// Batched launchers: one launch over the blocks of every simulation of a
// batch (all of one kernel configuration, given by `cfg`, the host copy of any
// member's descriptor).  Batches by block kind: `par` one block per kBlock
// particles, `bin` one per kBinBlock particles, `scan` one per sp_cells cells,
// `tile` one per tile, `blk` one per block of the force kernel,
// `one` one block per simulation; `cur` and `nxt` name the descriptors of the
// current and the other control copy.
hipError_t launch_store_dev(const Dev& a, const Dev& b, Dev* dst, hipStream_t s);
hipError_t launch_kick_drift_b(const Batch& par_cur, hipStream_t s);
hipError_t launch_sort_b(const Batch& bin_cur, const Batch& scan_nxt, hipStream_t s);
hipError_t launch_search_b(const Batch& tile_nxt, const Dev& cfg, hipStream_t s);
hipError_t launch_force_b(const Batch& blk_cur, const Batch& par_cur, const Dev& cfg, hipStream_t s,
                          ForceMode mode, bool sample);
hipError_t launch_integrate_b(const Batch& blk_cur, hipStream_t s, bool last, bool sample);
hipError_t launch_stress_final_b(const Batch& one_cur, const BatchOut& out, hipStream_t s);
hipError_t launch_offsets(double sr, double Lx, double Ly, double dt, int64_t step0, int64_t count,
                          double* out, hipStream_t s);
hipError_t launch_philox(const uint32_t* ctr, const uint32_t* key, uint32_t* out, int64_t count,
                         hipStream_t s);

// Offset of step n: fmod(gamma_dot L_y * (n dt), L_x) folded into [0, L_x).
// fmod is exact, so host and device agree bit for bit.
__host__ __device__ inline double le_offset(int64_t n, double dt, double sv, double Lx) {
  double t = (double)n * dt;
  double d = fmod(sv * t, Lx);
  if (d < 0.0) d += Lx;
  if (d >= Lx) d -= Lx;
  return d;
}

}  // namespace le
