// le_kernels.hip -- gfx950 kernels of the Lees-Edwards shear-flow MD step.
//
// Compiled with -ffp-contract=off: every product and sum below rounds as
// written, which keeps the boundary crossing, cell index and pair
// displacement bit-identical to their plain definitions; fused multiply-adds
// are requested explicitly (fma) only where results are compared with a
// tolerance (force law, accumulations).
//
// Data layout (all sorted by (cell, tag) at every neighbour-list build, the
// cells in beam order, see cell_slot):
//   positions  double4 AoS (x, y, z, wrap counts) -- one 32-byte gather per neighbour
//   velocities, forces  float64 SoA [3][np] -- streamed, coalesced
//   neighbour lists  units of 16 bytes, unit u of consecutive particles contiguous
#include <math.h>

#include <type_traits>

#include <hip/hip_ext.h>

#include "le_internal.h"

namespace le {

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ int xcd_map(int b, int nblocks) {
  // Blocks are dealt round-robin to the 8 XCDs; remap so that each XCD works
  // on one contiguous range of cell-sorted particles (its L2 then holds that
  // region's neighbour positions).
  const int X = 8;
  int q = nblocks / X, r = nblocks % X;
  int x = b % X, k = b / X;
  return x * q + (x < r ? x : r) + k;
}
__device__ __forceinline__ int xcd_block(int nblocks) { return xcd_map((int)blockIdx.x, nblocks); }

// The other way round: runs of C consecutive blocks are dealt round-robin to
// the XCDs, so that any stretch of the grid (the tiles of the members of a
// batch that rebuild at this step) is spread over all of them.
template <int C>
__device__ __forceinline__ int xcd_spread(int b, int nblocks) {
  const int X = 8, G = X * C;
  const int full = nblocks / G * G;
  if (b >= full) return b;
  const int x = b % X, k = b / X;
  return ((k / C) * X + x) * C + k % C;
}

// Simulation and local block of global block g of a batched launch: the last
// simulation whose first block is at or before g (simulations without blocks
// are skipped).  Uniform across the block.
__device__ __forceinline__ void locate(const Batch& b, int g, int& sim, int& bid) {
  int lo = 0, hi = b.nsims - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b.start[mid] <= g) lo = mid; else hi = mid - 1;
  }
  sim = lo;
  bid = g - b.start[lo];
}

// The descriptor of a batched launch's simulation.  It never changes while
// kernels run (written once at le_init), so it is read as constant memory:
// through an address-space-4 pointer the loads become scalar loads into SGPRs,
// as for the by-value descriptor of a single-simulation launch.
static_assert(sizeof(Dev) % 8 == 0, "the descriptor is a whole number of 8-byte words");
typedef const __attribute__((address_space(4))) Dev ConstDev;
__device__ __forceinline__ const Dev& stage_dev(const Dev* src) {
  return *(const Dev*)(ConstDev*)src;
}

__device__ __forceinline__ void latch(Flags* f, int32_t st) { atomicCAS(&f->status, 0, st); }

// Canonical periodic wrap into [0, L); returns the net number of box lengths
// subtracted (the Lees-Edwards crossing count for the gradient axis).
__device__ __forceinline__ double wrap1(double& x, double L) {
  double k = floor(x / L);
  double v = x - k * L;
  if (v < 0.0) { v += L; k -= 1.0; }
  if (v >= L) { v -= L; k += 1.0; }
  x = v;
  return k;
}

// The fourth word of each position holds the particle's wrap counts along y
// and z since le_init (two int32 in the bits of the double; only ever copied,
// never used in arithmetic).
__device__ __forceinline__ void img_get(double w, int& ky, int& kz) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(w);
  ky = (int)(uint32_t)(b >> 32);
  kz = (int)(uint32_t)(b & 0xffffffffull);
}
__device__ __forceinline__ double img_put(int ky, int kz) {
  const unsigned long long b = ((unsigned long long)(uint32_t)ky << 32) | (unsigned long long)(uint32_t)kz;
  return __longlong_as_double((long long)b);
}


__device__ __forceinline__ int cell_index(double v, double inv, int n) {
  int k = (int)(v * inv);
  if (k < 0) k = 0;
  if (k > n - 1) k = n - 1;
  return k;
}

// Place of a cell in the order of the slots.  Rows along x are grouped into
// beams of 2^by_sh x 2^bz_sh rows (narrower at the box's upper faces); the
// beams follow one another along y, then z, a beam's cells run slice by slice
// along x, and the rows of a slice in a serpentine (y up and down along z, every
// other slice backwards), so that consecutive slots lie in adjacent cells and a tile
// of consecutive slots is compact.
__device__ __forceinline__ int cell_slot(const Dev& d, int ix, int iy, int iz) {
  const int y0 = iy >> d.by_sh << d.by_sh, z0 = iz >> d.bz_sh << d.bz_sh;
  const int h = min(1 << d.by_sh, d.ny - y0), w = min(1 << d.bz_sh, d.nz - z0);
  const int zz = iz - z0;
  int r = (zz & 1) ? (zz + 1) * h - 1 - (iy - y0) : zz * h + (iy - y0);
  if (ix & 1) r = h * w - 1 - r;
  return d.nx * (z0 * d.ny + w * y0) + ix * (h * w) + r;
}

__device__ __forceinline__ int floor_div(int a, int b) {
  int q = a / b;
  if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
  return q;
}

__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Philox4x32-10: two 32x32->64 products per round with the published
// multipliers, key advanced by the published Weyl increments between rounds.
__device__ __forceinline__ void philox(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    // one 32 x 32 -> 64-bit product per multiplier (a single v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c[2];
    uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    // (the three-input exclusive or, one instruction instead of two)
    uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c[1], k0, 0x96);
    uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c[3], k1, 0x96);
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
  }
}

__device__ __forceinline__ double u01c(uint32_t r) {
  return fma((double)r, 1.0 / 4294967296.0, 0.5 / 4294967296.0 - 0.5);  // (exact)
}

// ---------------------------------------------------------- state loading
__global__ void k_load_state(Dev d, const double* __restrict__ x0, const double* __restrict__ u0,
                             const double* __restrict__ f0, int64_t step0, double Delta0) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = d.n, np = d.np;
  if (i < n) {
    double4 p;
    p.x = x0[i]; p.y = x0[n + i]; p.z = x0[2 * n + i]; p.w = 0.0;
    reinterpret_cast<double4*>(d.pos[0])[i] = p;
    for (int a = 0; a < 3; ++a) {
      d.vel[0][a * np + i] = u0 ? u0[a * n + i] : 0.0;  // no velocities: particles at rest
      d.frc[0][a * np + i] = f0 ? f0[a * n + i] : 0.0;
    }
    d.tag[0][i] = i;
  }
  if (i == 0) {
    // far-away sentinel at slot n pads neighbour batches: r^2 ~ 1e200 never passes a cutoff
    const double4 far = make_double4(1e100, 1e100, 1e100, 0.0);
    reinterpret_cast<double4*>(d.pos[0])[n] = far;
    reinterpret_cast<double4*>(d.pos[1])[n] = far;
    if (d.vt) d.vt[n] = VtRec{0.0, 0.0, 0.0, 0, 0};  // (its DPD record: finite, its weight is 0)
  }
  for (int c = i; c < d.ncell; c += gridDim.x * blockDim.x) d.cell_count[c] = 0;
  if (i == 0) {
    Ctrl* c = d.ctrl;
    c->step = step0;
    c->rebuild_step = step0;
    c->n_rebuilds = 0;
    c->Delta = Delta0;
    c->Delta_ref = Delta0;
    c->drift = 0.0;
    c->pos_cur = 0;
    c->aux_cur = 0;
    c->rebuild = 0;
    c->wraps = 0;
    d.flags->status = 0;
    for (int k = 0; k < kJoined; ++k) d.joined[k * kJoinedLine] = 0ull;
    for (int k = 0; k < kSlots * kLineInts; ++k) d.flags->max_nb_slot[k] = 0;
  }
  for (int k = i; k < kSlots * kLineU64; k += gridDim.x * blockDim.x) d.vmax[k] = 0ull;
}

// ------------------------------------------------------------- rebuild
// Three parts: (1) advance the step and decide, then bin by the cell of the crossed and
// wrapped position, (2) cell-count scan and, block by block, rank by tag, cross, wrap and
// permute, (3) neighbour lists.  They are three launches, two or one (launch_rebuild),
// each an empty one unless the lists are rebuilt for the current state.

// Advance the step counter and the offset, adopt the drifted positions, and
// decide whether the neighbour lists must be rebuilt before the next force
// evaluation.  Pair displacements evolve as d' = d + dt (c_i - c_j) +
// gamma_dot dt d_y e_x, so after a strain s = |gamma_dot| (t - t_build) and a
// peculiar path bound D = sum dt max|c|, a pair within rc now was within
// g (rc + 2 g D) at the build, g = s/2 + sqrt(1 + s^2/4) the norm of the
// inverse shear.  The lists (radius rc + skin) stay complete while that bound
// is below rc + skin.  Pure: every block evaluates it on its own copy.
__device__ __forceinline__ void control_advance(const Dev& d, Ctrl& c, unsigned long long vbits) {
  double vmax = sqrt(__longlong_as_double((long long)vbits));
  c.drift += d.dt * vmax;
  c.step += 1;
  c.Delta = le_offset(c.step, d.dt, d.sv, d.Lx);
  c.pos_cur ^= 1;
  double T = (double)(c.step - c.rebuild_step) * d.dt;
  c.wraps = (int)rint((c.Delta_ref + d.sv * T - c.Delta) / d.Lx);
  double s = fabs(d.shear_rate) * T;
  double g = 0.5 * s + sqrt(1.0 + 0.25 * s * s);
  double rc = sqrt(d.rc2);
  double need = g * (rc + 2.0 * g * c.drift);
  c.rebuild = (d.rlist <= rc || need >= d.rlist * (1.0 - 1e-9)) ? 1 : 0;
}

// The bookkeeping of a rebuild, applied to the state the rebuild produces:
// sorted copies go to the other buffers, the offset and step become the
// reference of the co-moving criterion.
__device__ __forceinline__ void rebuild_adopt(Ctrl& c, bool forced) {
  c.pos_cur ^= 1;
  c.aux_cur ^= 1;
  c.rebuild = forced ? kRebuildForced : kRebuildDue;
  c.rebuild_step = c.step;
  c.Delta_ref = c.Delta;
  c.drift = 0.0;
  c.wraps = 0;
  c.n_rebuilds += 1;
}

// (both words read unconditionally, so that the two loads overlap: this is
// all an empty launch of the chain does)
__device__ __forceinline__ bool rebuild_off(const Dev& d) {
  const int status = d.flags->status;
  const int rebuild = d.ctrl->rebuild;
  return (status != 0) | (rebuild == 0);
}

// Boundary crossing of one particle (Lees-Edwards shift; the velocity jump is
// -ky jump_sv) + periodic wrap of x and z.  Non-finite coordinates become 0.
__device__ __forceinline__ bool cross_wrap(const Dev& d, double Delta, double& x, double& y, double& z,
                                           double& ky, double& kz) {
  ky = wrap1(y, d.Ly);
  x = x - ky * Delta;
  wrap1(x, d.Lx);
  kz = wrap1(z, d.Lz);
  const bool fine = isfinite(x) && isfinite(y) && isfinite(z);
  if (!fine) { x = 0.0; y = 0.0; z = 0.0; }
  return fine;
}

// (1) Reads control copy d.ctrl and writes the next one (block 0).  With
// `control` the step is advanced first (after a drift).  On a rebuild: each
// particle's tag and slot go into the bucket of the cell that its position
// lies in after crossing and wrap, at its arrival rank.  Runs of equal cells
// within a wave take one atomic per run.  Reads positions and tags alone: the
// crossing is applied where the particle is copied, (2); applied and written
// here it cost the pass 12.6 instead of 9 us (400,000 beads).
//
// The control part: true on a rebuild, with the copies of the state being
// binned (sc) and of the sorted one (sn) in shared memory.
__device__ __forceinline__ bool sort_control(const Dev& d, Ctrl* __restrict__ next,
                                             unsigned long long* __restrict__ next_vmax, int force, int control,
                                             int bid, Ctrl& sc, Ctrl& sn) {
  __shared__ int go;
  if (threadIdx.x < 64) {
    // the drift's speed bound: max over the slot words (first wave)
    unsigned long long vb = threadIdx.x < kSlots ? d.vmax[threadIdx.x * kLineU64] : 0ull;
    for (int o = 32; o > 0; o >>= 1) {
      unsigned long long t = __shfl_xor(vb, o, 64);
      vb = t > vb ? t : vb;
    }
    const bool ok = d.flags->status == 0;
    Ctrl c = *d.ctrl;
    if (ok && control) control_advance(d, c, vb);
    const bool rb = ok && (force || c.rebuild);
    if (threadIdx.x == 0) {
      sc = c;
      c.rebuild = 0;
      if (rb) rebuild_adopt(c, force != 0);
      sn = c;
      if (bid == 0) *next = c;
      go = rb ? 1 : 0;
    }
    if (bid == 0 && threadIdx.x < kSlots) next_vmax[threadIdx.x * kLineU64] = 0ull;
  }
  __syncthreads();
  return go != 0;
}

template <int TH>
__device__ __forceinline__ void bin_body(const Dev& d, const Ctrl& sc, int bid) {
  // the look-back words of the scan start cleared (spread over the blocks)
  const int nbb = (d.n + kBinBlock - 1) / kBinBlock;  // blocks of this pass
  for (int k = bid * TH + (int)threadIdx.x; k < d.sp_blocks; k += nbb * TH) d.scan_status[k] = 0ull;
  if (bid == 0)
    for (int k = threadIdx.x; k < kSlots * kLineInts; k += TH) d.flags->max_nb_slot[k] = 0;
  for (int rd = 0; rd < kBinBlock / TH; ++rd) {
    const int i = bid * kBinBlock + rd * TH + (int)threadIdx.x;
    int cell = -1, tg = 0;
    if (i < d.n) {
      tg = d.tag[sc.aux_cur][i];
      const double4 p = reinterpret_cast<const double4*>(d.pos[sc.pos_cur])[i];
      double x = p.x, y = p.y, z = p.z, ky, kz;
      // (here too: all such particles meet in one cell, whose bucket they may overflow)
      if (!cross_wrap(d, sc.Delta, x, y, z, ky, kz)) latch(d.flags, LE_E_NONFINITE);
      int ix = cell_index(x, d.inv_lx, d.nx);
      int iy = cell_index(y, d.inv_ly, d.ny);
      int iz = cell_index(z, d.inv_lz, d.nz);
      cell = cell_slot(d, ix, iy, iz);
    }
    // runs of equal cells among consecutive lanes share one atomic
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(cell, 1, 64);
    const bool head = lane == 0 || prev != cell;
    const unsigned long long heads = __ballot(head);
    const int run0 = 63 - __clzll(heads & ((2ull << lane) - 1ull));  // lane 63: mask all ones
    const unsigned long long after = lane == 63 ? 0ull : (heads & ~((2ull << lane) - 1ull));
    const int run1 = after ? __ffsll((long long)after) - 1 : 64;  // first lane of the next run
    int base = 0;
    if (head && cell >= 0) base = atomicAdd(&d.cell_count[cell], run1 - lane);
    base = __shfl(base, run0, 64);
    if (cell >= 0) {
      const int r = base + (lane - run0);
      if (r < d.bcap) d.bucket[(size_t)cell * d.bcap + r] = make_int2(tg, i);
      else latch(d.flags, LE_E_CAPACITY);
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_control_bin(Dev d, Ctrl* __restrict__ next,
                                                        unsigned long long* __restrict__ next_vmax,
                                                        int force, int control) {
  __shared__ Ctrl sc, sn;
  if (sort_control(d, next, next_vmax, force, control, blockIdx.x, sc, sn)) bin_body<kBlock>(d, sc, blockIdx.x);
}

// Batched form: every simulation advances its step (control) and writes its
// other control copy (named by its descriptor).
__global__ void __launch_bounds__(kBlock) k_control_bin_b(Batch b) {
  __shared__ Ctrl sc, sn;
  int sm, bid;
  locate(b, blockIdx.x, sm, bid);
  const Dev& d = stage_dev(b.dev[sm]);
  if (sort_control(d, d.ctrl_other, d.vmax_other, 0, 1, bid, sc, sn)) bin_body<kBlock>(d, sc, bid);
}

// (2) One pass over the cells in blocks of sp_cells consecutive cells.  The
// exclusive scan of the cell counts into cell_start uses decoupled
// look-back: block b publishes its total in status word b (flag 1), adds the
// totals of its predecessors walking back (64 at a time, one per lane of the
// first wave) until one has published its inclusive prefix (flag 2), and
// publishes its own.  A word packs flag << 62 | value, so one 64-bit atomic
// carries both.  Every block publishes its total before it waits, and blocks
// start in grid order, so the oldest unfinished block never waits on one
// that has not started: every wait ends; a bounded spin latches LE_E_STATE
// rather than hang.  The counts are cleared for the next binning pass.
//
// With its slots known, the block moves the particles of its own cells: the
// final slot of a particle is its cell's start plus the number of cell-mates
// with a smaller tag, so the order is (cell, tag) whatever the arrival order.
// The bucket entry carries the particle's binned slot; its state is copied
// from there, crossed and wrapped, to the final slot in the other buffers.  No block reads what
// another writes, so the sort needs no further pass.
__device__ __forceinline__ unsigned long long scan_word(int flag, long long v) {
  return ((unsigned long long)flag << 62) | (unsigned long long)v;
}

template <int TH>
__device__ __forceinline__ void scan_permute_body(const Dev& d, const Ctrl& cn, int b) {
  __shared__ int lpre[kBlock + 1];  // exclusive prefix of the block's counts, total last
  __shared__ int wsum[TH / 64];
  __shared__ long long base_sh;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int c0 = b * d.sp_cells;
  const int ncb = min(d.sp_cells, d.ncell - c0);  // cells of this block (>= 1)
  const int v = (int)threadIdx.x < ncb ? d.cell_count[c0 + threadIdx.x] : 0;
  int incl = v;
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  int woff = 0, agg = 0;
  for (int w = 0; w < TH / 64; ++w) {
    if (w < wid) woff += wsum[w];
    agg += wsum[w];
  }
  if ((int)threadIdx.x < ncb) lpre[threadIdx.x] = woff + incl - v;
  if (threadIdx.x == 0) lpre[ncb] = agg;
  if (wid == 0) {
    // look back with the whole first wave: lane l reads the word of block
    // p - l, so one round covers 64 predecessors; the prefix is the sum of
    // the aggregates up to and including the nearest inclusive prefix
    unsigned long long* st = d.scan_status;
    const unsigned long long vmask = (1ull << 62) - 1ull;
    long long prefix = 0;
    if (lane == 0)
      __hip_atomic_store(&st[b], scan_word(b == 0 ? 2 : 1, agg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int p = b - 1;
    long long spins = 0;
    while (p >= 0) {
      const int q = p - lane;
      // before block 0 the prefix is an inclusive 0
      const unsigned long long w =
          q >= 0 ? __hip_atomic_load(&st[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : scan_word(2, 0);
      const int flag = (int)(w >> 62);
      const unsigned long long inc = __ballot(flag == 2);
      const unsigned long long zero = __ballot(flag == 0);
      const int first2 = inc ? __builtin_ctzll(inc) : 64;
      const unsigned long long need = first2 >= 63 ? ~0ull : ((2ull << first2) - 1ull);
      if (zero & need) {  // a predecessor in reach has not published yet
        // (nor will it after a latched error: blocks that find one at their start leave)
        ++spins;
        const bool fault =
            (spins & 15) == 0 && __hip_atomic_load(&d.flags->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        if (fault || spins > (1ll << 22)) {
          if (lane == 0) latch(d.flags, LE_E_STATE);
          prefix = -1;  // no prefix: the block moves nothing
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      long long val = lane <= first2 ? (long long)(w & vmask) : 0;
      for (int o = 32; o > 0; o >>= 1) val += __shfl_xor(val, o, 64);
      prefix += val;
      if (first2 < 64) break;
      p -= 64;
    }
    if (lane == 0) {
      if (b > 0 && prefix >= 0)
        __hip_atomic_store(&st[b], scan_word(2, prefix + agg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      base_sh = prefix;
    }
  }
  __syncthreads();
  if (base_sh < 0) return;
  const int base = (int)base_sh;
  if ((int)threadIdx.x < ncb) {
    d.cell_start[c0 + threadIdx.x] = base + lpre[threadIdx.x];
    d.cell_count[c0 + threadIdx.x] = 0;
  }
  if (c0 + ncb == d.ncell && threadIdx.x == 0) d.cell_start[d.ncell] = base + agg;  // = n

  // the block's particles, two per thread and round (their loads overlap):
  // k-th cell of the block with lpre[k] <= f < lpre[k + 1], arrival rank
  // r = f - lpre[k]; the bucket entry holds the tag and the binned slot
  const int np = d.np;
  const int pd = cn.pos_cur, ad = cn.aux_cur;  // destination buffers
  const int ps = 1 - pd, as = 1 - ad;          // binned (source) buffers
  // the final slot (-1: none), binned slot and tag of the block's f-th particle
  auto locate_f = [&](int f, int& ns, int& src, int& tg) {
    ns = -1;
    src = 0;
    tg = 0;
    if (f >= agg) return;
    int lo = 0, hi = ncb - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (lpre[mid] <= f) lo = mid; else hi = mid - 1;
    }
    const int r = f - lpre[lo];
    const int cnt = min(lpre[lo + 1] - lpre[lo], d.bcap);
    if (r >= cnt) return;  // beyond the bucket (LE_E_CAPACITY latched by the binning)
    const int2* B = d.bucket + (size_t)(c0 + lo) * d.bcap;
    const int2 e = B[r];
    int rank = 0;
    for (int q = 0; q < cnt; ++q) rank += (B[q].x < e.x) ? 1 : 0;
    const int s = base + lpre[lo] + rank;
    if ((unsigned)s < (unsigned)d.n && (unsigned)e.y < (unsigned)d.n) {  // (else a latched error)
      ns = s;
      src = e.y;
      tg = e.x;
    }
  };
  // The total forces move along only in a forced rebuild: one due within a
  // step call comes after the first half-kick, and the call's last step writes them anew.
  const bool with_f = cn.rebuild == kRebuildForced;
  const double Delta = cn.Delta;
  struct St { double4 p; double v0, v1, v2, f0, f1, f2; };
  auto load = [&](int i) -> St {
    const double* V = d.vel[as];
    const double* F = d.frc[as];
    St v{reinterpret_cast<const double4*>(d.pos[ps])[i], V[i], V[np + i], V[2 * np + i], 0.0, 0.0, 0.0};
    if (with_f) { v.f0 = F[i]; v.f1 = F[np + i]; v.f2 = F[2 * np + i]; }
    return v;
  };
  auto store = [&](int ns, int tg, St v) {
    if (ns < 0) return;
    double ky, kz;
    const bool fine = cross_wrap(d, Delta, v.p.x, v.p.y, v.p.z, ky, kz);
    v.v0 = v.v0 - ky * d.jump_sv;  // velocity jump (lab storage only)
    int cy, cz;
    img_get(v.p.w, cy, cz);
    v.p.w = img_put(cy + (int)ky, cz + (int)kz);
    if (!(fine && isfinite(v.v0) && isfinite(v.v1) && isfinite(v.v2))) latch(d.flags, LE_E_NONFINITE);
    reinterpret_cast<double4*>(d.pos[pd])[ns] = v.p;
    double* V = d.vel[ad];
    V[ns] = v.v0; V[np + ns] = v.v1; V[2 * np + ns] = v.v2;
    if (with_f) {
      double* F = d.frc[ad];
      F[ns] = v.f0; F[np + ns] = v.f1; F[2 * np + ns] = v.f2;
    }
    d.tag[ad][ns] = tg;
    d.slot_of_tag[tg] = ns;
  };
  for (int f0 = threadIdx.x; f0 < agg; f0 += 2 * TH) {
    int ns0, src0, tg0, ns1, src1, tg1;
    locate_f(f0, ns0, src0, tg0);
    locate_f(f0 + TH, ns1, src1, tg1);
    const St a0 = load(src0), a1 = load(src1);  // (slot 0 for an empty lane: in bounds, not stored)
    store(ns0, tg0, a0);
    store(ns1, tg1, a1);
  }
}

__global__ void __launch_bounds__(kBlock) k_scan_permute(Dev d) {
  if (rebuild_off(d)) return;
  scan_permute_body<kBlock>(d, *d.ctrl, blockIdx.x);
}

// Batched form: the blocks of one simulation are consecutive in the grid, so
// every block's predecessors were dispatched before it (the look-back waits
// only on them).
__global__ void __launch_bounds__(kBlock) k_scan_permute_b(Batch b) {
  int sm, bid;
  locate(b, blockIdx.x, sm, bid);
  const Dev& d = stage_dev(b.dev[sm]);
  if (rebuild_off(d)) return;
  scan_permute_body<kBlock>(d, *d.ctrl, bid);
}

// Kernels in one launch: blocks count themselves done, and the blocks of the next
// kernel wait until all have.  A block takes its place in the order of the work from
// a counter when it runs, not from its place in the grid: whatever it waits for is
// then done or being done by blocks that run already, and the wait ends, however
// many launches of other streams share the CUs.  (By the place in the grid, blocks
// that wait may fill the CUs of one XCD for blocks not yet dispatched on another,
// where the blocks of another launch wait likewise.)  The bound of the spin is never reached.
__device__ __forceinline__ int take_place(unsigned long long* next_place) {
  __shared__ int place;
  if (threadIdx.x == 0) place = (int)atomicAdd(next_place, 1ull);
  __syncthreads();
  return place;
}
// What the block wrote is out before it counts: every wave waits for its own stores
// ahead of the barrier, so that they are in the L2 that the release of the one
// thread that counts writes back (that release waits for the stores of its own wave alone;
// a release by every wave writes the L2 back eight times, 17,389 particles 24.1
// instead of 20.6 us a step).  The thread that has seen the count acquires for
// the block ahead of the barrier that lets it go on (an acquire by every wave invalidates
// the L2 eight times under the blocks that work already: 10,000 particles that rebuild
// every step 78 instead of 55 us).
__device__ __forceinline__ void add_count(unsigned long long* count) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(count, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool wait_count(const Dev& d, unsigned long long* count, int due) {
  __shared__ int ready;
  if (threadIdx.x == 0) {
    long long spins = 0;
    bool done = false, fault = false;
    // (a block that finds a latched error counts nothing)
    while (!(done = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= (unsigned long long)due) &&
           !(fault = __hip_atomic_load(&d.flags->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) &&
           ++spins < (1ll << 22))
      __builtin_amdgcn_s_sleep(10);
    if (!done && !fault) latch(d.flags, LE_E_STATE);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    ready = done && __hip_atomic_load(&d.flags->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
  }
  __syncthreads();
  return ready != 0;
}

// (1) and (2) in one launch.  A step that rebuilds nothing pays one empty
// launch less; one that does pays the hand-over, a write-back and a
// refill of the L2s, which grows with the system (see launch_rebuild).
__global__ void __launch_bounds__(kBlock) k_sort(Dev d, Ctrl* __restrict__ next,
                                                 unsigned long long* __restrict__ next_vmax, int control) {
  __shared__ Ctrl sc, sn;
  if (!sort_control(d, next, next_vmax, 0, control, blockIdx.x, sc, sn)) return;
  const int nbb = (d.n + kBinBlock - 1) / kBinBlock;
  const int b = take_place(&d.joined[kPlace * kJoinedLine]);  // (the search sets the counts back to zero)
  if (b < nbb) {
    bin_body<kBlock>(d, sc, b);
    add_count(&d.joined[kBinned * kJoinedLine]);
  } else if (wait_count(d, &d.joined[kBinned * kJoinedLine], nbb)) {
    scan_permute_body<kBlock>(d, sn, b - nbb);
  }
}

// Neighbour lists of radius r_list through the Lees-Edwards cell stencil.
// Rows that do not cross a gradient face use the 27-cell block with periodic
// x/z images.  A row reached across the top (bottom) face belongs to the image
// box shifted by +Delta (-Delta) along x; the cells of that row whose image
// overlaps [x_cell - r_list, x_cell + l_x + r_list] are the unwrapped indices
// k in [floor((ix l - r - sy Delta)/l), floor(((ix+1) l + r - sy Delta)/l)],
// at most four cells for l >= r (five with the rounding margin).  Each
// (cell, image) pair is visited once; with L > 2 r_list at most one image of
// a particle can lie within r_list, so no pair is counted twice.
//
// Tiles.  A tile is T consecutive slots (kTile, or kTileSmall in small
// systems).  The slots follow the beam order of the cells (cell_slot), so a tile covers a stretch [xa, xb] of one beam, or
// the end of one and the start of the next (its segments).  The cells that a
// segment's stencils reach, row by row, are staged into LDS in a fixed order
// while they fit (HALO positions).  With the halo layout, d.halo
// records the slot and image of every LDS position so that the force kernel can
// restage the same halo each step, and the lists hold LDS indices
// (16 bits); the global layout's lists hold slot and image code in one word.
// Lists are padded with sentinels (LDS index HALO, slot n) to whole batches.

// Units of particle i's list (see Dev): block b from the front, block b of
// walked entries from the back.
__device__ __forceinline__ size_t unit_front(const Dev& d, int b, int i) { return (size_t)b * d.np + i; }
__device__ __forceinline__ size_t unit_back(const Dev& d, int b, int i) {
  return (size_t)(d.units - 1 - b) * d.np + i;
}

// Unwrapped x-cell range [klo, khi] reached from cells xa..xb of a row across
// the gradient face with image sy (sy = 0: the plain periodic block).
__device__ __forceinline__ void x_range(const Dev& d, int xa, int xb, int sy, double Delta, double rmarg,
                                        int& klo, int& khi) {
  if (sy == 0) {
    klo = xa - 1; khi = xb + 1;
  } else {
    double sh = (double)sy * Delta;
    klo = (int)floor(((double)xa * d.lx - rmarg - sh) / d.lx);
    khi = (int)floor(((double)(xb + 1) * d.lx + rmarg - sh) / d.lx);
  }
}

// Exact list test of one pair: the plain-definition displacement between
// particle i and slot q under image (sx, sy, sz), r^2 < r_list^2.
__device__ __forceinline__ bool in_list_exact(const Dev& d, double4 pi, double4 pj, double shx,
                                              double shy, double shz, double shd) {
  double dy = (pi.y - pj.y) - shy;
  double dx = ((pi.x - pj.x) - shd) - shx;
  double dz = (pi.z - pj.z) - shz;
  double r2 = dx * dx + dy * dy;
  r2 = r2 + dz * dz;
  return r2 < d.rlist2;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kCand = 256;  // candidates a wave keeps before it tests them

// Bounding box (x, y, z minima, then the negated maxima), and the square of
// the distance from it within which a point may be within r_list of one of
// its points (rounding of the floats included: they are within 2^-24 of their
// values).
struct Box { float v[6], reach2; };
__device__ __forceinline__ float reach2_of(const Box& b, float rlist) {
  const float ext = fmaxf(fmaxf(fmaxf(fabsf(b.v[0]), fabsf(b.v[1])), fmaxf(fabsf(b.v[2]), fabsf(b.v[3]))),
                          fmaxf(fabsf(b.v[4]), fabsf(b.v[5])));
  const float reach = rlist * 1.00001f + 1e-6f * (ext + rlist);
  return reach * reach;
}
__device__ __forceinline__ bool in_reach(const Box& b, float x, float y, float z) {
  const float dx = fmaxf(fmaxf(b.v[0] - x, x + b.v[3]), 0.0f);
  const float dy = fmaxf(fmaxf(b.v[1] - y, y + b.v[4]), 0.0f);
  const float dz = fmaxf(fmaxf(b.v[2] - z, z + b.v[5]), 0.0f);
  return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)) <= b.reach2;
}

// Floats as integers of the same order (its own inverse), and the minimum over
// each row of 16 lanes by rotations within the row.
__device__ __forceinline__ int order_key(int b) { return b ^ ((b >> 31) & 0x7fffffff); }
__device__ __forceinline__ float row16_min(float f) {
  int v = order_key(__float_as_int(f));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, false));
  return __int_as_float(order_key(v));
}

// One stretch of a beam covered by a tile.  Its halo is the rows (y0 - 1 + ry,
// z0 - 1 + rz), ry in [0, h + 2), rz in [0, w + 2); row (rz (h + 2) + ry) has
// the nk cells klo[sy + 1] .. of the staging table from entry tb + row nk on.
struct Seg {
  int y0, z0, h, w;   // first row and height / width of the beam
  int xa, xb;         // cells of the stretch along x
  int klo[3], khi[3]; // unwrapped cells along x of its halo rows, by image sy = -1, 0, 1
  int nk, tb;
  double ox, oy, oz;  // origin of the staged floats: a particle of the stretch
};

// The lists of one tile by one block: a wave takes a cluster of 16 consecutive
// slots.  All four 16-lane rows hold the same 16 particles.
// The cluster's candidates are the staged cells of its bounding box in cells,
// 16 at a time: r^2 = s_i + s_j - 2 x_i x_j with s = |x|^2 is one 16x16x4
// FP32 matrix product (A: x, y, z, s of the candidates, B: -2x, -2y, -2z, 1 of
// the particles, C: s_i), 256 pairs in 32 cycles, and lane (q, p) receives the
// four candidates 4q .. 4q+3 of particle p.  An LDS ring per lane collects
// what it accepts; a full block of eight leaves as one 16-byte store at the
// particle's next block, and the four lanes' last, partial blocks are joined
// at the end, so that a list carries one padding.
//
// FP32 pre-test.  The staged floats are within u = 2^-24 (relative) of the
// coordinates about the segment's origin, and the product adds four rounded
// terms of at most 4 S, S = (|x_i| + r_list)^2, so r^2 is within 64 u S of its
// FP64 value for every candidate near r_list (farther ones are off by less
// than their distance from r_list).  Outside that band the FP32 value decides,
// inside it the plain FP64 displacement, so the list is exactly
// {r^2 < r_list^2}.
//
// Bound by the vector unit (LJ, 256,000 particles, r_list 3.05: 2850 vector
// instructions per cluster, 130 us, 62% busy) and, in small systems, by the chain of
// phases: against one lane per particle half with the tests on the vector unit, 1000
// particles take 25 instead of 111 us, 27,000 take 26 instead of 87, 256,000 as long
// as before and 400,000 beads of a melt 119 instead of 112 (65% busy); the compact halo
// that it leaves to the force kernel is what the large systems gain from.
template <int HALO, bool GL>
__device__ __forceinline__ void neighbors_body(const Dev& d, const Ctrl* c, const int tile) {
  constexpr int TH = kSearchThreads, NW = TH / 64;
  constexpr int kCells = TH;  // cells a tile's halo may have (staging table, one per thread)
  static_assert(NW * 16 == kTile, "one cluster per wave");
  constexpr int kLook = 6, kSeen = kLook * TH;  // positions a thread, a tile looks at
  static_assert(kLook * NW <= 64 && kSeen <= 0xffff, "one lane per (round, wave); 16-bit offsets");
  constexpr int kCut = 1 << 30;
  constexpr int kFull = 8;  // particles above which a cell that is walked counts as full
  const int T = d.tile;  // (of small tiles the first waves take the clusters)
  constexpr int RS = 13;            // words per lane of the ring: 26 LDS indices, odd stride (banks)
  constexpr int PAD = GL ? 4 : 8;  // list padding (entries per unit of 16 bytes)
  // x, y, z, |x|^2 (spare entries: a round may read up to 31 past the halo; the
  // stride keeps the four components on different banks)
  __shared__ float hc[4][HALO + 48];
  static_assert((HALO + 48) % 64 == 48, "components 16 banks apart");
  constexpr int kPad = HALO + 40;  // a candidate that no particle accepts (r^2 = 1e30)
  __shared__ uint32_t hent[GL ? HALO + 1 : 1];  // global-list entry of every staged position, sentinel last
  __shared__ int coff[kCells + 1];       // LDS offset of every cell of the halo
  __shared__ uint32_t cent[kCells];      // its first slot and image (og_entry)
  __shared__ __align__(16) uint16_t cand[NW][kCand];  // the candidates a wave has kept
  union Ring {
    uint32_t w[NW][64 * RS];
    uint16_t map[kSeen];  // staging: table entry of each position looked at, then the kept ones before it
  };
  __shared__ __align__(16) Ring ring;
  __shared__ Seg sgs[2];
  __shared__ Box wbox[NW][2], tbox[2];
  __shared__ int wkept[64], kept_sh;
  __shared__ int wsum[NW], wmax[NW], tot_sh, nseg_sh, nent_sh;
  const int np = d.np, n = d.n, units = d.units;
  const int s0 = tile * T;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int pn = c->pos_cur, an = c->aux_cur;  // sorted buffers of the new state
  const double4* P = reinterpret_cast<const double4*>(d.pos[pn]);
  const double Delta = c->Delta;
  const double rmarg = d.rlist * (1.0 + 1e-12) + 1e-12 * (d.Lx + d.Ly + d.Lz);

  // ---- segments, from the tile's first and last particle (thread g: segment g)
  const int send = min(s0 + T, n) - 1;
  if (threadIdx.x < 64) {
    const int g = threadIdx.x & 1;
    const double4 p0 = P[g == 0 ? s0 : send], pm = P[(s0 + send) >> 1];
    Seg s;
    const int cx = cell_index(p0.x, d.inv_lx, d.nx), cy = cell_index(p0.y, d.inv_ly, d.ny),
              cz = cell_index(p0.z, d.inv_lz, d.nz);
    const int nby = (d.ny + (1 << d.by_sh) - 1) >> d.by_sh;
    const int beam = (cz >> d.bz_sh) * nby + (cy >> d.by_sh);
    const int other = __shfl_xor(beam, 1, 64), ox = __shfl_xor(cx, 1, 64);
    const int step = g == 0 ? other - beam : beam - other;  // beams from the first to the last particle
    const int ns = step == 0 ? 1 : (step == 1 ? 2 : 0);     // 0: more than two, nothing is staged
    s.y0 = cy >> d.by_sh << d.by_sh;
    s.z0 = cz >> d.bz_sh << d.bz_sh;
    s.h = min(1 << d.by_sh, d.ny - s.y0);
    s.w = min(1 << d.bz_sh, d.nz - s.z0);
    s.xa = g == 0 ? cx : 0;
    s.xb = ns == 1 ? ox : (g == 0 ? d.nx - 1 : cx);
    s.nk = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      // rows across a gradient face only where the beam touches it
      const bool used = k == 1 || (k == 0 ? s.y0 == 0 : s.y0 + s.h == d.ny);
      s.klo[k] = s.khi[k] = 0;
      if (used) {
        x_range(d, s.xa, s.xb, k - 1, Delta, rmarg, s.klo[k], s.khi[k]);
        s.nk = max(s.nk, s.khi[k] - s.klo[k] + 1);
      }
    }
    // origin of the floats: the middle of the tile (the smallest coordinates), or an end
    s.ox = ns == 1 ? pm.x : p0.x; s.oy = ns == 1 ? pm.y : p0.y; s.oz = ns == 1 ? pm.z : p0.z;
    const int cells = (s.h + 2) * (s.w + 2) * s.nk, first = __shfl(cells, 0, 64);
    s.tb = g == 0 ? 0 : first;
    if (threadIdx.x < 2) sgs[threadIdx.x] = s;
    if (threadIdx.x == 1) {
      // (more cells than the table holds are nearly empty, and better walked)
      const int all = ns == 0 ? 0 : (ns == 1 ? first : first + cells);
      nseg_sh = all <= kCells ? ns : 0;
      nent_sh = all <= kCells ? all : 0;
    }
  }
  __syncthreads();
  const int nseg = nseg_sh, nent = nent_sh, tb1 = sgs[1].tb;

  // ---- the wave's particles (the same 16 in each row of 16 lanes), and the
  // bounding box of the tile's particles of each segment
  const int p16 = lane & 15, q = lane >> 4;
  const int i = s0 + wv * 16 + p16;
  const bool valid = wv * 16 < T && i < n;
  const double4 pi = P[valid ? i : s0];
  const int ix = cell_index(pi.x, d.inv_lx, d.nx);
  const int iy = cell_index(pi.y, d.inv_ly, d.ny);
  const int iz = cell_index(pi.z, d.inv_lz, d.nz);
  const int gi = nseg == 2 && !(iy >= sgs[0].y0 && iy < sgs[0].y0 + sgs[0].h && iz >= sgs[0].z0 &&
                                iz < sgs[0].z0 + sgs[0].w) ? 1 : 0;
  const float fx = (float)(pi.x - sgs[gi].ox), fy = (float)(pi.y - sgs[gi].oy), fz = (float)(pi.z - sgs[gi].oz);
  for (int g = 0; g < nseg; ++g) {
    const bool in = valid && gi == g;
    Box b = {{row16_min(in ? fx : 1e30f), row16_min(in ? fy : 1e30f), row16_min(in ? fz : 1e30f),
                    row16_min(in ? -fx : 1e30f), row16_min(in ? -fy : 1e30f), row16_min(in ? -fz : 1e30f)}, 0.0f};
    if (lane == 0) {
      wbox[wv][g] = b;
      wbox[wv][g].reach2 = reach2_of(b, d.rlist_f);
    }
  }

  // ---- staging table: one cell per thread, then the cells' offsets (uniform
  // branches: a tile that stages nothing goes on to its walk)
  if (nseg > 0) {
    const int e = (int)threadIdx.x;
    int st = 0, code = 0, cnt = 0;
    if (e < nent) {
      const Seg& s = sgs[nseg == 2 && e >= tb1 ? 1 : 0];
      const int h2 = s.h + 2, el = e - s.tb;
      const int row = el / s.nk, kk = el - row * s.nk;
      const int rz = row / h2, ry = row - rz * h2;
      int jy = s.y0 - 1 + ry, jz = s.z0 - 1 + rz;
      const int sy = jy < 0 ? -1 : (jy >= d.ny ? 1 : 0), sz = jz < 0 ? -1 : (jz >= d.nz ? 1 : 0);
      jy -= sy * d.ny;
      jz -= sz * d.nz;
      const int k = s.klo[sy + 1] + kk;
      if (k <= s.khi[sy + 1]) {
        const int sx = floor_div(k, d.nx);
        const int cell = cell_slot(d, k - sx * d.nx, jy, jz);
        st = d.cell_start[cell];
        cnt = d.cell_start[cell + 1] - st;
        code = pack_img(sx, sy, sz);
      }
    }
    cent[e] = og_entry((uint32_t)st, (uint8_t)code);
    int incl = cnt;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wv] = incl;
    if (threadIdx.x == 0) tot_sh = 0;
    __syncthreads();
    int off = incl - cnt, all = 0;
    for (int w2 = 0; w2 < NW; ++w2) {
      if (w2 < wv) off += wsum[w2];
      all += wsum[w2];
    }
    coff[e] = off;
    if (off + cnt <= kSeen) {  // the cells looked at are a prefix of the table
      for (int k = 0; k < cnt; ++k) ring.map[off + k] = (uint16_t)e;
      if (all > kSeen) atomicMax(&tot_sh, off + cnt);
    }
    if (threadIdx.x == TH - 1) coff[TH] = off + cnt;
    if (threadIdx.x == 0 && all <= kSeen) tot_sh = all;
    if (threadIdx.x < 2 && (int)threadIdx.x < nseg) {  // the tile's boxes: minimum over the waves
      Box b = wbox[0][threadIdx.x];
      for (int w2 = 1; w2 < NW; ++w2)
#pragma unroll
        for (int k = 0; k < 6; ++k) b.v[k] = fminf(b.v[k], wbox[w2][threadIdx.x].v[k]);
      b.reach2 = reach2_of(b, d.rlist_f);
      tbox[threadIdx.x] = b;
    }
  }
  __syncthreads();
  const int seen = nseg > 0 ? tot_sh : 0;
  // ---- stage the positions within reach of the segment's box: LDS position =
  // the number of kept ones before it, in the order of the table
  if (nseg > 0) {
    int slot[kLook], code[kLook];
    float x[kLook], y[kLook], z[kLook];
    unsigned long long kept[kLook];
#pragma unroll
    for (int u0 = 0; u0 < kLook; u0 += 2) {  // two loads in flight per thread, while there are positions
#pragma unroll
      for (int u = u0; u < u0 + 2; ++u) kept[u] = 0ull;
      if (u0 * TH >= seen) continue;
      double4 pj[2];
      int sgi[2];
#pragma unroll
      for (int u = u0; u < u0 + 2; ++u) {
        const int h = (int)threadIdx.x + u * TH;
        slot[u] = n;
        code[u] = pack_img(0, 0, 0);
        sgi[u - u0] = 0;
        if (h < seen) {
          const int e = ring.map[h];
          slot[u] = (int)(cent[e] & kSlotMask) + (h - coff[e]);
          code[u] = (int)(cent[e] >> kSlotBits);
          sgi[u - u0] = nseg == 2 && e >= tb1 ? 1 : 0;
        }
        pj[u - u0] = P[slot[u]];
      }
#pragma unroll
      for (int u = u0; u < u0 + 2; ++u) {
        const Seg& s = sgs[sgi[u - u0]];
        const double4 p = pj[u - u0];
        int sx, sy, sz;
        unpack_img((uint8_t)code[u], sx, sy, sz);
        x[u] = (float)((p.x + ((double)sy * Delta + (double)sx * d.Lx)) - s.ox);
        y[u] = (float)((p.y + (double)sy * d.Ly) - s.oy);
        z[u] = (float)((p.z + (double)sz * d.Lz) - s.oz);
        const bool keep = (int)threadIdx.x + u * TH < seen && in_reach(tbox[sgi[u - u0]], x[u], y[u], z[u]);
        kept[u] = __ballot(keep);
        if (lane == 0) wkept[u * NW + wv] = __popcll(kept[u]);
      }
    }
    __syncthreads();
    // kept positions before each (round, wave)
    const int v = lane < (seen + TH - 1) / TH * NW ? wkept[lane] : 0;
    int before = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(before, o, 64);
      if (lane >= o) before += t;
    }
    if (threadIdx.x == 63) kept_sh = before;
    before -= v;
#pragma unroll
    for (int u = 0; u < kLook; ++u) {
      if (u * TH >= seen) break;
      const int h = (int)threadIdx.x + u * TH;
      const int pos = __builtin_amdgcn_readlane(before, u * NW + wv) + __popcll(kept[u] & ((1ull << lane) - 1ull));
      if (h < seen) ring.map[h] = (uint16_t)pos;
      if (!((kept[u] >> lane) & 1ull) || pos >= HALO) continue;
      hc[0][pos] = x[u];
      hc[1][pos] = y[u];
      hc[2][pos] = z[u];
      hc[3][pos] = (float)((double)x[u] * (double)x[u] + (double)y[u] * (double)y[u] + (double)z[u] * (double)z[u]);
      const uint32_t e = og_entry((uint32_t)slot[u], (uint8_t)code[u]);
      if constexpr (GL) hent[pos] = e;
      else d.halo[(size_t)tile * HALO + pos] = e;
    }
  }
  if (threadIdx.x < 4) hc[threadIdx.x][kPad] = threadIdx.x == 3 ? 1e30f : 0.0f;
  if (GL && threadIdx.x == 0) hent[HALO] = og_entry((uint32_t)n, pack_img(0, 0, 0));
  __syncthreads();
  const int kept_all = nseg > 0 ? kept_sh : 0;
  if (threadIdx.x == 0) d.tile_nstage[tile] = min(kept_all, HALO);
  // the particle's own LDS position (its plain image), and the cells' offsets
  // among the kept positions (kCut: beyond what was looked at)
  int self_h = -1;
  if (valid && nseg > 0) {
    const Seg& s = sgs[gi];
    const int e = s.tb + ((iz - s.z0 + 1) * (s.h + 2) + (iy - s.y0 + 1)) * s.nk + (ix - s.xa + 1);
    const int h = coff[e] + (i - (int)(cent[e] & kSlotMask));
    if (h < seen) self_h = ring.map[h];
  }
  if (nseg > 0) {
    auto kept_before = [&](int o) { return o < seen ? (int)ring.map[o] : (o == seen ? kept_all : kCut); };
    const int before = kept_before(coff[threadIdx.x]), last = kept_before(coff[TH]);
    __syncthreads();
    coff[threadIdx.x] = before;
    if (threadIdx.x == 0) coff[TH] = last;
  }
  __syncthreads();

  // ---- scan
  uint32_t* const rw = ring.w[wv] + (p16 * 4 + q) * RS;  // the four lanes of a particle are neighbours
  uint16_t* const r16 = reinterpret_cast<uint16_t*>(rw);
  int cnt = 0;   // entries in this lane's ring
  int nblk = 0;  // blocks of eight written for the particle (the same in its four lanes)
  int nog = 0;   // entries of rows that were not staged (the same in the four lanes)
  auto og_store = [&](int k, uint32_t e) {
    if ((k >> 2) < units) reinterpret_cast<uint32_t*>(d.nl + unit_back(d, k >> 2, i))[k & 3] = e;
  };
  // full blocks leave the rings, lanes of a particle in order of q (called by the whole wave)
  auto flush = [&]() {
    const unsigned long long full = __ballot(cnt >= 8);
    const unsigned long long mine = (full >> p16) & 0x0001000100010001ull;
    if (cnt >= 8) {
      const int blk = nblk + __popcll(mine & ((1ull << (16 * q)) - 1ull));
      uint32_t t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = rw[k];
      if ((blk + 1) * (8 / PAD) <= units) {
        if constexpr (GL) {
          d.nl[unit_front(d, 2 * blk, i)] = make_uint4(hent[t[0] & 0xffff], hent[t[0] >> 16], hent[t[1] & 0xffff],
                                                          hent[t[1] >> 16]);
          d.nl[unit_front(d, 2 * blk + 1, i)] = make_uint4(hent[t[2] & 0xffff], hent[t[2] >> 16],
                                                              hent[t[3] & 0xffff], hent[t[3] >> 16]);
        } else {
          d.nl[unit_front(d, blk, i)] = make_uint4(t[0], t[1], t[2], t[3]);
        }
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) rw[k] = rw[k + 4];
      cnt -= 8;
    }
    nblk += __popcll(mine);
  };
  const size_t hbase = (size_t)tile * HALO;
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  for (int g = 0; g < nseg; ++g) {
    const Seg& s = sgs[g];
    const int y0 = uni(s.y0), z0 = uni(s.z0), h2 = uni(s.h) + 2, nk = uni(s.nk), stb = uni(s.tb);
    const bool low = y0 == 0, high = y0 + h2 - 2 == d.ny;  // the beam touches a gradient face
    const bool in_seg = valid && gi == g;
    const unsigned long long lanes = __ballot(in_seg);
    if (!lanes) continue;
    // bounding box of the cluster's cells: x from its first and last particle
    // (sorted along the beam), rows of y and z from their masks
    const int first = __builtin_ctzll(lanes), last = 15 - __builtin_clz((unsigned)(lanes & 0xffffull) << 16);
    const int xlo = __builtin_amdgcn_readlane(ix, first), xhi = __builtin_amdgcn_readlane(ix, last);
    int ym = in_seg ? (1 << (iy - y0)) | (1 << (16 + iz - z0)) : 0;
    for (int o = 8; o > 0; o >>= 1) ym |= __shfl_xor(ym, o, 64);
    ym = __builtin_amdgcn_readfirstlane(ym);
    const int ylo = __builtin_ctz((ym & 0xffff) | 0x10000), yhi = 31 - __builtin_clz((ym & 0xffff) | 1);
    const int zlo = __builtin_ctz(((unsigned)ym >> 16) | 0x10000), zhi = 31 - __builtin_clz(((unsigned)ym >> 16) | 1);
    // cells along x of the cluster's rows, by image sy
    int ka[3], kb[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ka[k] = kb[k] = 0;
      if (k == 1 || (k == 0 ? low : high)) x_range(d, xlo, xhi, k - 1, Delta, rmarg, ka[k], kb[k]);
    }
    // matrix operands and thresholds of the lane's particle
    const float si = (float)((double)fx * (double)fx + (double)fy * (double)fy + (double)fz * (double)fz);
    const float bv = q == 0 ? -2.0f * fx : (q == 1 ? -2.0f * fy : (q == 2 ? -2.0f * fz : 1.0f));
    const float c0 = in_seg ? si : 1e30f;
    const f32x4 cv = {c0, c0, c0, c0};
    const float R = __builtin_sqrtf(si) + d.rlist_f;
    const float margin = d.nb_rel * R * R;
    const float tlo = d.nb_lo - margin, thi = d.nb_hi + margin;
    const Box box = wbox[wv][g];
    // the first `count` kept candidates against the cluster's particles, 32 a
    // round (the particles themselves are among the first `own`)
    auto test = [&](int count, int own) {
      if (lane < 32) cand[wv][count + lane] = (uint16_t)kPad;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      float a0 = hc[q][cand[wv][p16]], a1 = hc[q][cand[wv][16 + p16]];
      for (int c0 = 0; c0 < count; c0 += 32) {
        const uint2 e0 = *reinterpret_cast<const uint2*>(&cand[wv][c0 + 4 * q]);
        const uint2 e1 = *reinterpret_cast<const uint2*>(&cand[wv][c0 + 16 + 4 * q]);
        const uint16_t hv[8] = {(uint16_t)e0.x, (uint16_t)(e0.x >> 16), (uint16_t)e0.y, (uint16_t)(e0.y >> 16),
                                (uint16_t)e1.x, (uint16_t)(e1.x >> 16), (uint16_t)e1.y, (uint16_t)(e1.y >> 16)};
        const f32x4 w0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, bv, cv, 0, 0, 0);
        const f32x4 w1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, bv, cv, 0, 0, 0);
        const int cn = c0 + 32 < count ? c0 + 32 : c0;  // the next round's operands
        a0 = hc[q][cand[wv][cn + p16]];
        a1 = hc[q][cand[wv][cn + 16 + p16]];
        float rr[8] = {w0[0], w0[1], w0[2], w0[3], w1[0], w1[1], w1[2], w1[3]};
        if (c0 < own) {
#pragma unroll
          for (int v = 0; v < 8; ++v)
            if (hv[v] == self_h) rr[v] = 1e30f;
        }
        // every candidate is written at the ring's next entry, and the count
        // moves on only past the accepted ones
        unsigned long long band = 0;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          r16[cnt] = hv[v];
          const bool in = rr[v] < tlo;
          cnt += in ? 1 : 0;
          band |= __ballot(in) ^ __ballot(rr[v] < thi);
        }
        if (band) {  // rare: the FP64 displacement decides
          unsigned todo = 0;
#pragma unroll
          for (int v = 0; v < 8; ++v) todo |= (rr[v] >= tlo && rr[v] < thi ? 1u : 0u) << v;
          while (todo) {
            const int v = __builtin_ctz(todo);
            todo &= todo - 1u;
            const int h = cand[wv][c0 + 16 * (v >> 2) + 4 * q + (v & 3)];
            uint32_t e;
            if constexpr (GL) e = hent[h];
            else e = d.halo[hbase + h];
            int sx2, sy2, sz2;
            unpack_img((uint8_t)(e >> kSlotBits), sx2, sy2, sz2);
            if (in_list_exact(d, pi, P[e & kSlotMask], (double)sx2 * d.Lx, (double)sy2 * d.Ly,
                              (double)sz2 * d.Lz, (double)sy2 * Delta)) {
              r16[cnt] = (uint16_t)h;
              ++cnt;
            }
          }
        }
        // (two rounds fill the ring: 7 + 16 of its 26 entries)
        if ((c0 & 32) || c0 + 32 >= count)
          while (__any(cnt >= 8)) flush();
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // rows of the box: lane r finds the LDS range of row r, if it was staged
    const int nry = yhi - ylo + 3, nrow = nry * (zhi - zlo + 3);
    for (int r0 = 0; r0 < nrow; r0 += 64) {
      int row_a = 0, row_b = 0, row_ry = 0, row_rz = 0;
      bool row_staged = false;
      if (r0 + lane < nrow) {
        row_rz = (r0 + lane) / nry;
        row_ry = ylo + (r0 + lane) - row_rz * nry;
        row_rz += zlo;
        const int jy0 = y0 - 1 + row_ry;
        const int syu = jy0 < 0 ? -1 : (jy0 >= d.ny ? 1 : 0);
        const int rb = stb + (row_rz * h2 + row_ry) * nk;
        const int lo = s.klo[syu + 1];
        const int k0 = syu == 0 ? ka[1] : (syu < 0 ? ka[0] : ka[2]);
        const int k1 = syu == 0 ? kb[1] : (syu < 0 ? kb[0] : kb[2]);
        row_staged = coff[rb + nk] <= HALO;
        if (row_staged) {
          row_a = coff[rb + (k0 - lo)];
          row_b = coff[rb + (k1 - lo) + 1];
        }
      }
      const bool row_self = row_ry > ylo && row_ry < yhi + 2 && row_rz > zlo && row_rz < zhi + 2;
      // Candidates of the staged rows within reach of the bounding box, four
      // rows at a time (one per 16 lanes), the particles' own rows first; then
      // the kept ones against the particles.
      int nc = 0, nself = 0;  // kept candidates; of which may hold the particles themselves
      for (int pass = 0; pass < 2; ++pass) {
        unsigned long long rows = __ballot(row_staged && row_self == (pass == 0) && row_a < row_b);
        while (rows) {
          int rsel = -1;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (rows) {
              const int r = __builtin_ctzll(rows);
              rows &= rows - 1ull;
              if (q == k) rsel = r;
            }
          }
          // (both shuffles by the whole wave: a lane without a row still serves its own)
          const int ra = __shfl(row_a, rsel & 63, 64), rb = __shfl(row_b, rsel & 63, 64);
          int h = ra + p16;
          const int hb = rsel >= 0 ? rb : 0;
          while (__any(h < hb)) {
            const int hh = min(h, HALO);
            const bool keep = h < hb && in_reach(box, hc[0][hh], hc[1][hh], hc[2][hh]);
            const unsigned long long m = __ballot(keep);
            if (keep) cand[wv][nc + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0))] = (uint16_t)h;
            nc += __popcll(m);
            h += 16;
            if (nc > kCand - 96) {  // (room for another 64 and the padding)
              test(nc, pass == 0 ? nc : nself);
              nc = nself = 0;
            }
          }
        }
        if (pass == 0) nself = nc;
      }
      test(nc, nself);
    }
  }
  // ---- rows that were not staged (the tile lies in more than two beams, or its halo has
  // too many cells or positions): the four lanes of a particle walk the rows of its
  // own stencil in global memory with the exact test, three rows at once, one cell
  // a lane, or where cells are full all four lanes one cell.  (Row by row of the whole
  // tile, up to a hundred where cells are nearly empty, the search of 200,000 particles at
  // density 0.007 took 353 us instead of 94; one cell a lane alone 138 us in a
  // droplet of 19 per cell instead of 120.)
  if (nseg == 0 || coff[nent] > HALO) {
    for (int dzc = -1; dzc <= 1; ++dzc) {
      int jz = iz + dzc;
      const int sz = jz < 0 ? -1 : (jz >= d.nz ? 1 : 0);
      jz -= sz * d.nz;
      // the three rows of a plane together: their cells' bounds are fetched at once
      int k[3], khi[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        bool walk = valid;
        if (nseg > 0) {
          const Seg& s = sgs[gi];
          walk = valid && coff[s.tb + ((iz - s.z0 + 1 + dzc) * (s.h + 2) + (iy - s.y0 + r) + 1) * s.nk] > HALO;
        }
        const int jy = iy + r - 1;
        k[r] = 0;
        khi[r] = -1;
        if (walk) x_range(d, ix, ix, jy < 0 ? -1 : (jy >= d.ny ? 1 : 0), Delta, rmarg, k[r], khi[r]);
      }
      while (__any(k[0] <= khi[0] || k[1] <= khi[1] || k[2] <= khi[2])) {
        int sx[3], start[3], stop[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          const int jy = iy + r - 1, sy = jy < 0 ? -1 : (jy >= d.ny ? 1 : 0);
          sx[r] = start[r] = stop[r] = 0;
          if (k[r] + q <= khi[r]) {
            sx[r] = floor_div(k[r] + q, d.nx);
            const int cell = cell_slot(d, k[r] + q - sx[r] * d.nx, jy - sy * d.ny, jz);
            start[r] = d.cell_start[cell];
            stop[r] = d.cell_start[cell + 1];
          }
          k[r] += 4;
        }
        auto try_slot = [&](int r, int slot, int end, int cx, double4 pj) {
          const int jy = iy + r - 1, sy = jy < 0 ? -1 : (jy >= d.ny ? 1 : 0);
          const bool in = slot < end && !(slot == i && cx == 0 && sy == 0 && sz == 0) &&
                          in_list_exact(d, pi, pj, (double)cx * d.Lx, (double)sy * d.Ly, (double)sz * d.Lz,
                                        (double)sy * Delta);
          const unsigned long long mine = (__ballot(in) >> p16) & 0x0001000100010001ull;
          if (in) og_store(nog + __popcll(mine & ((1ull << (16 * q)) - 1ull)),
                           og_entry((uint32_t)slot, pack_img(cx, sy, sz)));
          nog += __popcll(mine);
        };
        if (__any(max(stop[0] - start[0], max(stop[1] - start[1], stop[2] - start[2])) > kFull)) {
#pragma unroll
          for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 4; ++c) {
              const int from = p16 + 16 * c;
              const int cx = __shfl(sx[r], from, 64), end = __shfl(stop[r], from, 64);
              for (int slot = __shfl(start[r], from, 64) + q; __any(slot < end); slot += 4)
                try_slot(r, slot, end, cx, P[slot < end ? slot : s0]);
            }
        } else {
          while (__any(start[0] < stop[0] || start[1] < stop[1] || start[2] < stop[2])) {
            double4 pj[3];
#pragma unroll
            for (int r = 0; r < 3; ++r) pj[r] = P[start[r] < stop[r] ? start[r] : s0];
#pragma unroll
            for (int r = 0; r < 3; ++r) try_slot(r, start[r]++, stop[r], sx[r], pj[r]);
          }
        }
      }
    }
  }
  // ---- the four partial blocks of each particle are joined (the particle's
  // rings are neighbours in LDS: their first 16-byte aligned stretch holds them)
  const int r0 = __shfl(cnt, p16, 64), r1 = __shfl(cnt, p16 + 16, 64), r2 = __shfl(cnt, p16 + 32, 64),
            r3 = __shfl(cnt, p16 + 48, 64);
  const int below = (q > 0 ? r0 : 0) + (q > 1 ? r1 : 0) + (q > 2 ? r2 : 0);
  const int rest = r0 + r1 + r2 + r3;
  const int restp = (rest + PAD - 1) / PAD * PAD;
  {
    uint32_t t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = rw[k];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint32_t* const tw = ring.w[wv] + p16 * 4 * RS;
    uint16_t* const t16 = reinterpret_cast<uint16_t*>(tw);
#pragma unroll
    for (int k = 0; k < 7; ++k)
      if (k < cnt) t16[below + k] = (uint16_t)(t[k >> 1] >> (16 * (k & 1)));
    for (int k = rest + q; k < restp; k += 4) t16[k] = (uint16_t)HALO;  // (with GL: hent[HALO], slot n)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int b0 = nblk * (8 / PAD);  // blocks of PAD entries written so far
    if (valid) {
      for (int b = q; b * PAD < restp; b += 4) {
        if (b0 + b >= units) continue;
        if constexpr (GL) {
          const uint16_t* e = t16 + 4 * b;
          d.nl[unit_front(d, b0 + b, i)] = make_uint4(hent[e[0]], hent[e[1]], hent[e[2]], hent[e[3]]);
        } else {
          d.nl[unit_front(d, b0 + b, i)] = *reinterpret_cast<const uint4*>(tw + 4 * b);
        }
      }
    }
  }
  const int entries = nblk * 8 + rest;
  {  // telemetry (entries per particle): one atomic per block
    int mx = q == 0 && valid ? entries + nog : 0;
    for (int o = 8; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) wmax[wv] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < NW; ++w) mx = max(mx, wmax[w]);
      atomicMax(&d.flags->max_nb_slot[(tile % kSlots) * kLineInts], mx);
    }
  }
  if (!valid || q != 0) return;
  int nst = nblk * 8 + restp, nogp = (nog + kOtherBatch - 1) / kOtherBatch * kOtherBatch;
  if (max(nst, nogp) > d.cap || nst / PAD + nogp / kOtherBatch > units) {
    latch(d.flags, LE_E_CAPACITY);
    nst = nogp = 0;
  } else {
    for (; nog < nogp; ++nog) og_store(nog, og_entry((uint32_t)n, pack_img(0, 0, 0)));
  }
  d.n_plain[i] = nst;
  d.n_og[i] = nogp;
  if (d.chain_len > 0) {
    int tg_ = d.tag[an][i];
    int lo = -1, hi = -1;
    if (tg_ < d.n_bonded) {
      int kk = tg_ % d.chain_len;
      if (kk > 0) lo = d.slot_of_tag[tg_ - 1];
      if (kk < d.chain_len - 1) hi = d.slot_of_tag[tg_ + 1];
    }
    d.bond[i] = lo;
    d.bond[np + i] = hi;
  }
}

template <class TC, bool GL>
__global__ void __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(4))) k_neighbors(Dev d) {
  if (rebuild_off(d)) return;  // (the same two words for every wave)
  if (blockIdx.x == 0 && threadIdx.x == 0) d.joined[kPlace * kJoinedLine] = d.joined[kBinned * kJoinedLine] = 0ull;  // (of k_sort)
  neighbors_body<TC::HALO, GL>(d, d.ctrl, xcd_block(d.ntiles));
}

// (1) to (3) in one launch.  The blocks of the search wait for all of the scan;
// the last of them to have waited sets the counts back to zero.
template <class TC, bool GL>
__global__ void __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(4)))
    k_rebuild(Dev d, Ctrl* __restrict__ next, unsigned long long* __restrict__ next_vmax, int control) {
  __shared__ Ctrl sc, sn;
  if (!sort_control(d, next, next_vmax, 0, control, blockIdx.x, sc, sn)) return;
  const int nbb = (d.n + kBinBlock - 1) / kBinBlock;
  int b = take_place(&d.joined[kPlace * kJoinedLine]);
  if (b < nbb) {
    bin_body<kSearchThreads>(d, sc, b);
    add_count(&d.joined[kBinned * kJoinedLine]);
    return;
  }
  b -= nbb;
  if (b < d.sp_blocks) {
    if (!wait_count(d, &d.joined[kBinned * kJoinedLine], nbb)) return;
    scan_permute_body<kSearchThreads>(d, sn, b);
    add_count(&d.joined[kSorted * kJoinedLine]);
    return;
  }
  b -= d.sp_blocks;
  if (!wait_count(d, &d.joined[kSorted * kJoinedLine], d.sp_blocks)) return;
  if (threadIdx.x == 0 && atomicAdd(&d.joined[kWaited * kJoinedLine], 1ull) == (unsigned long long)d.ntiles - 1ull)
    for (int k = 0; k < kJoined; ++k) d.joined[k * kJoinedLine] = 0ull;
  neighbors_body<TC::HALO, GL>(d, &sn, xcd_map(b, d.ntiles));
}

constexpr int kSpreadRun = 4;  // consecutive tiles per run of the batched list search

// Batched form: only the members that rebuild at this step have work, so the
// blocks are spread over the XCDs in short runs (xcd_spread) rather than in
// one contiguous range per XCD; then the tile is located.
template <class TC, bool GL>
__global__ void __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(4))) k_neighbors_b(Batch b) {
  int sm, tile;
  locate(b, xcd_spread<kSpreadRun>((int)blockIdx.x, (int)gridDim.x), sm, tile);
  const Dev& d = stage_dev(b.dev[sm]);
  if (rebuild_off(d)) return;
  neighbors_body<TC::HALO, GL>(d, d.ctrl, tile);
}

// ---------------------------------------------------------- integrator
// Block maximum of |c|^2 into one of the kSlots words; called by every
// thread of a block of exactly NTH threads (the LDS array holds one entry per
// wave of that block; launches pass the kernel's own block size).
template <int NTH>
__device__ __forceinline__ void vmax_commit(const Dev& d, double v2, int lb, int nw = NTH / 64) {
  static_assert(NTH % 64 == 0 && NTH <= 1024, "whole waves, at most 16");
  __shared__ double wm[NTH / 64];
  double m = 0.0;
  if ((int)(threadIdx.x >> 6) < nw) {
    m = wave_max(v2);
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w) m = fmax(m, wm[w]);
    atomicMax(&d.vmax[(lb % kSlots) * kLineU64], (unsigned long long)__double_as_longlong(m));
  }
}

// Sum the per-block stress partials (fixed order) and write the stress
// -(K + W)/V, or with virial_only the pair virial W, into out6.  Called by one
// whole block of kBlock threads.
__device__ void reduce_partials(const Dev& d, double* out6, bool virial_only) {
  __shared__ double red[kBlock / 64][kStressComps];
  double acc[kStressComps];
#pragma unroll
  for (int k = 0; k < kStressComps; ++k) acc[k] = 0.0;
  for (int b = threadIdx.x; b < d.nblocks; b += blockDim.x) {
#pragma unroll
    for (int k = 0; k < kStressComps; ++k) acc[k] += d.partials[b * kStressComps + k];
  }
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kStressComps; ++k) {
    double v = acc[k];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) red[wid][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    double kin = 0.0, vir = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) {
      kin += red[w][threadIdx.x];
      vir += red[w][6 + threadIdx.x];
    }
    out6[threadIdx.x] = virial_only ? vir : -(kin + vir) * d.inv_vol;
  }
}

// First half-kick and drift from a state with full-step velocities:
// u += dt/(2m) F ; x_new = x + dt u (into the other position buffer).  The
// step is advanced by the next control kernel.
__device__ __forceinline__ void kick_drift_body(const Dev& d, int bid) {
  __shared__ int skip;
  Ctrl* c = d.ctrl;
  if (threadIdx.x == 0) skip = d.flags->status;
  __syncthreads();
  if (skip) return;
  int i = bid * kBlock + threadIdx.x;
  const int np = d.np;
  double v2 = 0.0;
  if (i < d.n) {
    const int pc = c->pos_cur, ac = c->aux_cur;
    double4 p = reinterpret_cast<const double4*>(d.pos[pc])[i];
    double* U = d.vel[ac];
    const double* F = d.frc[ac];
    double ux = U[i] + d.h * F[i];
    double uy = U[np + i] + d.h * F[np + i];
    double uz = U[2 * np + i] + d.h * F[2 * np + i];
    double cx = ux - d.c_sr * (p.y - 0.5 * d.Ly);
    v2 = cx * cx + uy * uy + uz * uz;
    U[i] = ux; U[np + i] = uy; U[2 * np + i] = uz;
    double4 q;
    q.x = p.x + d.dt * (ux + d.drift_sr * (p.y - 0.5 * d.Ly));
    q.y = p.y + d.dt * uy;
    q.z = p.z + d.dt * uz;
    q.w = p.w;
    reinterpret_cast<double4*>(d.pos[1 - pc])[i] = q;
    if (!(isfinite(q.x) && isfinite(q.y) && isfinite(q.z))) latch(d.flags, LE_E_NONFINITE);
  }
  vmax_commit<kBlock>(d, v2, bid);
}

__global__ void __launch_bounds__(kBlock) k_kick_drift(Dev d) { kick_drift_body(d, blockIdx.x); }

__global__ void __launch_bounds__(kBlock) k_kick_drift_b(Batch b) {
  int sm, bid;
  locate(b, blockIdx.x, sm, bid);
  kick_drift_body(stage_dev(b.dev[sm]), bid);
}

// ---------------------------------------------------------- force kernel
template <bool VIR>
__device__ __forceinline__ void add_pair(double f, double dx, double dy, double dz, double& fx,
                                         double& fy, double& fz, double* w) {
  fx = fma(f, dx, fx); fy = fma(f, dy, fy); fz = fma(f, dz, fz);
  if (VIR) {
    double ax = f * dx, ay = f * dy, az = f * dz;
    w[0] = fma(dx, ax, w[0]); w[1] = fma(dy, ay, w[1]); w[2] = fma(dz, az, w[2]);
    w[3] = fma(dx, ay, w[3]); w[4] = fma(dx, az, w[4]); w[5] = fma(dy, az, w[5]);
  }
}

// Scalar LJ force factor f (force on i = f d) for r^2 = r2, zero outside the
// cutoff: f = 24 eps s^3 (2 s^3 - 1) / r^2 with s = sigma^2 / r^2.  The FP64 form without
// a cap leaves the factor 48 eps / sigma^2 (Dev::lj_c) to the sums over pairs and
// returns s^4 (s^3 - 1/2): powers of the ratio alone, which do not under- or
// overflow for small or large units of length.
// Branch-free so that the candidates of one batch are independent
// instruction streams the compiler can interleave.  The FP64 form is bound by
// the vector unit's issue, so it counts instructions: 1/r^2 from the hardware
// reciprocal (within 2^-22) and one third-order step (its residual e leaves
// e^3), and the cutoff clears the high word of 1/r^2 alone, whose square
// then underflows to zero.  With CAP (FP64 only) the magnitude |f| r is limited
// to cap: |f| <= cap / r.
template <bool MIXED, bool CAP = false>
__device__ __forceinline__ double lj_masked(const Dev& d, double r2) {
  static_assert(!(MIXED && CAP), "the capped force law is FP64");
  const bool in = r2 < d.rc2;
  if (MIXED) {
    float r2f = (float)r2;
    float inv = __builtin_amdgcn_rcpf(r2f);
    inv = inv * (2.0f - r2f * inv);  // one Newton step: ~1 ulp
    float s2 = (float)d.sig2 * inv;
    float s6 = s2 * s2 * s2;
    float f = (float)d.eps24 * s6 * (2.0f * s6 - 1.0f) * inv;
    return (double)(in ? f : 0.0f);
  } else {
    double inv = __builtin_amdgcn_rcp(r2);
    const double e = fma(-r2, inv, 1.0);
    inv = fma(inv, fma(e, e, e), inv);
    inv = __hiloint2double(in ? __double2hiint(inv) : 0, __double2loint(inv));
    const double s = d.sig2 * inv, s2 = s * s;
    double f = (s2 * s2) * fma(s2, s, -0.5);
    if (CAP) {
      f = d.lj_c * f;
      const double lim = d.force_cap / sqrt(r2);
      f = fmin(fmax(f, -lim), lim);
    }
    return f;
  }
}

// Lees-Edwards nearest-image displacement a - b (the integers by rounding;
// valid for bonded beads, which are far closer than half a box).
__device__ __forceinline__ void near_disp(const Dev& d, double4 a, double4 b, double Delta, double& dx,
                                          double& dy, double& dz) {
  const double dy0 = a.y - b.y;
  const double sy = rint(dy0 / d.Ly);
  dy = dy0 - sy * d.Ly;
  const double dx0 = (a.x - b.x) - sy * Delta;
  const double sx = rint(dx0 / d.Lx);
  dx = dx0 - sx * d.Lx;
  const double dz0 = a.z - b.z;
  const double sz = rint(dz0 / d.Lz);
  dz = dz0 - sz * d.Lz;
}

// Cosine angle term (Eq. angle) read as V = k (1 + cos theta), minimum at a
// straight chain: theta the angle between b1 = x_a - x_j and b2 = x_b - x_j at
// the middle bead j.  Forces on the two ends (F_j = -(F_a + F_b)):
//   F_a = -k [b2 / (l1 l2) - cos(theta) b1 / l1^2],  F_b likewise.
__device__ __forceinline__ void angle_cos(const double b1[3], const double b2[3], double k, double Fa[3],
                                          double Fb[3]) {
  const double l11 = b1[0] * b1[0] + b1[1] * b1[1] + b1[2] * b1[2];
  const double l22 = b2[0] * b2[0] + b2[1] * b2[1] + b2[2] * b2[2];
  const double l12 = sqrt(l11) * sqrt(l22);
  const double c = (b1[0] * b2[0] + b1[1] * b2[1] + b1[2] * b2[2]) / l12;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    Fa[a] = -k * (b2[a] / l12 - c * b1[a] / l11);
    Fb[a] = -k * (b1[a] / l12 - c * b2[a] / l22);
  }
}

// DPD pair terms (Eqs. dissipative, random, omega) on particle i from one
// partner: d = x_i - x_j(image), v = u_i - u_j(image) (the image's streaming
// velocity already removed), r2 = |d|^2.  Adds f d with
// f = [-gamma w^2 (d.v / r) + sqrt(24 gamma kT / dt) w theta_ij] / r,
// w = 1 - r / r_c, zero at and beyond r_c.  theta_ij is word 0 of the Philox
// block with counter (step, smaller tag, larger tag), so both members of the
// pair draw the same number and their forces cancel.
__device__ __forceinline__ void dpd_pair(const Dev& d, uint32_t s_lo, uint32_t s_hi, int ti, int tj,
                                         double vx, double vy, double vz, double dx, double dy,
                                         double dz, double r2, double& ax, double& ay, double& az) {
  // 1/r from the hardware reciprocal square root (within 2^-22) and one
  // third-order step (its residual e leaves e^3), then r = r2 / r
  double ir = __builtin_amdgcn_rsq(r2);
  const double e = fma(-(r2 * ir), ir, 1.0);
  ir = fma(ir * e, fma(e, 0.375, 0.5), ir);
  const double wgt = fmax(fma(-(r2 * ir), d.dpd_inv_rc, 1.0), 0.0);
  const double ev = fma(dz, vz, fma(dy, vy, dx * vx)) * ir;
  uint32_t c[4] = {s_lo, s_hi, (uint32_t)min(ti, tj), (uint32_t)max(ti, tj)};
  philox(c, d.seed_lo, d.dpd_key_hi);
  const double f = (wgt * ir) * fma(-(d.dpd_gamma * wgt), ev, d.dpd_pref * u01c(c[0]));
  ax = fma(f, dx, ax); ay = fma(f, dy, ay); az = fma(f, dz, az);
}

// Block reduction of 12 per-thread sums into partials[block][12] (fixed
// order: wave butterflies, then waves in index order).  Called by every thread
// of a block of exactly NTH threads (one LDS row per wave of that block).
template <int NTH>
__device__ __forceinline__ void block_partials(double* vals, double* out, int lb,
                                               int nwrite = kStressComps, int nw = NTH / 64) {
  static_assert(NTH % 64 == 0 && NTH <= 1024, "whole waves, at most 16");
  __shared__ double red[NTH / 64][kStressComps];
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (wid < nw) {
#pragma unroll
    for (int k = 0; k < kStressComps; ++k) {
      double v = vals[k];
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0) red[wid][k] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x < nwrite) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w][threadIdx.x];
    out[lb * kStressComps + threadIdx.x] = s;
  }
}

// One evaluation of the conservative force for every particle, and then,
// depending on MODE:
//   kForcesOnly  write F^c in tag order (+ kinetic and virial partials)
//   kInitForce   F = F^c + Langevin(u) of the current step into frc
//   kStepLast    F as above from the half-step velocity, u += dt/(2m) F
//   kStepFused   as kStepLast, then the next half-kick and drift
//   kDpdForce    F = F^c + DPD pair terms of the current (half-step)
//                velocities into frc; k_integrate then moves the particles
//                (velocities of partners must not change while it runs)
// Langevin force (Eq. langevin on the peculiar velocity, Eq. vi):
//   F = F^c - gamma m c + sqrt(24 gamma m kT / dt) theta,  c = u - gamma_dot (y - L_y/2) e_x
// (with the friction on the lab velocity, c = u of the image inside the box).
// With the LDS halo the block has kForceThreads / tile threads per particle:
// threads t, t + tile, ... take the particle's batches in turn (more waves per
// CU for the same LDS), and hand their partial sums to the first through LDS
// before the epilogue.  Staging what lies within reach of a compact tile (about
// 1250 positions for 128 LJ particles instead of 1900, 550 for beads of a
// melt), lists in blocks of 4 and 22 vector instructions per entry took the
// plain step from 43 to 36.5 us for 256,000 LJ particles and, against gathers from
// global memory, from 37 to 26.7 us for 400,000 beads (traced); it is bound by the vector unit's
// issue (77% busy) and the waves' imbalance, six waves per SIMD in 80 registers.
// DPD steps with the halo gather the velocities (from vt, with the slots kept
// in LDS beside the positions) of the partners within the DPD cutoff alone: all
// from memory, four gathers per entry, the kernel waited for them (256,000 LJ
// particles: 113 -> 93 us; 2000 49 -> 29 us per step), four waves per SIMD in 128
// registers, two blocks of 57 KB LDS per CU.
// Without the halo the launch bound of four tiles per block makes the
// compiler keep fewer registers (more waves; DPD 138 -> 132 us); the launch
// itself uses one tile.
template <int MODE, bool MIXED, bool BONDS, bool SAMPLE, class TC, bool CAP>
__device__ __forceinline__ void force_body(const Dev& d, const int lb, double* __restrict__ f_out) {
  constexpr bool STAGED = TC::HALO > 0;
  static_assert(!CAP || (!STAGED && !MIXED && MODE != kDpdForce), "capped forces: FP64, global layout");
  constexpr bool VIR = SAMPLE || (MODE == kForcesOnly);
  constexpr bool DPD = MODE == kDpdForce;
  constexpr int kTh = TC::kForceThreads;                // threads per block
  const int kP = STAGED ? d.tile : kTile;               // particles per block (a power of 2)
  const int TPP = STAGED ? kTh / kP : 1;                // threads per particle
  constexpr int HALO = TC::HALO;
  constexpr int kH = STAGED ? HALO + 1 : 1;  // no halo: every partner from global memory
  static_assert(HALO % kTh == 0, "whole staging rounds");
  static_assert(!STAGED || 3 * kH >= kTh * 9, "the halo holds the partial-sum exchange");
  __shared__ double hbuf[3 * kH];
  double* const hx = hbuf;
  double* const hy = hbuf + kH;
  double* const hz = hbuf + 2 * kH;
  __shared__ uint32_t hent[DPD && STAGED ? kH : 1];  // slot and image of every staged position
  __shared__ int skip;
  Ctrl* c = d.ctrl;
  if (threadIdx.x == 0) skip = d.flags->status;
  __syncthreads();
  if (skip) return;
  const int half = STAGED ? (int)threadIdx.x >> d.tile_sh : 0;
  const int tl = (int)threadIdx.x & (kP - 1);  // particle within the tile
  const int i = lb * kP + tl;
  const bool valid = i < d.n;
  const int np = d.np;
  const int pc = c->pos_cur, ac = c->aux_cur;
  const double Delta = c->Delta;
  const int W = c->wraps;
  const double4* P = reinterpret_cast<const double4*>(d.pos[pc]);
  // Per-particle data and the first list blocks are requested before and
  // during the halo staging so that their latency overlaps it (loads use a
  // clamped index; values of invalid lanes are never used).
  const int ic = valid ? i : 0;
  const double4 pi_ld = P[ic];
  const int npl_ld = STAGED ? d.n_plain[ic] : 0;
  const double* Uv = d.vel[ac];
  const double u0_ld = Uv[ic], u1_ld = Uv[np + ic], u2_ld = Uv[2 * np + ic];
  const int tag_ld = d.tag[ac][ic];
  // staged entries: block b of 4 (half a unit) of the particle's list
  const uint2* __restrict__ l4s = reinterpret_cast<const uint2*>(d.nl + ic);
  const int nb = STAGED ? npl_ld / 4 : 0;
  auto boff = [&](int b) -> size_t { return b < nb ? (size_t)(b >> 1) * (2 * np) + (b & 1) : 0; };
  uint2 t0 = make_uint2(0u, 0u), t1 = t0;
  // Stage the tile's halo: the slots recorded at the last build with their
  // current positions, each shifted by its periodic / Lees-Edwards image
  // (sy Delta + sx L_x, sy L_y, sz L_z; the x image absorbs the offset's
  // wraps since the build).  A partner's displacement is then x_i - x_h.  All
  // slot loads, then all position loads, are in flight together.
  if (STAGED) {
    const int nst = d.tile_nstage[lb];
    const uint32_t* hs = d.halo + (size_t)lb * HALO;
    constexpr int U = STAGED ? HALO / kTh : 1;
    // the last round only where the tile has that many positions
    constexpr int U0 = U > 1 ? U - 1 : 1;
    const uint32_t sent = og_entry((uint32_t)d.n, pack_img(0, 0, 0));
    auto stage = [&](auto r0, auto r1, bool lists) {
      constexpr int R0 = decltype(r0)::value, N = decltype(r1)::value - R0;
      uint32_t ent[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        // always load from an index inside this tile's table, then select the value
        int h = threadIdx.x + (R0 + u) * kTh;
        int hh = h < nst ? h : 0;
        const uint32_t ev = hs[hh];
        ent[u] = (h < nst) ? ev : sent;
      }
      if (lists) {
        t0 = l4s[boff(half)];
        t1 = l4s[boff(half + TPP)];
      }
      // every position is loaded and written (past nst: the sentinel slot, an
      // unused LDS entry), so that no load is sunk into a condition and all of
      // them are in flight together
      double4 pj[N];
#pragma unroll
      for (int u = 0; u < N; ++u) pj[u] = P[ent[u] & kSlotMask];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int h = threadIdx.x + (R0 + u) * kTh;
        const uint32_t code = ent[u] >> kSlotBits;
        if (__any(code != pack_img(0, 0, 0))) {  // (no image of any: most waves away from the faces)
          int sx, sy, sz;
          unpack_img((uint8_t)code, sx, sy, sz);
          sx += sy * W;
          pj[u].x = pj[u].x + ((double)sy * Delta + (double)sx * d.Lx);
          pj[u].y = pj[u].y + (double)sy * d.Ly;
          pj[u].z = pj[u].z + (double)sz * d.Lz;
        }
        hx[h] = pj[u].x;
        hy[h] = pj[u].y;
        hz[h] = pj[u].z;
        if (DPD) hent[h] = ent[u];
      }
    };
    stage(std::integral_constant<int, 0>{}, std::integral_constant<int, U0>{}, true);
    if constexpr (U > U0) {
      if (nst > U0 * kTh) stage(std::integral_constant<int, U0>{}, std::integral_constant<int, U>{}, false);
    }
    if (threadIdx.x == 0) {
      hx[HALO] = 1e100; hy[HALO] = 1e100; hz[HALO] = 1e100;
      if (DPD) hent[HALO] = sent;
    }
    __syncthreads();
  }
  double fx = 0.0, fy = 0.0, fz = 0.0;
  double gx = 0.0, gy = 0.0, gz = 0.0;  // DPD pair terms (kept out of the virial)
  double w[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const double4 pi = valid ? pi_ld : make_double4(0.0, 0.0, 0.0, 0.0);
  const uint32_t st_lo = (uint32_t)(uint64_t)c->step, st_hi = (uint32_t)((uint64_t)c->step >> 32);
  const VtRec* __restrict__ VT = d.vt;
  if (valid) {
    // staged partners (already shifted to their image): the particle's list is
    // a sequence of blocks of 4, of which this thread takes blocks half, half +
    // TPP, ... (a wave runs to its longest list: with blocks of 8, lists of
    // 100 entries ran as 128); one 8-byte index load per block, two of this
    // thread's blocks ahead.  Past the list the first block is loaded and not used.
    for (int b = half; b < nb; b += TPP) {
      const uint2 t2 = l4s[boff(b + 2 * TPP)];
      const int j[4] = {(int)(t0.x & 0xffff), (int)(t0.x >> 16), (int)(t0.y & 0xffff), (int)(t0.y >> 16)};
      double xj[4], yj[4], zj[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) { xj[u] = hx[j[u]]; yj[u] = hy[j[u]]; zj[u] = hz[j[u]]; }
      if constexpr (DPD && STAGED) {
        // the velocities of the partners within the DPD cutoff are gathered (of
        // the others the sentinel's: one line for all) while the conservative
        // force is computed
        double dx[4], dy[4], dz[4], r2[4];
        uint32_t ej[4];
        VtRec vj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ej[u] = hent[j[u]];
        bool image = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          dx[u] = pi.x - xj[u]; dy[u] = pi.y - yj[u]; dz[u] = pi.z - zj[u];
          r2[u] = fma(dz[u], dz[u], fma(dy[u], dy[u], dx[u] * dx[u]));
          vj[u] = VT[r2[u] < d.dpd_rc2 ? ej[u] & kSlotMask : (uint32_t)d.n];
          image |= ej[u] >> kSlotBits != pack_img(0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          add_pair<VIR>(lj_masked<MIXED>(d, r2[u]), dx[u], dy[u], dz[u], fx, fy, fz, w);
        double vx[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) vx[u] = u0_ld - vj[u].x;
        if (__any(image)) {  // the image s_y boxes up streams faster by s_y gamma_dot L_y
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            int sx, sy, sz;
            unpack_img((uint8_t)(ej[u] >> kSlotBits), sx, sy, sz);
            vx[u] = vx[u] - (double)sy * d.sv;
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          dpd_pair(d, st_lo, st_hi, tag_ld, vj[u].tag, vx[u], u1_ld - vj[u].y, u2_ld - vj[u].z, dx[u], dy[u], dz[u],
                   r2[u], gx, gy, gz);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          double dx = pi.x - xj[u], dy = pi.y - yj[u], dz = pi.z - zj[u];
          const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
          add_pair<VIR>(lj_masked<MIXED>(d, r2), dx, dy, dz, fx, fy, fz, w);
        }
      }
      t0 = t1;
      t1 = t2;
    }
    // partners that were not staged: global memory, exact image arithmetic;
    // the next round's indices requested ahead.  With the halo the threads of
    // a particle take rounds in turn.
    const int nfo = STAGED ? 0 : d.n_plain[i] / kOtherBatch;
    const int nbo = nfo + d.n_og[i] / kOtherBatch;
    const int last_ob = d.units - 1;
    auto ooff = [&](int q) -> size_t {
      const int b = STAGED || q >= nfo ? last_ob - min(q - nfo, last_ob) : q;
      return (size_t)b * np + i;
    };
    const uint4* __restrict__ l4 = d.nl;
    // GB blocks of 4 per round: one for the plain global layout (fewer
    // gathers in flight leave room for more waves: KG 49 -> 48 us) and for the rows that the
    // halo did not hold, two for DPD from global memory (one block: 138 -> 195 us)
    constexpr int GB = DPD && !STAGED ? 2 : 1;
    uint4 jn[GB];
#pragma unroll
    for (int k = 0; k < GB; ++k) jn[k] = l4[ooff(half * GB + k)];
    {
    for (int b = half * GB; b < nbo; b += TPP * GB) {
      // slots, and the four image codes of a block repacked into one word
      // (fewer live registers while the gathers are in flight)
      uint32_t sl[4 * GB], cq[GB];
#pragma unroll
      for (int k = 0; k < GB; ++k) {
        const uint4 jq = jn[k];
        jn[k] = l4[ooff(b + TPP * GB + k)];
        const bool in = b + k < nbo;  // the entries of this block are the list's
        sl[4 * k] = (in ? jq.x : (uint32_t)d.n) & kSlotMask;
        sl[4 * k + 1] = (in ? jq.y : (uint32_t)d.n) & kSlotMask;
        sl[4 * k + 2] = (in ? jq.z : (uint32_t)d.n) & kSlotMask;
        sl[4 * k + 3] = (in ? jq.w : (uint32_t)d.n) & kSlotMask;
        cq[k] = (jq.x >> kSlotBits) | ((jq.y >> kSlotBits) << 8) | ((jq.z >> kSlotBits) << 16) |
                (jq.w & ~kSlotMask);
        // opaque to the optimiser, so that the codes stay one packed word
        // instead of being unpacked from the entries ahead of their use
        asm("" : "+v"(cq[k]));
      }
      double4 pj[4 * GB];
#pragma unroll
      for (int u = 0; u < 4 * GB; ++u) pj[u] = P[sl[u]];
      // DPD: the partners' velocities and tags, one 32-byte gather each
      VtRec vj[DPD ? 4 * GB : 1];
      if (DPD) {
#pragma unroll
        for (int u = 0; u < 4 * GB; ++u) vj[u] = VT[sl[u]];
        // every gather of the round issued before the first use (without this
        // fence the scheduler sinks each to its use, one wait per gather)
        __builtin_amdgcn_sched_barrier(0);
      }
      // four at a time: displacements, less the image shifts where any lane has
      // one (most waves are away from the faces); a DPD image s_y boxes up
      // streams faster by s_y gamma_dot L_y
#pragma unroll
      for (int k = 0; k < GB; ++k) {
        double dx[4], dy[4], dz[4], vx[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double4 p = pj[4 * k + u];
          dx[u] = pi.x - p.x; dy[u] = pi.y - p.y; dz[u] = pi.z - p.z;
          vx[u] = DPD ? u0_ld - vj[DPD ? 4 * k + u : 0].x : 0.0;
        }
        // (without DPD the test costs more than it saves: it spills registers in batches)
        if (!DPD || __any(cq[k] != 0x01010101u * pack_img(0, 0, 0))) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            int sx, sy, sz;
            unpack_img((uint8_t)(cq[k] >> (8 * u)), sx, sy, sz);
            sx += sy * W;
            dy[u] = dy[u] - (double)sy * d.Ly;
            dx[u] = (dx[u] - (double)sy * Delta) - (double)sx * d.Lx;
            dz[u] = dz[u] - (double)sz * d.Lz;
            if (DPD) vx[u] = vx[u] - (double)sy * d.sv;
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double r2 = fma(dz[u], dz[u], fma(dy[u], dy[u], dx[u] * dx[u]));
          add_pair<VIR>(lj_masked<MIXED, CAP>(d, r2), dx[u], dy[u], dz[u], fx, fy, fz, w);
          if (DPD) {
            const VtRec v = vj[DPD ? 4 * k + u : 0];
            dpd_pair(d, st_lo, st_hi, tag_ld, v.tag, vx[u], u1_ld - v.y, u2_ld - v.z, dx[u], dy[u], dz[u], r2, gx,
                     gy, gz);
          }
        }
      }
    }
    }
    if (!MIXED && !CAP) {  // (see lj_masked)
      fx *= d.lj_c; fy *= d.lj_c; fz *= d.lj_c;
      if (VIR) for (int q = 0; q < 6; ++q) w[q] *= d.lj_c;
    }
    if (BONDS && half == 0) {
      // FENE (Eq. fene), always float64; displacement by the nearest image
      int jb[2];
      double4 pb[2];
      for (int b = 0; b < 2; ++b) {
        int j = d.bond[b * np + i];
        jb[b] = j;
        if (j < 0) continue;
        double4 pj = P[j];
        pb[b] = pj;
        double dx, dy, dz;
        near_disp(d, pi, pj, Delta, dx, dy, dz);
        double r2 = dx * dx + dy * dy;
        r2 = r2 + dz * dz;
        if (!(r2 < d.fene_r02)) {
          latch(d.flags, LE_E_BOND);
          continue;
        }
        double f = -d.fene_k / (1.0 - r2 / d.fene_r02);
        add_pair<VIR>(f, dx, dy, dz, fx, fy, fz, w);
      }
      if (d.angle_k != 0.0) {
        // cosine angle term (Eq. angle): the angles centred at i (its virial
        // is counted here), at the bead below (i is its second end) and at
        // the bead above (i is its first end)
        double b1[3], b2[3], Fa[3], Fb[3];
        if (jb[0] >= 0 && jb[1] >= 0) {
          near_disp(d, pb[0], pi, Delta, b1[0], b1[1], b1[2]);
          near_disp(d, pb[1], pi, Delta, b2[0], b2[1], b2[2]);
          angle_cos(b1, b2, d.angle_k, Fa, Fb);
          fx -= Fa[0] + Fb[0]; fy -= Fa[1] + Fb[1]; fz -= Fa[2] + Fb[2];
          if (VIR) {
            // w holds twice the virial (pairs and bonds are met from both
            // ends), so the angle's single contribution enters doubled
            w[0] += 2.0 * (b1[0] * Fa[0] + b2[0] * Fb[0]);
            w[1] += 2.0 * (b1[1] * Fa[1] + b2[1] * Fb[1]);
            w[2] += 2.0 * (b1[2] * Fa[2] + b2[2] * Fb[2]);
            w[3] += 2.0 * (b1[0] * Fa[1] + b2[0] * Fb[1]);
            w[4] += 2.0 * (b1[0] * Fa[2] + b2[0] * Fb[2]);
            w[5] += 2.0 * (b1[1] * Fa[2] + b2[1] * Fb[2]);
          }
        }
        for (int b = 0; b < 2; ++b) {
          const int j = jb[b];
          if (j < 0) continue;
          const int j2 = d.bond[b * np + j];  // the next bead beyond j
          if (j2 < 0) continue;
          const double4 p2 = P[j2];
          // angle (j2, j, i) below or (i, j, j2) above; i's force is that of its end
          near_disp(d, p2, pb[b], Delta, b1[0], b1[1], b1[2]);
          near_disp(d, pi, pb[b], Delta, b2[0], b2[1], b2[2]);
          angle_cos(b1, b2, d.angle_k, Fa, Fb);
          fx += Fb[0]; fy += Fb[1]; fz += Fb[2];
        }
      }
    }
  }
  if (DPD) { fx += gx; fy += gy; fz += gz; }
  if (STAGED) {
    // the other threads of each particle hand over their partial sums (the
    // halo array is free once every thread has left the pair loops); the
    // first adds them in thread order
    __syncthreads();
    if (half > 0) {
      double* ex = hbuf + ((half - 1) * kP + tl) * 9;
      ex[0] = fx; ex[1] = fy; ex[2] = fz;
      if (VIR) for (int q = 0; q < 6; ++q) ex[3 + q] = w[q];
    }
    __syncthreads();
    if (half == 0) {
      for (int t = 1; t < TPP; ++t) {
        const double* ex = hbuf + ((t - 1) * kP + tl) * 9;
        fx += ex[0]; fy += ex[1]; fz += ex[2];
        if (VIR) for (int q = 0; q < 6; ++q) w[q] += ex[3 + q];
      }
    } else {
      for (int q = 0; q < 6; ++q) w[q] = 0.0;
    }
  }
  const bool ep = valid && half == 0;  // threads that finish a particle
  double kin[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double v2 = 0.0;
  if (MODE == kForcesOnly) {
    if (ep) {
      int t = tag_ld;
      if (f_out) {
        f_out[t] = fx; f_out[d.n + t] = fy; f_out[2 * d.n + t] = fz;
      }
      double cx = u0_ld - d.c_sr * (pi.y - 0.5 * d.Ly);
      double cy = u1_ld, cz = u2_ld;
      double m = d.mass;
      kin[0] = m * cx * cx; kin[1] = m * cy * cy; kin[2] = m * cz * cz;
      kin[3] = m * cx * cy; kin[4] = m * cx * cz; kin[5] = m * cy * cz;
    }
  } else if (DPD) {
    if (ep) {
      double* F = d.frc[ac];
      F[i] = fx; F[np + i] = fy; F[2 * np + i] = fz;
    }
  } else if (ep) {
    double* U = d.vel[ac];
    double ux = u0_ld, uy = u1_ld, uz = u2_ld;
    int t = tag_ld;
    uint32_t ctr[4] = {st_lo, st_hi, (uint32_t)t, 0u};
    philox(ctr, d.seed_lo, d.seed_hi);
    // friction velocity: peculiar (Eq. vi), or the lab velocity of the image
    // inside the box (positions are wrapped lazily, so a particle above the
    // top face still carries the velocity it had before crossing)
    double cx = d.thermostat == LE_THERMO_LANGEVIN_LAB ? ux - d.sv * floor(pi.y / d.Ly)
                                                       : ux - d.c_sr * (pi.y - 0.5 * d.Ly);
    double Fx = (fx - d.gamma_m * cx) + d.pref * u01c(ctr[0]);
    double Fy = (fy - d.gamma_m * uy) + d.pref * u01c(ctr[1]);
    double Fz = (fz - d.gamma_m * uz) + d.pref * u01c(ctr[2]);
    if (MODE == kInitForce) {
      double* F = d.frc[ac];
      F[i] = Fx; F[np + i] = Fy; F[2 * np + i] = Fz;
    } else {
      ux = ux + d.h * Fx; uy = uy + d.h * Fy; uz = uz + d.h * Fz;
      if (SAMPLE) {
        double m = d.mass;
        double cxn = ux - d.c_sr * (pi.y - 0.5 * d.Ly);
        kin[0] = m * cxn * cxn; kin[1] = m * uy * uy; kin[2] = m * uz * uz;
        kin[3] = m * cxn * uy; kin[4] = m * cxn * uz; kin[5] = m * uy * uz;
      }
      if (MODE == kStepLast) {
        double* F = d.frc[ac];
        F[i] = Fx; F[np + i] = Fy; F[2 * np + i] = Fz;
      } else {
        ux = ux + d.h * Fx; uy = uy + d.h * Fy; uz = uz + d.h * Fz;
        double cxh = ux - d.c_sr * (pi.y - 0.5 * d.Ly);
        v2 = cxh * cxh + uy * uy + uz * uz;
        double4 q;
        q.x = pi.x + d.dt * (ux + d.drift_sr * (pi.y - 0.5 * d.Ly));
        q.y = pi.y + d.dt * uy;
        q.z = pi.z + d.dt * uz;
        q.w = pi.w;
        reinterpret_cast<double4*>(d.pos[1 - pc])[i] = q;
        if (!(isfinite(q.x) && isfinite(q.y) && isfinite(q.z))) latch(d.flags, LE_E_NONFINITE);
      }
      U[i] = ux; U[np + i] = uy; U[2 * np + i] = uz;
    }
  }
  // (the waves of the threads that finish particles)
  const int nw = (kP + 63) / 64;
  if (MODE == kStepFused) vmax_commit<kTh>(d, v2, lb, nw);
  if (VIR) {
    double vals[kStressComps];
#pragma unroll
    for (int k = 0; k < 6; ++k) { vals[k] = kin[k]; vals[6 + k] = 0.5 * w[k]; }
    block_partials<kTh>(vals, d.partials, lb, kStressComps, nw);
  }
}

// Waves per SIMD that the halo kernels are compiled for: six in 80 registers
// (plain steps), four in 128 (DPD); beads of sparse tiles in a batch, whose descriptor takes
// registers too, five (six spill: 16 melts 74 instead of 71 us a step).  Beads of dense
// tiles in a batch stay at six and spill 52 bytes: their blocks of eight waves fit a CU three
// times at six and twice at five or four (8 x 20,000 beads with a cutoff of 2.5: 70.6 us a step, 75.3
// at four); so do sampled DPD steps, 20 to 64 bytes, at four (8 x 20,000 particles 118 us, at
// three 135).  Without the halo the compiler chooses (DPD of 256,000 from
// global memory: 145 us a step; held to three waves it spills, 148).
constexpr int force_waves(int mode, int halo, bool sample, bool batch_bonds = false) {
  if (halo == 0) return 1;
  if (mode == kDpdForce) return 4;
  if (sample || mode == kForcesOnly) return 1;
  return batch_bonds && halo == TileSparse::HALO ? 5 : 6;
}

template <int MODE, bool MIXED, bool BONDS, bool SAMPLE, class TC, bool CAP = false>
__global__ void __launch_bounds__(TC::HALO ? TC::kForceThreads : 4 * kTile, force_waves(MODE, TC::HALO, SAMPLE))
    k_force(Dev d, double* __restrict__ f_out, double* __restrict__ sample_out) {
  (void)sample_out;
  force_body<MODE, MIXED, BONDS, SAMPLE, TC, CAP>(d, xcd_block(d.nblocks), f_out);
}

// Batched form (the step modes; no per-particle output): one launch over the
// tiles of every simulation of the batch.  Global layout: XCD-remapped over
// the whole grid (partner gathers hit the L2 of the XCD that holds the
// region); LDS halo: runs of 16 tiles dealt round-robin to the XCDs, which
// evens out members of unequal cost per tile (64-request batch 0.711 ->
// 0.699 ms per step; the KG melts of the global layout gain nothing from it).
template <int MODE, bool MIXED, bool BONDS, bool SAMPLE, class TC, bool CAP = false>
__global__ void __launch_bounds__(TC::HALO ? TC::kForceThreads : 4 * kTile, force_waves(MODE, TC::HALO, SAMPLE, BONDS)) k_force_b(Batch b) {
  int sm, lb;
  const int g = TC::kSpread ? xcd_spread<16>((int)blockIdx.x, (int)gridDim.x) : xcd_map((int)blockIdx.x, (int)gridDim.x);
  locate(b, g, sm, lb);
  force_body<MODE, MIXED, BONDS, SAMPLE, TC, CAP>(stage_dev(b.dev[sm]), lb, nullptr);
}

// DPD: pack the current velocities and tags of every slot into vt, so that the
// force kernel gathers one 32-byte record per partner (that of the sentinel slot n
// never changes).
__device__ __forceinline__ void pack_vt_body(const Dev& d, int bid) {
  if (d.flags->status) return;
  const Ctrl* c = d.ctrl;
  const int i = bid * kBlock + threadIdx.x;
  const int np = d.np;
  if (i < d.n) {
    const double* U = d.vel[c->aux_cur];
    d.vt[i] = VtRec{U[i], U[np + i], U[2 * np + i], d.tag[c->aux_cur][i], 0};
  }
}

__global__ void __launch_bounds__(kBlock) k_pack_vt(Dev d) { pack_vt_body(d, blockIdx.x); }

__global__ void __launch_bounds__(kBlock) k_pack_vt_b(Batch b) {
  int sm, bid;
  locate(b, blockIdx.x, sm, bid);
  pack_vt_body(stage_dev(b.dev[sm]), bid);
}

// DPD steps, after k_force<kDpdForce>: u += dt/(2m) F (the step's second
// half-kick); with SAMPLE the kinetic stress partials of the new full-step
// velocities go to partials[block][0..5] (the force kernel wrote the virial
// to [6..11]); unless LAST, the next half-kick and drift follow as in the
// fused Langevin step.  One thread per slot, blocks of kTile.
template <bool LAST, bool SAMPLE>
__device__ __forceinline__ void integrate_body(const Dev& d, int bid) {
  __shared__ int skip;
  Ctrl* c = d.ctrl;
  if (threadIdx.x == 0) skip = d.flags->status;
  __syncthreads();
  if (skip) return;
  const int i = bid * kTile + threadIdx.x;
  const int np = d.np;
  double kin[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double v2 = 0.0;
  if (i < d.n) {
    const int pc = c->pos_cur, ac = c->aux_cur;
    const double4 p = reinterpret_cast<const double4*>(d.pos[pc])[i];
    double* U = d.vel[ac];
    const double* F = d.frc[ac];
    const double Fx = F[i], Fy = F[np + i], Fz = F[2 * np + i];
    double ux = U[i] + d.h * Fx;
    double uy = U[np + i] + d.h * Fy;
    double uz = U[2 * np + i] + d.h * Fz;
    if (SAMPLE) {
      const double m = d.mass;
      const double cx = ux - d.c_sr * (p.y - 0.5 * d.Ly);
      kin[0] = m * cx * cx; kin[1] = m * uy * uy; kin[2] = m * uz * uz;
      kin[3] = m * cx * uy; kin[4] = m * cx * uz; kin[5] = m * uy * uz;
    }
    if (!LAST) {
      ux = ux + d.h * Fx; uy = uy + d.h * Fy; uz = uz + d.h * Fz;
      const double cxh = ux - d.c_sr * (p.y - 0.5 * d.Ly);
      v2 = cxh * cxh + uy * uy + uz * uz;
      double4 q;
      q.x = p.x + d.dt * (ux + d.drift_sr * (p.y - 0.5 * d.Ly));
      q.y = p.y + d.dt * uy;
      q.z = p.z + d.dt * uz;
      q.w = p.w;
      reinterpret_cast<double4*>(d.pos[1 - pc])[i] = q;
      if (!(isfinite(q.x) && isfinite(q.y) && isfinite(q.z))) latch(d.flags, LE_E_NONFINITE);
    }
    U[i] = ux; U[np + i] = uy; U[2 * np + i] = uz;
  }
  if (!LAST) vmax_commit<kTile>(d, v2, bid);
  if (SAMPLE) {
    double vals[kStressComps];
#pragma unroll
    for (int k = 0; k < 6; ++k) { vals[k] = kin[k]; vals[6 + k] = 0.0; }
    block_partials<kTile>(vals, d.partials, bid, 6);
  }
}

template <bool LAST, bool SAMPLE>
__global__ void __launch_bounds__(kTile) k_integrate(Dev d) { integrate_body<LAST, SAMPLE>(d, blockIdx.x); }

template <bool LAST, bool SAMPLE>
__global__ void __launch_bounds__(kTile) k_integrate_b(Batch b) {
  int sm, bid;
  locate(b, blockIdx.x, sm, bid);
  integrate_body<LAST, SAMPLE>(stage_dev(b.dev[sm]), bid);
}

// Stand-alone reduction of the block partials (le_forces, le_stress).
__global__ void k_stress_final(Dev d, double* out6, int virial_only) {
  __shared__ int skip;
  if (threadIdx.x == 0) skip = d.flags->status;
  __syncthreads();
  if (skip) return;
  reduce_partials(d, out6, virial_only != 0);
}

// Batched form: block k reduces simulation k's partials into out.ptr[k].
__global__ void k_stress_final_b(Batch b, BatchOut out) {
  const Dev& d = stage_dev(b.dev[blockIdx.x]);
  __shared__ int skip;
  if (threadIdx.x == 0) skip = d.flags->status;
  __syncthreads();
  if (skip) return;
  reduce_partials(d, out.ptr[blockIdx.x], false);
}

// Copy the current control state and speed-bound words into the other copy
// (a no-op for the simulation; lets a captured graph start on its copy).
__global__ void k_ctrl_copy(const Ctrl* __restrict__ src, Ctrl* __restrict__ dst,
                            const unsigned long long* __restrict__ vsrc,
                            unsigned long long* __restrict__ vdst) {
  if (threadIdx.x == 0) *dst = *src;
  for (int k = threadIdx.x; k < kSlots * kLineU64; k += blockDim.x) vdst[k] = vsrc[k];
}

// ---------------------------------------------------------- observables
// Each wave adds its particles' bins (their images in the box, with the
// matching lab u_x) to its own row of LDS sums, the waves of a block are added
// in wave order and the blocks in a fixed tree, so the sums are reproducible.
// Cell-sorted particles of one wave fall into a few bins, so a wave takes one
// bin at a time: all lanes of that bin by one butterfly, and, past a few, one particle
// at a time (1000 particles and 256 bins 30 us by butterflies alone).  At most kObsBlocks
// blocks (two a CU; a block takes several rounds of kBlock particles), and a
// final pass over many blocks: with one thread per bin over the particles of
// a block and one block over all partial rows, 256,000 particles and 50 bins took
// 28 + 250 us.
constexpr int kObsStride = 3 * LE_MAX_BINS + 4;
constexpr int kObsBlocks = 512;
constexpr int kObsCols = 16;  // columns per block of the final pass
constexpr int kObsRows = kBlock / kObsCols;
constexpr int kObsBins = 8;    // bins that a wave takes by butterflies
constexpr int kObsLane = LE_MAX_BINS / 64;  // bins a lane keeps after those
static_assert(LE_MAX_BINS % 64 == 0, "whole bins per lane");

static inline int obs_blocks(int n) {
  const int nb = (n + kBlock - 1) / kBlock;
  return nb < kObsBlocks ? nb : kObsBlocks;
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double read_lane(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

__global__ void __launch_bounds__(kBlock) k_obs_partial(Dev d, int nbins, int nblk) {
  constexpr int kW = kBlock / 64;
  __shared__ double acc[kW][3 * LE_MAX_BINS];
  __shared__ double red[kW][4];
  if (d.flags->status) return;
  const Ctrl* c = d.ctrl;
  const int np = d.np;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int k = lane; k < 3 * nbins; k += 64) acc[wid][k] = 0.0;
  const double4* P = reinterpret_cast<const double4*>(d.pos[c->pos_cur]);
  const double* U = d.vel[c->aux_cur];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  const int rounds = (d.n + nblk * kBlock - 1) / (nblk * kBlock);
  for (int rd = 0; rd < rounds; ++rd) {
    const int i = ((int)blockIdx.x * rounds + rd) * kBlock + (int)threadIdx.x;
    int b = -1;
    double ux = 0.0, mc2 = 0.0;
    if (i < d.n) {
      const double4 p = P[i];
      const double u0 = U[i], u1 = U[np + i], u2 = U[2 * np + i];
      double y = p.y;
      const double ky = wrap1(y, d.Ly);
      ux = (u0 - ky * d.jump_sv) + d.drift_sr * (y - 0.5 * d.Ly);  // lab u_x of the in-box image
      b = (int)(y / d.Ly * (double)nbins);
      if (b < 0) b = 0;
      if (b > nbins - 1) b = nbins - 1;
      const double cx = u0 - d.c_sr * (p.y - 0.5 * d.Ly);
      mc2 = d.mass * (cx * cx + u1 * u1 + u2 * u2);
      v[0] += mc2;
      v[1] += ux; v[2] += u1; v[3] += u2;
    }
    unsigned long long rem = __ballot(b >= 0);
    for (int k = 0; k < kObsBins && rem; ++k) {
      const int bb = __builtin_amdgcn_readlane(b, __builtin_ctzll(rem));
      const bool mine = b == bb;
      const unsigned long long m = __ballot(mine);
      rem &= ~m;
      const double su = wave_sum(mine ? ux : 0.0), sk = wave_sum(mine ? mc2 : 0.0);
      if (lane == 0) {
        acc[wid][bb] += (double)__popcll(m);
        acc[wid][nbins + bb] += su;
        acc[wid][2 * nbins + bb] += sk;
      }
    }
    if (rem) {  // many bins: a lane keeps every 64th, and the particles left go by one at a time
      double s[kObsLane][3] = {};
      while (rem) {
        const int l = __builtin_ctzll(rem);
        rem &= rem - 1ull;
        const int bb = __builtin_amdgcn_readlane(b, l);
        const double xl = read_lane(ux, l), kl = read_lane(mc2, l);
#pragma unroll
        for (int q = 0; q < kObsLane; ++q)
          if (bb == lane + 64 * q) { s[q][0] += 1.0; s[q][1] += xl; s[q][2] += kl; }
      }
#pragma unroll
      for (int q = 0; q < kObsLane; ++q)
        if (lane + 64 * q < nbins)
          for (int a = 0; a < 3; ++a) acc[wid][a * nbins + lane + 64 * q] += s[q][a];
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double t = wave_sum(v[k]);
    if (lane == 0) red[wid][k] = t;
  }
  __syncthreads();
  double* out = d.obs_part + (size_t)blockIdx.x * kObsStride;
  for (int k = threadIdx.x; k < 3 * nbins; k += kBlock) {
    double t = 0.0;
    for (int w = 0; w < kW; ++w) t += acc[w][k];
    out[k] = t;
  }
  if (threadIdx.x < 4) {
    double t = 0.0;
    for (int w = 0; w < kW; ++w) t += red[w][threadIdx.x];
    out[3 * nbins + threadIdx.x] = t;
  }
}

// kObsCols columns per block, kObsRows threads per column: each adds every
// kObsRows-th block's partial, then the threads of a column are added in order.
__global__ void __launch_bounds__(kBlock) k_obs_final(Dev d, int nbins, int nblk, double* out) {
  __shared__ double part[kObsRows][kObsCols];
  if (d.flags->status) return;
  const int col = threadIdx.x % kObsCols, row = threadIdx.x / kObsCols;
  const int k = (int)blockIdx.x * kObsCols + col;
  double t = 0.0;
  if (k < 3 * nbins + 4)
    for (int b = row; b < nblk; b += kObsRows) t += d.obs_part[(size_t)b * kObsStride + k];
  part[row][col] = t;
  __syncthreads();
  if (row != 0 || k >= 3 * nbins + 4) return;
  for (int r = 1; r < kObsRows; ++r) t += part[r][col];
  if (k == 3 * nbins) t = t / (3.0 * (double)d.n - 3.0);
  else if (k > 3 * nbins) t = t / (double)d.n;
  out[k] = t;
}

// Unwrapped y, z of every particle (slot order in, tag order out).
__global__ void __launch_bounds__(kBlock) k_unwrapped(Dev d, double* __restrict__ out) {
  if (d.flags->status) return;
  const Ctrl* c = d.ctrl;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= d.n) return;
  const double4 p = reinterpret_cast<const double4*>(d.pos[c->pos_cur])[i];
  int ky, kz;
  img_get(p.w, ky, kz);
  const int t = d.tag[c->aux_cur][i];
  out[t] = p.y + (double)ky * d.Ly;
  out[d.n + t] = p.z + (double)kz * d.Lz;
}

// Mean squared y, z displacement against ref (tag order): block partials in
// obs_part, then one block sums them in block order.
__global__ void __launch_bounds__(kBlock) k_msd_partial(Dev d, const double* __restrict__ ref) {
  __shared__ double red[kBlock / 64][2];
  if (d.flags->status) return;
  const Ctrl* c = d.ctrl;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  double v[2] = {0.0, 0.0};
  if (i < d.n) {
    const double4 p = reinterpret_cast<const double4*>(d.pos[c->pos_cur])[i];
    int ky, kz;
    img_get(p.w, ky, kz);
    const int t = d.tag[c->aux_cur][i];
    const double dy = (p.y + (double)ky * d.Ly) - ref[t];
    const double dz = (p.z + (double)kz * d.Lz) - ref[d.n + t];
    v[0] = dy * dy;
    v[1] = dz * dz;
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int k = 0; k < 2; ++k) {
    double t = v[k];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) red[wid][k] = t;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += red[w][threadIdx.x];
    d.obs_part[(size_t)blockIdx.x * kObsStride + threadIdx.x] = t;
  }
}

__global__ void __launch_bounds__(kBlock) k_msd_final(Dev d, int nblk, double* out2) {
  __shared__ double red[kBlock / 64][2];
  if (d.flags->status) return;
  double v[2] = {0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += kBlock) {
    v[0] += d.obs_part[(size_t)b * kObsStride];
    v[1] += d.obs_part[(size_t)b * kObsStride + 1];
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int k = 0; k < 2; ++k) {
    double t = v[k];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if (lane == 0) red[wid][k] = t;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += red[w][threadIdx.x];
    out2[threadIdx.x] = t / (double)d.n;
  }
}

// ----------------------------------------------------------- state out
__global__ void k_state_out(Dev d, double* x, double* u, int32_t* cell_of, int32_t* order) {
  if (d.flags->status) return;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const Ctrl* c = d.ctrl;
  const int np = d.np, n = d.n;
  const int ac = c->aux_cur;
  int t = d.tag[ac][i];
  double4 p = reinterpret_cast<const double4*>(d.pos[c->pos_cur])[i];
  if (x) { x[t] = p.x; x[n + t] = p.y; x[2 * n + t] = p.z; }
  if (u) for (int a = 0; a < 3; ++a) u[a * n + t] = d.vel[ac][a * np + i];
  if (cell_of) {
    int ix = cell_index(p.x, d.inv_lx, d.nx);
    int iy = cell_index(p.y, d.inv_ly, d.ny);
    int iz = cell_index(p.z, d.inv_lz, d.nz);
    cell_of[t] = (iz * d.ny + iy) * d.nx + ix;
  }
  if (order) {
    // slots follow the beam order; the reported order is by (cell id, tag): the
    // first slot of the particle's cell in id order (in cell_count, see
    // k_id_start) plus its rank within the cell
    const int ix = cell_index(p.x, d.inv_lx, d.nx);
    const int iy = cell_index(p.y, d.inv_ly, d.ny);
    const int iz = cell_index(p.z, d.inv_lz, d.nz);
    order[d.cell_count[(iz * d.ny + iy) * d.nx + ix] + (i - d.cell_start[cell_slot(d, ix, iy, iz)])] = t;
  }
}

// First slot of every cell with the cells in the order of their ids, into
// cell_count (cleared again by k_clear_counts once the order is written); only
// le_build_cells with an order asks for it.  A block takes kIdCells cells: their
// counts and sum first (sums in scan_status, whose words the sort no longer needs: it
// has at least one per 256 cells), then each block adds the sums before its own and
// scans.  (One block over all cells took 1.4 ms for 1.2 million.)
constexpr int kIdCells = 1024;

__device__ __forceinline__ long long wave_sum_ll(long long v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ void __launch_bounds__(kIdCells) k_id_sums(Dev d) {
  __shared__ int ws[kIdCells / 64];
  if (d.flags->status) return;
  const int c = (int)blockIdx.x * kIdCells + (int)threadIdx.x;
  int v = 0;
  if (c < d.ncell) {
    const int k = cell_slot(d, c % d.nx, c / d.nx % d.ny, c / d.nx / d.ny);
    v = d.cell_start[k + 1] - d.cell_start[k];
    d.cell_count[c] = v;
  }
  const int t = (int)wave_sum_ll(v);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    int sum = 0;
    for (int w = 0; w < kIdCells / 64; ++w) sum += ws[w];
    d.scan_status[blockIdx.x] = (unsigned long long)sum;
  }
}

__global__ void __launch_bounds__(kIdCells) k_id_start(Dev d) {
  __shared__ int ws[kIdCells / 64];
  __shared__ long long before[kIdCells / 64];
  if (d.flags->status) return;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  long long mine = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += kIdCells) mine += (long long)d.scan_status[b];
  mine = wave_sum_ll(mine);
  const int c = (int)blockIdx.x * kIdCells + (int)threadIdx.x;
  const int v = c < d.ncell ? d.cell_count[c] : 0;
  int incl = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) ws[wid] = incl;
  if (lane == 0) before[wid] = mine;
  __syncthreads();
  int off = incl - v;
  for (int w = 0; w < kIdCells / 64; ++w) off += (int)before[w] + (w < wid ? ws[w] : 0);
  if (c < d.ncell) d.cell_count[c] = off;
}

__global__ void __launch_bounds__(kBlock) k_clear_counts(Dev d) {
  if (d.flags->status) return;
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c < d.ncell) d.cell_count[c] = 0;
}

__global__ void k_pairs_out(Dev d, int64_t* pairs, int64_t cap, unsigned long long* counter) {
  if (d.flags->status) return;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const int32_t* tag = d.tag[d.ctrl->aux_cur];
  const uint32_t* hs = d.halo + (size_t)(i / d.tile) * d.halo_cap;
  const int ti = tag[i];
  const int npl = d.n_plain[i], nog = d.n_og[i];
  for (int k = 0; k < npl + nog; ++k) {
    int slot;
    if (k < npl && d.staged) {
      const int h = reinterpret_cast<const uint16_t*>(d.nl + unit_front(d, k >> 3, i))[k & 7];
      if (h == d.halo_cap) continue;
      slot = (int)(hs[h] & kSlotMask);
    } else {
      const int m = k < npl ? k : k - npl;
      const size_t u = k < npl ? unit_front(d, m >> 2, i) : unit_back(d, m >> 2, i);
      slot = (int)(reinterpret_cast<const uint32_t*>(d.nl + u)[m & 3] & kSlotMask);
      if (slot == d.n) continue;
    }
    int tj = tag[slot];
    if (ti < tj) {
      unsigned long long idx = atomicAdd(counter, 1ull);
      if ((int64_t)idx < cap) { pairs[2 * idx] = ti; pairs[2 * idx + 1] = tj; }
    }
  }
}

// Copy the latched status word to a caller's device int32 (stream-ordered).
__global__ void k_status_out(const Flags* __restrict__ f, int32_t* __restrict__ out) {
  if (threadIdx.x == 0) *out = f->status;
}

// ------------------------------------------------------------- test hooks
__global__ void k_offsets(double sv, double Lx, double dt, int64_t step0, int64_t count, double* out) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < count) out[k] = le_offset(step0 + k, dt, sv, Lx);
}

__global__ void k_philox(const uint32_t* ctr, const uint32_t* key, uint32_t* out, int64_t count) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  uint32_t c[4] = {ctr[4 * k], ctr[4 * k + 1], ctr[4 * k + 2], ctr[4 * k + 3]};
  philox(c, key[2 * k], key[2 * k + 1]);
  for (int a = 0; a < 4; ++a) out[4 * k + a] = c[a];
}

// ---------------------------------------------------------------- launchers
static inline int blocks_for(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

hipError_t launch_load_state(const Dev& d, hipStream_t s, const double* x0, const double* u0,
                             const double* f0, int64_t step0, double Delta0) {
  int nb = blocks_for(d.n > d.ncell ? d.n : d.ncell);
  hipLaunchKernelGGL(k_load_state, dim3(nb), dim3(kBlock), 0, s, d, x0, u0, f0, step0, Delta0);
  return hipGetLastError();
}

// Calls f with the tile configuration of the halo layout.
template <typename F>
static void with_halo_tiles(const Dev& d, F f) {
  if (d.tiles == kTilesSparse) f(TileSparse{});
  else f(TileDense{});
}
// The same for the list search of either layout, with whether its lists hold
// global slots.
template <typename F>
static void with_search_tiles(const Dev& d, F f) {
  if (d.staged) with_halo_tiles(d, [&](auto t) { f(t, std::false_type{}); });
  else if (d.tiles == kTilesSparse) f(TileSparse{}, std::true_type{});
  else f(TileDenseGlobal{}, std::true_type{});
}

hipError_t launch_rebuild(const Dev& d, Ctrl* next, unsigned long long* next_vmax, hipStream_t s,
                          bool force, bool control) {
  // kernels after the first see the control copy it writes
  Dev dn = d;
  dn.ctrl = next;
  dn.vmax = next_vmax;
  const int nbb = (d.n + kBinBlock - 1) / kBinBlock;
  // Launches within a step: one up to kOneLaunch particles, two up to kSortOneLaunch,
  // three above.  Fewer save 2.2 us each in a step that rebuilds nothing and cost the
  // hand-over in one that does, so the lines move with the life of the lists.  In us a
  // step (one, two, three launches), lists that live for 10 to 14 steps: 17,389 LJ particles 17.0,
  // 19.7, 22.6; 24,000 17.7, 19.3, 22.6; 40,000 22.8, 23.3, 25.6; 64,000 27.2, 24.0, 26.5; 80,000
  // 31.9, 29.9, 30.4; 100,000 38.6, 35.0, 34.7; beads 30,000 15.2, 17.2, 20.4; 50,000 19.5, 18.8, 21.1;
  // 130,000 29.5, 24.1, 24.6; 200,000 40.1, 34.5, 31.9.  Lists that live for 4: 30,000 24.5, 23.3, 25.9;
  // 64,000 39.2, 30.1, 30.2; 80,000 45.6, 38.9, 37.0.  A forced rebuild has work for all (27,000
  // particles: 74 us with three, 78 with two), and so has a batch, where some member
  // rebuilds on most steps (64 of them: 563 and 600 us).
  // Nearly empty cells make many blocks of the scan, which the search's blocks
  // dwarf and every step launches, so the blocks are limited too: a gas of 1000 with
  // 333 blocks takes 11.9, 14.4 and 17.6 us, with 616 14.0, 15.3 and 17.9 (and 14.2 and, with
  // three, 13.3 where an empty launch costs 1.3 us), with 4,819 38.3, 25.6 and 19.9;
  // 10,000 with 681 17.1, 16.9 and 18.7; 60,000 with 700 blocks of the sort 21.5 with two
  // and with three.
  const bool few_sort = nbb + d.sp_blocks <= kWaitBlocks, few = nbb + d.sp_blocks + d.ntiles <= kWaitBlocks;
  if (!force && d.n <= kOneLaunch && few) {
    with_search_tiles(d, [&](auto t, auto gl) {
      using TC = decltype(t);
      hipLaunchKernelGGL((k_rebuild<TC, decltype(gl)::value>), dim3(nbb + d.sp_blocks + d.ntiles),
                         dim3(kSearchThreads), 0, s, d, next, next_vmax, control ? 1 : 0);
    });
    return hipGetLastError();
  }
  if (!force && d.n <= kSortOneLaunch && few_sort) {
    hipLaunchKernelGGL(k_sort, dim3(nbb + d.sp_blocks), dim3(kBlock), 0, s, d, next, next_vmax, control ? 1 : 0);
  } else {
    hipLaunchKernelGGL(k_control_bin, dim3(nbb), dim3(kBlock), 0, s, d, next, next_vmax, force ? 1 : 0,
                       control ? 1 : 0);
    hipLaunchKernelGGL(k_scan_permute, dim3(d.sp_blocks), dim3(kBlock), 0, s, dn);
  }
  with_search_tiles(d, [&](auto t, auto gl) {
    using TC = decltype(t);
    hipLaunchKernelGGL((k_neighbors<TC, decltype(gl)::value>), dim3(d.ntiles), dim3(kSearchThreads), 0, s, dn);
  });
  return hipGetLastError();
}
hipError_t launch_kick_drift(const Dev& d, hipStream_t s) {
  hipLaunchKernelGGL(k_kick_drift, dim3(blocks_for(d.n)), dim3(kBlock), 0, s, d);
  return hipGetLastError();
}

// The force launches go through hipExtLaunchKernelGGL so that optional
// events (e0, e1) take the timestamps of the dispatch itself.
template <typename K>
static void launch_k(K k, dim3 g, dim3 b, hipStream_t s, hipEvent_t e0, hipEvent_t e1, const Dev& d,
                     double* f_out, double* so) {
  if (e0 || e1) hipExtLaunchKernelGGL(k, g, b, 0, s, e0, e1, 0, d, f_out, so);
  else hipLaunchKernelGGL(k, g, b, 0, s, d, f_out, so);
}
template <int MODE, bool SAMPLE, class TC>
static void launch_force_s(const Dev& d, hipStream_t s, double* f_out, double* so, hipEvent_t e0,
                           hipEvent_t e1) {
  constexpr bool STAGED = TC::HALO > 0;
  dim3 g(d.nblocks), b(TC::kForceThreads);
  const bool bonds = d.chain_len > 0;
  const bool mixed = d.precision == LE_MIXED;
  if constexpr (!STAGED && MODE != kDpdForce) {
    if (d.force_cap > 0.0) {  // the host guarantees FP64 and the global layout
      if (bonds) launch_k(k_force<MODE, false, true, SAMPLE, TileNone, true>, g, b, s, e0, e1, d, f_out, so);
      else launch_k(k_force<MODE, false, false, SAMPLE, TileNone, true>, g, b, s, e0, e1, d, f_out, so);
      return;
    }
  }
  if (mixed) {
    if (bonds) launch_k(k_force<MODE, true, true, SAMPLE, TC>, g, b, s, e0, e1, d, f_out, so);
    else launch_k(k_force<MODE, true, false, SAMPLE, TC>, g, b, s, e0, e1, d, f_out, so);
  } else {
    if (bonds) launch_k(k_force<MODE, false, true, SAMPLE, TC>, g, b, s, e0, e1, d, f_out, so);
    else launch_k(k_force<MODE, false, false, SAMPLE, TC>, g, b, s, e0, e1, d, f_out, so);
  }
}
template <int MODE, bool SAMPLE>
static void launch_force_t(const Dev& d, hipStream_t s, double* f_out, double* so, hipEvent_t e0,
                           hipEvent_t e1) {
  if (!d.staged) launch_force_s<MODE, SAMPLE, TileNone>(d, s, f_out, so, e0, e1);
  else with_halo_tiles(d, [&](auto t) { launch_force_s<MODE, SAMPLE, decltype(t)>(d, s, f_out, so, e0, e1); });
}

hipError_t launch_force(const Dev& d, hipStream_t s, ForceMode mode, bool sample, double* f_out,
                        double* sample_out, hipEvent_t e0, hipEvent_t e1) {
  switch (mode) {
    case kForcesOnly: launch_force_t<kForcesOnly, false>(d, s, f_out, nullptr, e0, e1); break;
    case kInitForce: launch_force_t<kInitForce, false>(d, s, f_out, nullptr, e0, e1); break;
    case kStepLast:
      if (sample) launch_force_t<kStepLast, true>(d, s, f_out, sample_out, e0, e1);
      else launch_force_t<kStepLast, false>(d, s, f_out, nullptr, e0, e1);
      break;
    case kStepFused:
      if (sample) launch_force_t<kStepFused, true>(d, s, f_out, sample_out, e0, e1);
      else launch_force_t<kStepFused, false>(d, s, f_out, nullptr, e0, e1);
      break;
    case kDpdForce:
      if (!d.vt) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_pack_vt, dim3(blocks_for(d.n)), dim3(kBlock), 0, s, d);
      if (sample) launch_force_t<kDpdForce, true>(d, s, f_out, sample_out, e0, e1);
      else launch_force_t<kDpdForce, false>(d, s, f_out, nullptr, e0, e1);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_integrate(const Dev& d, hipStream_t s, bool last, bool sample) {
  dim3 g(d.nblocks), b(kTile);
  if (last) {
    if (sample) hipLaunchKernelGGL((k_integrate<true, true>), g, b, 0, s, d);
    else hipLaunchKernelGGL((k_integrate<true, false>), g, b, 0, s, d);
  } else {
    if (sample) hipLaunchKernelGGL((k_integrate<false, true>), g, b, 0, s, d);
    else hipLaunchKernelGGL((k_integrate<false, false>), g, b, 0, s, d);
  }
  return hipGetLastError();
}

hipError_t launch_stress_final(const Dev& d, hipStream_t s, double* out6, bool virial_only) {
  hipLaunchKernelGGL(k_stress_final, dim3(1), dim3(kBlock), 0, s, d, out6, virial_only ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_ctrl_copy(const Ctrl* src, Ctrl* dst, const unsigned long long* vsrc,
                            unsigned long long* vdst, hipStream_t s) {
  hipLaunchKernelGGL(k_ctrl_copy, dim3(1), dim3(64), 0, s, src, dst, vsrc, vdst);
  return hipGetLastError();
}
hipError_t launch_observables(const Dev& d, hipStream_t s, int nbins, double* out) {
  const int nblk = obs_blocks(d.n), ncol = 3 * nbins + 4;
  hipLaunchKernelGGL(k_obs_partial, dim3(nblk), dim3(kBlock), 0, s, d, nbins, nblk);
  hipLaunchKernelGGL(k_obs_final, dim3((ncol + kObsCols - 1) / kObsCols), dim3(kBlock), 0, s, d, nbins, nblk,
                     out);
  return hipGetLastError();
}
hipError_t launch_unwrapped(const Dev& d, hipStream_t s, double* out) {
  hipLaunchKernelGGL(k_unwrapped, dim3(blocks_for(d.n)), dim3(kBlock), 0, s, d, out);
  return hipGetLastError();
}
hipError_t launch_msd(const Dev& d, hipStream_t s, const double* ref, double* out2) {
  const int nblk = blocks_for(d.n);
  hipLaunchKernelGGL(k_msd_partial, dim3(nblk), dim3(kBlock), 0, s, d, ref);
  hipLaunchKernelGGL(k_msd_final, dim3(1), dim3(kBlock), 0, s, d, nblk, out2);
  return hipGetLastError();
}
hipError_t launch_state_out(const Dev& d, hipStream_t s, double* x, double* u, int32_t* cell_of,
                            int32_t* order) {
  if (order) {
    const dim3 nb((unsigned)((d.ncell + kIdCells - 1) / kIdCells));
    hipLaunchKernelGGL(k_id_sums, nb, dim3(kIdCells), 0, s, d);
    hipLaunchKernelGGL(k_id_start, nb, dim3(kIdCells), 0, s, d);
  }
  hipLaunchKernelGGL(k_state_out, dim3(blocks_for(d.n)), dim3(kBlock), 0, s, d, x, u, cell_of, order);
  if (order) hipLaunchKernelGGL(k_clear_counts, dim3(blocks_for(d.ncell)), dim3(kBlock), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_pairs_out(const Dev& d, hipStream_t s, int64_t* pairs, int64_t cap,
                            unsigned long long* counter) {
  hipLaunchKernelGGL(k_pairs_out, dim3(blocks_for(d.n)), dim3(kBlock), 0, s, d, pairs, cap, counter);
  return hipGetLastError();
}

// ------------------------------------------------------- batched launchers
__global__ void k_store_dev(Dev a, Dev b, Dev* dst) {
  if (threadIdx.x == 0) {
    dst[0] = a;
    dst[1] = b;
  }
}

hipError_t launch_store_dev(const Dev& a, const Dev& b, Dev* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_store_dev, dim3(1), dim3(64), 0, s, a, b, dst);
  return hipGetLastError();
}

static inline dim3 grid_of(const Batch& b) { return dim3((unsigned)b.start[b.nsims]); }

hipError_t launch_kick_drift_b(const Batch& par_cur, hipStream_t s) {
  hipLaunchKernelGGL(k_kick_drift_b, grid_of(par_cur), dim3(kBlock), 0, s, par_cur);
  return hipGetLastError();
}

hipError_t launch_sort_b(const Batch& bin_cur, const Batch& scan_nxt, hipStream_t s) {
  hipLaunchKernelGGL(k_control_bin_b, grid_of(bin_cur), dim3(kBlock), 0, s, bin_cur);
  hipLaunchKernelGGL(k_scan_permute_b, grid_of(scan_nxt), dim3(kBlock), 0, s, scan_nxt);
  return hipGetLastError();
}

hipError_t launch_search_b(const Batch& tile_nxt, const Dev& cfg, hipStream_t s) {
  with_search_tiles(cfg, [&](auto t, auto gl) {
    using TC = decltype(t);
    hipLaunchKernelGGL((k_neighbors_b<TC, decltype(gl)::value>), grid_of(tile_nxt), dim3(kSearchThreads), 0, s,
                       tile_nxt);
  });
  return hipGetLastError();
}

template <int MODE, bool SAMPLE, class TC>
static void launch_force_bs(const Batch& b, const Dev& cfg, hipStream_t s) {
  constexpr bool STAGED = TC::HALO > 0;
  const dim3 g = grid_of(b), blk(TC::kForceThreads);
  const bool bonds = cfg.chain_len > 0;
  if constexpr (!STAGED && MODE != kDpdForce) {
    if (cfg.force_cap > 0.0) {
      if (bonds) hipLaunchKernelGGL((k_force_b<MODE, false, true, SAMPLE, TileNone, true>), g, blk, 0, s, b);
      else hipLaunchKernelGGL((k_force_b<MODE, false, false, SAMPLE, TileNone, true>), g, blk, 0, s, b);
      return;
    }
  }
  if (cfg.precision == LE_MIXED) {
    if (bonds) hipLaunchKernelGGL((k_force_b<MODE, true, true, SAMPLE, TC>), g, blk, 0, s, b);
    else hipLaunchKernelGGL((k_force_b<MODE, true, false, SAMPLE, TC>), g, blk, 0, s, b);
  } else {
    if (bonds) hipLaunchKernelGGL((k_force_b<MODE, false, true, SAMPLE, TC>), g, blk, 0, s, b);
    else hipLaunchKernelGGL((k_force_b<MODE, false, false, SAMPLE, TC>), g, blk, 0, s, b);
  }
}

template <int MODE, bool SAMPLE>
static void launch_force_bt(const Batch& b, const Dev& cfg, hipStream_t s) {
  if (!cfg.staged) launch_force_bs<MODE, SAMPLE, TileNone>(b, cfg, s);
  else with_halo_tiles(cfg, [&](auto t) { launch_force_bs<MODE, SAMPLE, decltype(t)>(b, cfg, s); });
}

hipError_t launch_force_b(const Batch& blk_cur, const Batch& par_cur, const Dev& cfg, hipStream_t s,
                          ForceMode mode, bool sample) {
  switch (mode) {
    case kStepLast:
      if (sample) launch_force_bt<kStepLast, true>(blk_cur, cfg, s);
      else launch_force_bt<kStepLast, false>(blk_cur, cfg, s);
      break;
    case kStepFused:
      if (sample) launch_force_bt<kStepFused, true>(blk_cur, cfg, s);
      else launch_force_bt<kStepFused, false>(blk_cur, cfg, s);
      break;
    case kDpdForce:
      if (!cfg.vt) return hipErrorInvalidValue;
      hipLaunchKernelGGL(k_pack_vt_b, grid_of(par_cur), dim3(kBlock), 0, s, par_cur);
      if (sample) launch_force_bt<kDpdForce, true>(blk_cur, cfg, s);
      else launch_force_bt<kDpdForce, false>(blk_cur, cfg, s);
      break;
    default:
      return hipErrorInvalidValue;  // the other modes are not batched
  }
  return hipGetLastError();
}

hipError_t launch_integrate_b(const Batch& blk_cur, hipStream_t s, bool last, bool sample) {
  const dim3 g = grid_of(blk_cur), b(kTile);
  if (last) {
    if (sample) hipLaunchKernelGGL((k_integrate_b<true, true>), g, b, 0, s, blk_cur);
    else hipLaunchKernelGGL((k_integrate_b<true, false>), g, b, 0, s, blk_cur);
  } else {
    if (sample) hipLaunchKernelGGL((k_integrate_b<false, true>), g, b, 0, s, blk_cur);
    else hipLaunchKernelGGL((k_integrate_b<false, false>), g, b, 0, s, blk_cur);
  }
  return hipGetLastError();
}

hipError_t launch_stress_final_b(const Batch& one_cur, const BatchOut& out, hipStream_t s) {
  hipLaunchKernelGGL(k_stress_final_b, dim3((unsigned)one_cur.nsims), dim3(kBlock), 0, s, one_cur, out);
  return hipGetLastError();
}

hipError_t launch_status_out(const Dev& d, hipStream_t s, int32_t* out) {
  hipLaunchKernelGGL(k_status_out, dim3(1), dim3(64), 0, s, d.flags, out);
  return hipGetLastError();
}

hipError_t launch_offsets(double sr, double Lx, double Ly, double dt, int64_t step0, int64_t count,
                          double* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_offsets, dim3(blocks_for(count)), dim3(kBlock), 0, s, sr * Ly, Lx, dt, step0,
                     count, out);
  return hipGetLastError();
}

hipError_t launch_philox(const uint32_t* ctr, const uint32_t* key, uint32_t* out, int64_t count,
                         hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_philox, dim3(blocks_for(count)), dim3(kBlock), 0, s, ctr, key, out, count);
  return hipGetLastError();
}

}  // namespace le
