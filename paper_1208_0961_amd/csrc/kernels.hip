// kernels.hip -- gfx950 kernels of the PIC Boltzmann step (arXiv:1208.0961).
//
// State layout: two buffers with a fixed capacity of `cap` slots per cell;
// a slot is a 48-byte record (px py pz x y z) and an id in an array of its
// own; cell c owns slots [c cap, c cap + count[c]).  One
// buffer holds the current state, the other receives the next binning.
//
// A step t is stream + reflect + bin (Eq. (2), walls, cells), then the
// collisions of every cell (Eq. (3), claims, CM kinematics).  The kernels:
//   k_stream_bin   one wave per source cell: stream + reflect each particle,
//                  find its new cell, append it there (wave-aggregated slot
//                  atomics, one round trip per wave).       HBM: 52 B + 52 B
//   k_step<F>      one wave per cell: ids to LDS, canonical (id) order by
//                  rank counting, all n(n-1)/2 pair tests over the lanes with
//                  a Philox block each, ballot compaction of the pairs that
//                  can pass, exact Eq. (3) test on those, greedy claim in
//                  pair order, CM kinematics (written back in place, or
//                  with F kept in LDS).  With F (fused) the same wave then
//                  streams and bins its particles for step t+1, so the
//                  binning traffic overlaps the ALU-bound pair tests.
//   k_step_group   a workgroup of four waves on four dense cells: the waves
//                  share the four cells' pair tests.
//   k_step_packed  whole cells packed into waves of up to 64 particles, one
//                  a lane (sparse cells); k_step_large / k_step_over step
//                  larger cells where that kernel does not itself.
//   k_step_wide    a workgroup of 4, 8 or 16 waves per cell (boxes of few
//                  dense cells).
//   observe        per-cell sums of E, p_x, p_x^2/E and counts, then
//                  fixed-order slab sums.
//   gather         state export by id.
// A run of n steps is one stream_bin, n-1 fused steps and one collide-only
// step, which leaves the state binned and collided (positions of step t+n-1).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstddef>
#include <type_traits>

#include "internal.hpp"

namespace cuba {

namespace {

constexpr int kBlock = 256;
constexpr uint32_t kCellsPerBlock = kBlock / 64;

// Waves per SIMD the one-wave-per-cell kernels are held to: six with the
// LDS of 512-slot cells (80 VGPRs; the rare paths for overflowing cells
// would otherwise raise the count for all), four with that of 1024 (the
// LDS allows no more).
template <uint32_t kCap>
constexpr int cell_waves() {
  return kCap <= kSmallCap ? 6 : 4;
}

// Device views of the particle buffers with global-address-space pointers:
// every kernel converts its Cells once at entry, so that all buffer accesses
// compile to global (not flat) memory instructions, also where the pointers
// are loaded from memory (the batch table) rather than passed as arguments.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;

// The particles' records (six doubles: px py pz x y z, 16-byte aligned) and
// ids.
struct GState {
  gptr<double> rec;
  gptr<uint32_t> id;
};

struct GCells {
  GState st;
  gptr<uint32_t> count;
  uint32_t cap;
  SpillDesc *sp;
  uint32_t q;  // the spill counter set of the binning this view holds or receives
};

__device__ __forceinline__ GCells to_global(const Cells &c) {
  GCells g;
  g.st.rec = (gptr<double>)c.st.rec;
  g.st.id = (gptr<uint32_t>)c.st.id;
  g.count = (gptr<uint32_t>)c.count;
  g.cap = c.cap;
  g.sp = c.sp;
  g.q = 0u;
  return g;
}

// The view of a buffer holding (or receiving) the binning of step b.
__device__ __forceinline__ GCells binning(GCells c, uint32_t b) {
  c.q = spill_set(b);
  return c;
}

__device__ __forceinline__ uint32_t atomic_add(gptr<uint32_t> p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Slot = old value of ctr[key] + rank of this lane among the active lanes
// of its wave with the same key.  The lanes are grouped by key with ballots
// first (ALU only); then every group leader issues its atomic in the same
// instruction, so the wave waits for one atomic round trip, not one per key.
__device__ __forceinline__ uint32_t aggregated_fetch_add(gptr<uint32_t> ctr, uint32_t key,
                                                         bool active) {
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t leader = lane, rank = 0, size = 0;
  uint64_t todo = __ballot(active);
  while (todo != 0) {
    const int l = __builtin_ctzll(todo);
    const uint32_t lkey = (uint32_t)__builtin_amdgcn_readlane((int)key, l);
    const uint64_t group = __ballot(active && key == lkey);
    if (active && key == lkey) {
      leader = (uint32_t)l;
      rank = (uint32_t)__popcll(group & below);
      size = (uint32_t)__popcll(group);
    }
    todo &= ~group;
  }
  uint32_t base = 0;
  if (active && leader == lane) base = atomic_add(ctr + key, size);
  base = __shfl(base, (int)leader);
  return base + rank;
}

// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X
// (workgroup b runs on XCD b mod 8), each XCD with its own L2.  This
// bijection on [0, nblocks) gives each XCD runs of kRun consecutive logical
// blocks, interleaved over the XCDs: neighbouring cells (which share cache
// lines at their boundaries and exchange particles) stay on one L2, while
// work that varies along the cell range stays balanced.
constexpr uint32_t kXcds = 8;
template <uint32_t kRun>
__device__ __forceinline__ uint32_t xcd_runs(uint32_t b, uint32_t nblocks) {
  constexpr uint32_t kSuper = kXcds * kRun;
  const uint32_t full = nblocks / kSuper * kSuper;
  if (b >= full) return b;
  const uint32_t s = b / kSuper, r = b % kSuper;
  return s * kSuper + (r % kXcds) * kRun + r / kXcds;
}

// One particle in registers.
struct Particle {
  double x, y, z, px, py, pz;
  uint32_t id;
};

// A record is 48 contiguous bytes, moved as three 16-byte accesses: a
// scattered particle touches one or two cache lines instead of one in each
// of six arrays, and so does a cell of a few particles.  Against six arrays
// of doubles: the 32^3 fm^3 set's step 1.92 -> 1.49 ms, its stream-bin 1.95
// -> 1.15 ms and its initial binning 5.88 -> 2.00 ms; 0.33 M particles in
// 160 000 cells 49 -> 35 us a step; cells of ~100 particles 2-3 % (their
// contiguous accesses were whole lines before, their movers' were not).
// Two waves per cell at ~400 particles a cell lost 1.5 %.
typedef double Double2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ gptr<Double2> record(const GState &st, size_t o) {
  return (gptr<Double2>)(st.rec + 6u * o);
}

__device__ __forceinline__ Particle load_particle(const GState &st, size_t o) {
  const gptr<Double2> r = record(st, o);
  const Double2 a = r[0], b = r[1], c = r[2];
  return Particle{b.y, c.x, c.y, a.x, a.y, b.x, st.id[o]};
}

__device__ __forceinline__ void put_particle(const GState &st, size_t o, const Particle &q) {
  const gptr<Double2> r = record(st, o);
  r[0] = Double2{q.px, q.py};
  r[1] = Double2{q.pz, q.x};
  r[2] = Double2{q.y, q.z};
  st.id[o] = q.id;
}

__device__ __forceinline__ void load_momentum(const GState &st, size_t o, double &px, double &py,
                                              double &pz) {
  const Double2 a = record(st, o)[0];
  px = a.x;
  py = a.y;
  pz = st.rec[6u * o + 2u];
}

__device__ __forceinline__ void put_momentum(const GState &st, size_t o, double px, double py,
                                             double pz) {
  record(st, o)[0] = Double2{px, py};
  st.rec[6u * o + 2u] = pz;
}

// A particle that took slot `slot` >= cap of cell c2 goes to a spill slot
// of dst, tagged with its cell; the one particle that takes slot cap lists
// the cell among the overflowing ones.  The spill slots hold every particle
// of the context, so the index check only guards against an internal error.
__device__ __forceinline__ void spill_particle(const GCells &dst, uint32_t c2, uint32_t slot,
                                               const Particle &q, DevStatus *status) {
  SpillDesc *const sp = dst.sp;
  uint32_t *const h = sp->hdr + 2u * dst.q;
  const uint32_t i = atomicAdd(&h[0], 1u);
  if (i < sp->capacity) {
    put_particle(dst.st, sp->base + i, q);
    sp->cell[i] = c2;
  } else {
    atomicOr(&status->err, kErrSpill);
  }
  if (slot == dst.cap) sp->ocell[atomicAdd(&h[1], 1u)] = c2;
}

// Stores a particle at slot `slot` of cell c2 of dst: in the cell's block,
// or past its capacity in the spill region.
__device__ __forceinline__ void store_particle(const GCells &dst, uint32_t c2, uint32_t slot,
                                               const Particle &q, DevStatus *status) {
  if (slot < dst.cap)
    put_particle(dst.st, (size_t)c2 * dst.cap + slot, q);
  else
    spill_particle(dst, c2, slot, q, status);
}

// Appends a particle to cell c2 of dst (a slot by the wave-aggregated
// counter atomic).
__device__ __forceinline__ void append(const GCells &dst, uint32_t c2, bool active,
                                       const Particle &q, DevStatus *status) {
  const uint32_t slot = aggregated_fetch_add(dst.count, c2, active);
  if (active) store_particle(dst, c2, slot, q, status);
}

// Orders the calling wave's LDS accesses before and after this point for
// its own lanes (LDS executes one wave's operations in order; the fence
// keeps the compiler from moving accesses across and waits for them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// A wave's own table of the cells its particles go to: kSlotTable entries
// by a hash of the cell, and kSlotTable2 for the cells whose entry another
// cell holds.
constexpr uint32_t kSlotTable = 256, kSlotTable2 = 64;
struct SlotTable {
  uint32_t cell[kSlotTable + kSlotTable2];  // the entry's cell, then its first slot
  uint32_t cnt[kSlotTable + kSlotTable2];   // zero between calls
};

__device__ __forceinline__ void clear_slot_table(SlotTable &tab) {
  for (uint32_t i = lane_id(); i < kSlotTable + kSlotTable2; i += 64u) tab.cnt[i] = 0u;
}

// As aggregated_fetch_add for waves whose particles go to many cells (the
// kernels that step several cells a wave, where 64 particles take ~40
// distinct ones): the lanes write their cell to its entry and those that
// read it back share the entry; LDS atomics number its lanes, whose first
// adds their count to the cell's counter.  A lane that shares no entry adds
// 1 by itself.  Some ten LDS accesses, where the loop over distinct cells
// takes ~8 VALU instructions a cell: 0.33 M particles in 160 000 cells 2.15
// -> 1.94 ms for 50 steps, 2 M there 9.5 -> 9.3 ms, the 32^3 fm^3 set (10
// steps) 25.7 -> 25.4 ms.  (An atomic a particle instead of one a cell and
// wave: the 32^3 fm^3 set 33.3 ms, the atomics' own rate bounding it.)
__device__ __forceinline__ uint32_t table_fetch_add(gptr<uint32_t> ctr, uint32_t key,
                                                    bool active, SlotTable &tab) {
  const uint32_t hash = key * 0x9E3779B1u;
  uint32_t h = hash >> 24;
  static_assert(kSlotTable == 256 && kSlotTable2 == 64, "hash bits");
  if (active) tab.cell[h] = key;
  wave_lds_sync();
  bool own = active && tab.cell[h] == key;
  if (__ballot(active && !own) != 0ull) {
    if (active && !own) {
      h = kSlotTable + ((hash >> 18) & (kSlotTable2 - 1u));
      tab.cell[h] = key;
    }
    wave_lds_sync();
    own = active && tab.cell[h] == key;
  }
  uint32_t rank = 0;
  if (own) rank = atomicAdd(&tab.cnt[h], 1u);
  wave_lds_sync();
  uint32_t base = 0;
  if (active && rank == 0u) {
    base = atomic_add(ctr + key, own ? tab.cnt[h] : 1u);
    if (own) {
      tab.cell[h] = base;
      tab.cnt[h] = 0u;
    }
  }
  wave_lds_sync();
  if (own) base = tab.cell[h] + rank;
  wave_lds_sync();
  return base;
}

// append through the wave's slot table.
__device__ __forceinline__ void append_table(const GCells &dst, uint32_t c2, bool active,
                                             const Particle &q, DevStatus *status,
                                             SlotTable &tab) {
  const uint32_t slot = table_fetch_add(dst.count, c2, active, tab);
  if (active) store_particle(dst, c2, slot, q, status);
}

// The buffer laid out like c, `shift` bytes away.
template <typename T>
__device__ __forceinline__ gptr<T> shift_ptr(gptr<T> p, int64_t shift) {
  return (gptr<T>)((gptr<char>)p + shift);
}

// The destination of a collision launch of step t: src shifted by the
// distance between the two buffers, receiving the binning of step t + 1.
__device__ __forceinline__ GCells shifted(const GCells &c, int64_t shift);
__device__ __forceinline__ GCells dst_of(const GCells &src, int64_t shift, uint32_t t);

__device__ __forceinline__ GCells shifted(const GCells &c, int64_t shift) {
  GCells d;
  d.st.rec = shift_ptr(c.st.rec, shift);
  d.st.id = shift_ptr(c.st.id, shift);
  d.count = shift_ptr(c.count, shift);
  d.cap = c.cap;
  d.sp = (SpillDesc *)((char *)c.sp + shift);
  d.q = c.q;
  return d;
}

__device__ __forceinline__ GCells dst_of(const GCells &src, int64_t shift, uint32_t t) {
  return binning(shifted(src, shift), t + 1u);
}

// Appends two particles per lane (a and b, up to 128 per wave) to cells ca
// and cb of dst: the 128 keys are grouped by ballots (ALU only), the group's
// leader (its lowest lane, among the a particles first) adds the group size
// to the cell's count, and all leaders' atomics are in flight together, so
// the wave waits for one round trip for both halves.  A lane may lead one
// group through its a particle and one through its b particle.
__device__ __forceinline__ void append_two(const GCells &dst, uint32_t ca, bool act_a,
                                           const Particle &qa, uint32_t cb, bool act_b,
                                           const Particle &qb, DevStatus *status) {
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t lead_a = lane, lead_b = lane, sel_a = 0, sel_b = 0, rank_a = 0, rank_b = 0;
  uint32_t size_via_a = 0, size_via_b = 0;
  uint64_t todo_a = __ballot(act_a), todo_b = __ballot(act_b);
  while ((todo_a | todo_b) != 0) {
    const bool from_a = todo_a != 0;
    const int l = __builtin_ctzll(from_a ? todo_a : todo_b);
    const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)(from_a ? ca : cb), l);
    const bool in_a = act_a && ca == key, in_b = act_b && cb == key;
    const uint64_t ma = __ballot(in_a), mb = __ballot(in_b);
    const uint32_t na = (uint32_t)__popcll(ma);
    if (in_a) {
      lead_a = (uint32_t)l;
      sel_a = from_a ? 0u : 1u;
      rank_a = (uint32_t)__popcll(ma & below);
    }
    if (in_b) {
      lead_b = (uint32_t)l;
      sel_b = from_a ? 0u : 1u;
      rank_b = na + (uint32_t)__popcll(mb & below);
    }
    if (lane == (uint32_t)l) {
      if (from_a) size_via_a = na + (uint32_t)__popcll(mb);
      else size_via_b = (uint32_t)__popcll(mb);
    }
    todo_a &= ~ma;
    todo_b &= ~mb;
  }
  uint32_t base0 = 0, base1 = 0;
  if (size_via_a != 0) base0 = atomic_add(dst.count + ca, size_via_a);
  if (size_via_b != 0) base1 = atomic_add(dst.count + cb, size_via_b);
  const uint32_t a0 = __shfl(base0, (int)lead_a), a1 = __shfl(base1, (int)lead_a);
  const uint32_t b0 = __shfl(base0, (int)lead_b), b1 = __shfl(base1, (int)lead_b);
  if (act_a) store_particle(dst, ca, (sel_a ? a1 : a0) + rank_a, qa, status);
  if (act_b) store_particle(dst, cb, (sel_b ? b1 : b0) + rank_b, qb, status);
}

// Particles of a cell held in its block (the rest, if any, are spilled).
__device__ __forceinline__ uint32_t occupancy(const GCells &c, uint32_t cell) {
  const uint32_t n = c.count[cell];
  return n < c.cap ? n : c.cap;
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, uint32_t v,
                                                     int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < count) p[i] = v;
}

__global__ __launch_bounds__(64) void k_store_f64(double *p, double v) {
  if (threadIdx.x == 0) *p = v;
}

// Up to kWriteWords words carried as a kernel argument and stored to device
// memory in stream order (the host copy needs to live only until the launch
// returns, and no host-to-device copy waits for the stream).
constexpr uint32_t kWriteWords = 64;
struct WriteWords {
  uint32_t w[kWriteWords];
};
__global__ __launch_bounds__(64) void k_write_words(uint32_t *dst, WriteWords v,
                                                    uint32_t nwords) {
  for (uint32_t i = threadIdx.x; i < nwords; i += 64) dst[i] = v.w[i];
}

// Initial state (id order) -> validated and binned without streaming.
__global__ __launch_bounds__(kBlock) void k_init_bin(
    const double *__restrict__ x, const double *__restrict__ y,
    const double *__restrict__ z, const double *__restrict__ px,
    const double *__restrict__ py, const double *__restrict__ pz, Cells dst_arg,
    int64_t n, Geometry g, DevStatus *status, uint32_t binning_step) {
  const GCells dst = binning(to_global(dst_arg), binning_step);
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool active = i < n;
  double a = 0, b = 0, c = 0, qa = 0, qb = 0, qc = 0;
  uint32_t cell = 0;
  if (active) {
    a = x[i];
    b = y[i];
    c = z[i];
    qa = px[i];
    qb = py[i];
    qc = pz[i];
    const bool ok = __builtin_isfinite(a) && __builtin_isfinite(b) &&
                    __builtin_isfinite(c) && __builtin_isfinite(qa) &&
                    __builtin_isfinite(qb) && __builtin_isfinite(qc) && a >= 0.0 &&
                    a <= g.L[0] && b >= 0.0 && b <= g.L[1] && c >= 0.0 &&
                    c <= g.L[2] && norm3(qa, qb, qc) > 0.0;
    if (!ok) atomicOr(&status->err, kErrRange);
    cell = cell_id(g, a, b, c);
  }
  // slots through the wave's table, whatever the order of the particles.  The
  // whole set-up of 16 M particles, sorted by cell / shuffled: with an atomic a
  // lane 3.1 (a wave's lanes all at one counter) / 1.16 ms, with a loop over
  // the distinct cells 0.53 / 2.35 ms, with the table 0.45 / 1.20 ms
  const Particle q{a, b, c, qa, qb, qc, (uint32_t)i};
  __shared__ SlotTable tab[kBlock / 64];
  clear_slot_table(tab[threadIdx.x / 64]);
  append_table(dst, cell, active, q, status, tab[threadIdx.x / 64]);
}

// Cells holding more than 8, 16, 32, 64 and kFitsSmall particles, added into
// over[5]: a grid stride over the cells, counts kept per wave, summed per
// block in LDS, then an atomic per class and block (one atomic per wave and
// counter serialised on the addresses at 2 M cells).
__global__ __launch_bounds__(kBlock) void k_occupancy_over(Cells cur_arg, uint32_t n_cells,
                                                           uint32_t *over) {
  const GCells cur = to_global(cur_arg);
  __shared__ uint32_t part[kBlock / 64][kOverClasses];
  uint32_t acc[kOverClasses] = {};
  for (uint32_t c0 = blockIdx.x * kBlock; c0 < n_cells; c0 += gridDim.x * kBlock) {
    const uint32_t c = c0 + threadIdx.x;
    const uint32_t n = c < n_cells ? cur.count[c] : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kOverClasses; ++k)
      acc[k] += (uint32_t)__popcll(__ballot(n > (k < 4u ? 8u << k : kFitsSmall)));
  }
  const uint32_t w = threadIdx.x / 64;
  if (lane_id() == 0)
    for (uint32_t k = 0; k < kOverClasses; ++k) part[w][k] = acc[k];
  __syncthreads();
  if (threadIdx.x < kOverClasses) {
    uint32_t sum = 0;
    for (uint32_t i = 0; i < kBlock / 64; ++i) sum += part[i][threadIdx.x];
    if (sum != 0) atomicAdd(&over[threadIdx.x], sum);
  }
}

// Stream + reflect + bin the spilled members of overflowing cell cv of src
// (found by a scan of the spill slots) into dst.  The whole wave.
__device__ __forceinline__ void stream_spilled(const GCells &src, const GCells &dst, uint32_t cv,
                                               const Geometry &g, DevStatus *status,
                                               uint32_t *trace_cell) {
  const SpillDesc *const sp = src.sp;
  const uint32_t ns = min(sp->hdr[2u * src.q], sp->capacity);
  const size_t sbase = sp->base;
  const uint32_t lane = lane_id();
  for (uint32_t i0 = 0; i0 < ns; i0 += 64u) {
    const uint32_t i = i0 + lane;
    const bool hit = i < ns && sp->cell[i] == cv;
    if (__ballot(hit) == 0) continue;
    Particle q{};
    uint32_t c2 = 0;
    if (hit) {
      q = load_particle(src.st, sbase + i);
      advance<true>(g, q.x, q.y, q.z, q.px, q.py, q.pz);
      c2 = cell_id(g, q.x, q.y, q.z);
      if (trace_cell) trace_cell[q.id] = c2;
    }
    append(dst, c2, hit, q, status);
  }
}

// Clears the spill counter set of `c` that no launch uses now: the one of
// the binning two steps after (or before) the one c holds.
__device__ __forceinline__ void clear_idle_spill_set(const GCells &c) {
  uint32_t *const h = c.sp->hdr + 2u * (c.q ^ 1u);
  h[0] = 0u;
  h[1] = 0u;
}

// Stream + reflect + bin the particles of the source cells c0 .. c_end - 1
// (at most 64 / G of them), G lanes per cell; G = 64 is one wave per cell.
// Clears the source counts, so the source buffer can receive the next
// binning.
template <uint32_t G>
__device__ __forceinline__ void cells_stream_bin(const GCells &src, const GCells &dst,
                                                 uint32_t c0, uint32_t c_end,
                                                 const Geometry &g, DevStatus *status,
                                                 uint32_t *trace_cell, SlotTable &tab) {
  const uint32_t lane = lane_id();
  const uint32_t c = c0 + lane / G, gl = lane % G;
  const bool in_range = c < c_end;
  const uint32_t cnt = in_range ? src.count[c] : 0u;
  const uint32_t n = cnt < src.cap ? cnt : src.cap;  // the block part
  const size_t base = (size_t)c * src.cap;
  // then the spilled members of overflowing cells
  const uint64_t ovm = __ballot(in_range && gl == 0 && cnt > src.cap);
  if (ovm != 0) {
    for (uint64_t m = ovm; m != 0; m &= m - 1ull) {
      const uint32_t cv = (uint32_t)__builtin_amdgcn_readlane((int)c, __builtin_ctzll(m));
      stream_spilled(src, dst, cv, g, status, trace_cell);
    }
  }
  if (G == 64) {
    // one cell: 128 particles per round, both halves' atomics in flight together
    for (uint32_t j0 = 0; j0 < n; j0 += 128) {
      const uint32_t ja = j0 + lane, jb = j0 + 64 + lane;
      const bool act_a = ja < n, act_b = jb < n;
      Particle qa{}, qb{};
      if (act_a) qa = load_particle(src.st, base + ja);
      if (act_b) qb = load_particle(src.st, base + jb);
      uint32_t ca = 0, cb = 0;
      if (act_a) {
        advance<true>(g, qa.x, qa.y, qa.z, qa.px, qa.py, qa.pz);
        ca = cell_id(g, qa.x, qa.y, qa.z);
        if (trace_cell) trace_cell[qa.id] = ca;
      }
      if (act_b) {
        advance<true>(g, qb.x, qb.y, qb.z, qb.px, qb.py, qb.pz);
        cb = cell_id(g, qb.x, qb.y, qb.z);
        if (trace_cell) trace_cell[qb.id] = cb;
      }
      append_two(dst, ca, act_a, qa, cb, act_b, qb, status);
    }
    if (in_range && gl == 0) src.count[c] = 0u;
    return;
  }
  clear_slot_table(tab);
  for (uint32_t j0 = 0; __ballot(j0 < n) != 0; j0 += G) {
    const uint32_t j = j0 + gl;
    const bool active = j < n;
    Particle q{};
    uint32_t c2 = 0;
    if (active) {
      q = load_particle(src.st, base + j);
      advance<true>(g, q.x, q.y, q.z, q.px, q.py, q.pz);
      c2 = cell_id(g, q.x, q.y, q.z);
      if (trace_cell) trace_cell[q.id] = c2;
    }
    append_table(dst, c2, active, q, status, tab);
  }
  if (in_range && gl == 0) src.count[c] = 0u;
}

// Four waves per block; each wave takes 64 / G consecutive source cells;
// src holds the binning of step t - 1, dst receives that of step t.
template <uint32_t G>
__global__ __launch_bounds__(kBlock) void k_stream_bin(Cells src_arg, Cells dst_arg,
                                                       uint32_t n_cells, Geometry g,
                                                       DevStatus *status,
                                                       uint32_t *trace_cell, uint32_t t) {
  const GCells src = binning(to_global(src_arg), t - 1u);
  const GCells dst = binning(to_global(dst_arg), t);
  constexpr uint32_t kPer = 64 / G;
  const uint32_t c0 =
      (xcd_runs<2>(blockIdx.x, gridDim.x) * kCellsPerBlock + threadIdx.x / 64) * kPer;
  if (c0 >= n_cells) return;
  if (c0 == 0 && lane_id() == 0) clear_idle_spill_set(src);
  const uint32_t c_end = c0 + kPer < n_cells ? c0 + kPer : n_cells;
  __shared__ SlotTable tab[kCellsPerBlock];
  cells_stream_bin<G>(src, dst, c0, c_end, g, status, trace_cell, tab[threadIdx.x / 64]);
}

// Slots in the destination cells of a wave's particles that all move from
// cell c0 to c0 or one of its 26 neighbours, direction
// dir = 9 (dx + 1) + 3 (dy + 1) + (dz + 1) for axis offsets dx, dy, dz in
// {-1, 0, 1} (x-major ids: the neighbour is c0 + dx sx + dy sy + dz).  LDS
// atomics number each direction's lanes; lane d then adds direction d's
// count to that cell's counter, one global atomic for every direction in
// use, so the wave makes one round trip and no loop over its distinct
// destinations.  s_dir: 54 words of LDS owned by the wave.  Every lane of
// the wave calls it; an inactive lane passes dir 13 and ignores the result.
__device__ __forceinline__ uint32_t neighbour_fetch_add(gptr<uint32_t> ctr, uint32_t c0,
                                                        uint32_t sx, uint32_t sy, uint32_t dir,
                                                        bool active, uint32_t *s_dir) {
  const uint32_t lane = lane_id();
  if (lane < 27u) s_dir[lane] = 0u;
  wave_lds_sync();
  uint32_t rank = 0;
  if (active) rank = atomicAdd(&s_dir[dir], 1u);
  wave_lds_sync();
  if (lane < 27u) {
    const uint32_t cnt = s_dir[lane];
    uint32_t base = 0;
    if (cnt != 0u) {
      const int32_t dx = (int32_t)(lane / 9u) - 1, dy = (int32_t)(lane / 3u % 3u) - 1,
                    dz = (int32_t)(lane % 3u) - 1;
      const uint32_t key =
          (uint32_t)((int32_t)c0 + dx * (int32_t)sx + dy * (int32_t)sy + dz);
      base = atomic_add(ctr + key, cnt);
    }
    s_dir[27u + lane] = base;
  }
  wave_lds_sync();
  return s_dir[27u + dir] + rank;
}

// Exclusive scan of the counts into compact offsets (trace only; the counts
// are left intact).  Tile-local pass, then carries from earlier tiles.
__global__ __launch_bounds__(kBlock) void k_scan_tiles(Cells cur_arg,
                                                       uint32_t *offsets,
                                                       uint32_t *tile_sums,
                                                       int64_t n_cells) {
  const GCells cur = to_global(cur_arg);
  __shared__ uint32_t s_wave[kBlock / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
  const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
  uint32_t v[8];
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t idx = base + j;
    const uint32_t cnt = idx < n_cells ? cur.count[idx] : 0u;
    v[j] = sum;
    sum += cnt;
  }
  uint32_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_up(incl, o);
    if ((int)lane >= o) incl += up;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  uint32_t wave_off = 0;
  for (uint32_t w = 0; w < wave; ++w) wave_off += s_wave[w];
  const uint32_t excl = wave_off + incl - sum;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t idx = base + j;
    if (idx < n_cells) offsets[idx] = excl + v[j];
  }
  if (threadIdx.x == kBlock - 1) tile_sums[blockIdx.x] = wave_off + incl;
}

__global__ __launch_bounds__(kBlock) void k_scan_carry(uint32_t *offsets,
                                                       const uint32_t *tile_sums,
                                                       int64_t n_cells) {
  __shared__ uint32_t s_red[kBlock / 64];
  const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
  uint32_t part = 0;
  for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kBlock) part += tile_sums[j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o);
  if (lane == 0) s_red[wave] = part;
  __syncthreads();
  uint32_t carry = 0;
  for (int w = 0; w < kBlock / 64; ++w) carry += s_red[w];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 8;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t idx = base + j;
    if (idx < n_cells) offsets[idx] += carry;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
    offsets[n_cells] = carry + tile_sums[blockIdx.x];
}

// ---------------------------------------------------------------------------
// Collisions: one wave64 (one workgroup) per cell (several: k_step_wide).
// ---------------------------------------------------------------------------
// A cell being stepped: member j is slot base + j of the buffer's arrays,
// or, in an overflowing cell (ov), for j >= cap spill slot sbase + sidx[j -
// cap] (at_spill).  ov is uniform over the workgroup, so normal cells take
// the first form without a per-lane choice.  Once an overflowing cell's
// slots are listed in LDS (slots; unless unlisted), at() reads them there,
// which keeps fewer values live than the two-part form.
struct CellView {
  uint32_t c, n, t;
  size_t base;
  uint32_t cap;
  bool ov, unlisted;
  size_t sbase;
  const uint32_t *sidx;
  const uint32_t *slots;
  __device__ __forceinline__ size_t at_spill(uint32_t j) const {
    if (ov && j >= cap) return sbase + sidx[j - cap];
    return base + j;
  }
  __device__ __forceinline__ size_t at(uint32_t j) const {
    if (ov) return unlisted ? at_spill(j) : slots[j];
    return base + j;
  }
};

// kBlockSync: the workgroup is this one wave, and its barriers order the
// LDS accesses; otherwise a wave that shares its workgroup with others
// synchronises with itself only.
template <bool kBlockSync>
__device__ __forceinline__ void cell_sync() {
  if (kBlockSync)
    __syncthreads();
  else
    wave_lds_sync();
}

// Exact Eq. (3) test of the nf filtered pairs in s_filt (increasing pair
// index), then greedy claim in that order.  Entries are rewritten as
// flag | a << 10 | b.  claimed_bits holds, per lane, the claimed flags of
// canonical indices lane + 64 j.  One wave; see cell_sync for kBlockSync.
template <bool kTrace, bool kBlockSync = true>
__device__ __forceinline__ void resolve_filtered(
    uint32_t nf, const CellView &cv, const PairArgs &pa, const GState &st,
    const uint16_t *s_perm, uint32_t *s_filt, uint32_t *s_claim,
    uint32_t &nclaim, uint32_t &claimed_bits, uint32_t &n_acc,
    const TraceArgs &tr, DevStatus *status) {
  const uint32_t lane = lane_id();
  cell_sync<kBlockSync>();
  for (uint32_t i = lane; i < nf; i += 64) {
    const uint32_t k = s_filt[i];
    const Words4 w = philox10(k, cv.c, cv.t, 0u, pa.key0, pa.key1);
    const double u = uniform53(w.w0, w.w1);
    uint32_t a, b;
    pair_of_index(k, cv.n, a, b);
    const size_t ia = cv.at(s_perm[a]), ib = cv.at(s_perm[b]);
    double ax, ay, az, bx, by, bz;
    load_momentum(st, ia, ax, ay, az);
    load_momentum(st, ib, bx, by, bz);
    const bool acc = u < p22(ax, ay, az, bx, by, bz, pa.kfac);
    n_acc += acc ? 1u : 0u;
    s_filt[i] = acc ? (0x80000000u | (a << 10) | b) : 0u;
    if (kTrace && acc && tr.cand) {
      const uint32_t slot = atomicAdd(&tr.counts[0], 1u);
      if (slot < tr.cand_cap) {
        tr.cand[3 * (size_t)slot + 0] = cv.c;
        tr.cand[3 * (size_t)slot + 1] = a;
        tr.cand[3 * (size_t)slot + 2] = b;
      } else {
        atomicOr(&status->err, kErrTrace);
      }
    }
  }
  cell_sync<kBlockSync>();
  // the accepted entries in list order: a row of 64 entries at a time, its
  // accepted ones taken from their lanes in lane order
  for (uint32_t i0 = 0; i0 < nf; i0 += 64u) {
    const uint32_t vr = i0 + lane < nf ? s_filt[i0 + lane] : 0u;
    for (uint64_t m = __ballot((vr & 0x80000000u) != 0u); m != 0; m &= m - 1ull) {
      const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)vr,
                                                             (int)__builtin_ctzll(m));
      const uint32_t a = (v >> 10) & 1023u, b = v & 1023u;
      const bool own_a = (a & 63u) == lane, own_b = (b & 63u) == lane;
      const bool hit = (own_a && ((claimed_bits >> (a >> 6)) & 1u)) ||
                       (own_b && ((claimed_bits >> (b >> 6)) & 1u));
      if (__ballot(hit) == 0) {
        if (own_a) claimed_bits |= 1u << (a >> 6);
        if (own_b) claimed_bits |= 1u << (b >> 6);
        if (lane == 0) s_claim[nclaim] = v;
        ++nclaim;
      }
    }
  }
  cell_sync<kBlockSync>();
}

// Pair tests k = k_begin .. k_end - 1 of a cell by one wave, lane-strided,
// two rows of 64 pairs per iteration while two rows remain.  A pair whose
// Philox word w1 rules out acceptance (u >= w1 2^-32 > P22) is dropped at
// once; the others are appended to filt (nf entries, increasing k; at most
// kFiltCap).  kResolve: when filt nears full its entries are resolved
// (exact test and claims) and the tests go on; otherwise the tests stop
// there.  Returns the first pair not tested (k_end when all were).
template <bool kResolve, bool kTrace, bool kBlockSync, uint32_t kFiltCap>
__device__ __forceinline__ uint32_t test_pairs(
    uint32_t k_begin, uint32_t k_end, const CellView &cv, const PairArgs &pa,
    const GState &st, const uint16_t *s_perm, uint32_t *filt, uint32_t &nf,
    uint32_t *s_claim, uint32_t &nclaim, uint32_t &claimed_bits, uint32_t &n_acc,
    const TraceArgs &tr, DevStatus *status) {
  static_assert(kFiltCap >= 256, "filter buffer");
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  const uint32_t lim = pa.w1_max;
  uint32_t k0 = k_begin;
  for (; k0 + 128u <= k_end; k0 += 128u) {
    const uint32_t ka = k0 + lane, kb = k0 + 64u + lane;
    const uint32_t wa = philox10_w1(ka, cv.c, cv.t, 0u, pa.key0, pa.key1);
    const uint32_t wb = philox10_w1(kb, cv.c, cv.t, 0u, pa.key0, pa.key1);
    const bool pass_a = wa <= lim, pass_b = wb <= lim;
    const uint64_t ma = __ballot(pass_a), mb = __ballot(pass_b);
    if ((ma | mb) != 0) {
      if (pass_a) filt[nf + (uint32_t)__popcll(ma & below)] = ka;
      nf += (uint32_t)__popcll(ma);
      if (pass_b) filt[nf + (uint32_t)__popcll(mb & below)] = kb;
      nf += (uint32_t)__popcll(mb);
      if (nf > kFiltCap - 128u) {
        if (!kResolve) return k0 + 128u;
        resolve_filtered<kTrace, kBlockSync>(nf, cv, pa, st, s_perm, filt, s_claim, nclaim,
                                             claimed_bits, n_acc, tr, status);
        nf = 0;
      }
    }
  }
  for (; k0 < k_end; k0 += 64u) {
    const uint32_t k = k0 + lane;
    bool pass = false;
    if (k < k_end) pass = philox10_w1(k, cv.c, cv.t, 0u, pa.key0, pa.key1) <= lim;
    const uint64_t m = __ballot(pass);
    if (m != 0) {
      if (pass) filt[nf + (uint32_t)__popcll(m & below)] = k;
      nf += (uint32_t)__popcll(m);
      if (nf > kFiltCap - 64u) {
        if (!kResolve) return k0 + 64u < k_end ? k0 + 64u : k_end;
        resolve_filtered<kTrace, kBlockSync>(nf, cv, pa, st, s_perm, filt, s_claim, nclaim,
                                             claimed_bits, n_acc, tr, status);
        nf = 0;
      }
    }
  }
  return k_end;
}

// Cells of more than kBucketRankMin particles rank their ids through
// kRankBuckets buckets by value; smaller cells (one particle a lane) count
// all ids, a shorter chain of independent LDS reads than the buckets'
// reductions, scan and atomics.
constexpr uint32_t kRankBuckets = 256;
constexpr uint32_t kBucketRankMin = 63;

// Minimum / maximum over the wave's 64 lanes (every lane active), the same
// in every lane.  DPP
// moves within the VALU instead of LDS permutes: within quads, half rows
// and rows, then row 15's result into rows 1 and 3 and row 31's into rows
// 2 and 3, so that lane 63 holds the whole wave's; lanes a move does not
// write keep their own value.
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Inclusive prefix sum over the wave's lanes (every lane active): DPP
// shifts by 1, 2, 4 and 8 within rows (lanes without a source add 0), then
// row 15's sum into rows 1 and 3 and row 31's into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);
  return x;
}

// Inclusive prefix maximum over the wave's lanes (every lane active).
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false));
  return x;
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  return wave_reduce(v, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  return wave_reduce(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}

// LDS of a cell: buf holds the cell's ids while the canonical
// order is built; after that its first half holds the filtered pairs and its
// second half the claimed pairs.
template <bool kFused, uint32_t kCap>
struct CellLds {
  __align__(16) uint32_t buf[kCap];
  uint16_t perm[kCap];
  __align__(16) uint32_t bkt[kRankBuckets + 4];  // bucket ends, then starts
  __align__(16) uint32_t sorted[kCap];           // ids in bucket order
  uint32_t ov_pool_lo, ov_pool_hi, ov_ok, pad;   // an overflowing cell's scratch
};

// The launch of step t clears the scratch that no launch uses now: src's
// idle spill counter set and the pool counter of step t + 1.
__device__ __forceinline__ void clear_idle_scratch(const GCells &src, uint32_t t) {
  clear_idle_spill_set(src);
  src.sp->pool->hdr[(t + 1u) & 1u] = 0ull;
}

// Observation sums of a cell (Sec. 5 profiles): sum E, sum p_x and
// sum p_x^2 / E of the momenta after the step's collisions, accumulated per
// lane, then reduced over the wave and written with the cell's count by
// lane 0 (obs: kCellSums doubles a cell).
__device__ __forceinline__ void obs_add(double px, double py, double pz, double &se,
                                        double &sp, double &sxx) {
  const double e = norm3(px, py, pz);
  se += e;
  sp += px;
  sxx += (px * px) / e;
}

__device__ __forceinline__ void obs_write_wave(double *obs, uint32_t c, uint32_t cnt,
                                               double se, double sp, double sxx) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    se += __shfl_down(se, o);
    sp += __shfl_down(sp, o);
    sxx += __shfl_down(sxx, o);
  }
  if (lane_id() == 0) {
    double *const out = obs + kCellSums * (size_t)c;
    out[0] = se;
    out[1] = sp;
    out[2] = sxx;
    out[3] = (double)cnt;
  }
}

// Wave 0 of an overflowing cell's workgroup: takes scratch from the pool
// (counter t & 1) for the slots of the cell's spilled members -- and, for a
// cell of more than kHeld, its canonical order, claimed flags and
// claims -- and lists those slots (a scan of the spill slots, in increasing
// order).  Leaves the scratch offset and a success flag in LDS.
template <uint32_t kHeld, bool kFused, uint32_t kCap>
__device__ void find_spilled(const GCells &src, const CellView &cv, CellLds<kFused, kCap> &lds,
                             DevStatus *status) {
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  const SpillDesc *const sd = src.sp;
  OverflowPool *const pool = sd->pool;
  const uint32_t n = cv.n, nsp = cv.ov ? n - cv.cap : 0u;
  const uint32_t ns = min(sd->hdr[2u * src.q], sd->capacity);
  uint64_t need = nsp;
  if (n > kHeld) need += (uint64_t)n + n / 2u + 1u + (n + 31u) / 32u;
  uint32_t lo = 0, hi = 0;
  if (lane == 0) {
    const unsigned long long b = atomicAdd(&pool->hdr[cv.t & 1u], (unsigned long long)need);
    lo = (uint32_t)b;
    hi = (uint32_t)(b >> 32);
  }
  lo = (uint32_t)__shfl((int)lo, 0);
  hi = (uint32_t)__shfl((int)hi, 0);
  const uint64_t b = ((uint64_t)hi << 32) | lo;
  bool ok = b + need <= pool->capacity;
  if (ok) {
    uint32_t *const mem = pool->buf + b;
    uint32_t found = 0;
    for (uint32_t i0 = 0; nsp != 0u && i0 < ns; i0 += 64u) {
      const uint32_t i = i0 + lane;
      const bool hit = i < ns && sd->cell[i] == cv.c;
      const uint64_t mk = __ballot(hit);
      if (hit) {
        const uint32_t slot = found + (uint32_t)__popcll(mk & below);
        if (slot < nsp) mem[slot] = i;
      }
      found += (uint32_t)__popcll(mk);
    }
    ok = found == nsp;
  }
  if (lane == 0) {
    if (!ok) atomicOr(&status->err, kErrSpill);
    lds.ov_pool_lo = lo;
    lds.ov_pool_hi = hi;
    lds.ov_ok = ok ? 1u : 0u;
  }
}

// The collisions of a cell larger than the LDS holds (then,
// kFused, the binning of its members), by one wave with its canonical
// order, claimed flags and claims in global scratch: ranks by counting
// smaller ids against chunks staged in LDS, pair tests 64 at a time in
// increasing k (Philox w1 filter, then Eq. (3)), each row's accepted pairs
// claimed in k order, then the kinematics.  A cell past the 32-bit pair
// index skips its collisions (flagged); its members are still binned.
template <bool kFused, bool kTrace, uint32_t kCap>
__device__ void large_cell_step(const GCells &src, const GCells &dst, const CellView &cv,
                                const PairArgs &pa, const Geometry &g, DevStatus *status,
                                const TraceArgs &tr, CellLds<kFused, kCap> &lds,
                                double *obs) {
  const uint32_t lane = lane_id();
  const uint32_t n = cv.n;
  uint32_t *const perm = const_cast<uint32_t *>(cv.sidx) + (cv.ov ? n - cv.cap : 0u);
  uint32_t *const claims = perm + n;
  uint32_t *const bits = claims + n / 2u + 1u;
  const GState &st = src.st;
  uint32_t npairs = 0;  // < 2^32 below the pair-index bound
  uint32_t nclaim = 0, n_acc = 0;
  if (n > kMaxPairIndexCell) {
    if (lane == 0) atomicOr(&status->err, kErrPairIndex);
  } else {
    for (uint32_t j0 = 0; j0 < n; j0 += 64u) {
      const uint32_t j = j0 + lane;
      const uint32_t me = j < n ? st.id[cv.at_spill(j)] : 0xFFFFFFFFu;
      uint32_t r = 0;
      for (uint32_t i0 = 0; i0 < n; i0 += kCap) {
        const uint32_t cnt = min(kCap, n - i0);
        wave_lds_sync();
        for (uint32_t i = lane; i < cnt; i += 64u) lds.buf[i] = st.id[cv.at_spill(i0 + i)];
        wave_lds_sync();
        if (j < n)
          for (uint32_t i = 0; i < cnt; ++i) r += lds.buf[i] < me ? 1u : 0u;
      }
      if (j < n) {
        perm[r] = j;
        if (kTrace && tr.perm) tr.perm[tr.offsets[cv.c] + r] = me;
      }
    }
    for (uint32_t w = lane; w < (n + 31u) / 32u; w += 64u) bits[w] = 0u;
    wave_lds_sync();
    npairs = (uint32_t)((uint64_t)n * (n - 1u) / 2u);
    // k0 + 64 stays below 2^32: npairs <= 4 294 930 221
    for (uint32_t k0 = 0; pa.any && k0 < npairs; k0 += 64u) {
      const uint32_t k = k0 + lane;
      bool acc = false;
      if (k < npairs && philox10_w1(k, cv.c, cv.t, 0u, pa.key0, pa.key1) <= pa.w1_max) {
        const Words4 w = philox10(k, cv.c, cv.t, 0u, pa.key0, pa.key1);
        uint32_t a, b;
        pair_of_index64(k, n, a, b);
        const size_t ia = cv.at_spill(perm[a]), ib = cv.at_spill(perm[b]);
        double ax, ay, az, bx, by, bz;
        load_momentum(st, ia, ax, ay, az);
        load_momentum(st, ib, bx, by, bz);
        acc = uniform53(w.w0, w.w1) < p22(ax, ay, az, bx, by, bz, pa.kfac);
        if (kTrace && acc && tr.cand) {
          const uint32_t slot = atomicAdd(&tr.counts[0], 1u);
          if (slot < tr.cand_cap) {
            tr.cand[3 * (size_t)slot + 0] = cv.c;
            tr.cand[3 * (size_t)slot + 1] = a;
            tr.cand[3 * (size_t)slot + 2] = b;
          } else {
            atomicOr(&status->err, kErrTrace);
          }
        }
      }
      n_acc += acc ? 1u : 0u;
      for (uint64_t m = __ballot(acc); m != 0; m &= m - 1ull) {
        const uint32_t kk = k0 + (uint32_t)__builtin_ctzll(m);
        uint32_t a, b;
        pair_of_index64(kk, n, a, b);
        const uint32_t wa = bits[a >> 5], wb = bits[b >> 5];
        if (((wa >> (a & 31u)) & 1u) == 0u && ((wb >> (b & 31u)) & 1u) == 0u) {
          if (lane == 0) {
            if ((a >> 5) == (b >> 5)) {
              bits[a >> 5] = wa | (1u << (a & 31u)) | (1u << (b & 31u));
            } else {
              bits[a >> 5] = wa | (1u << (a & 31u));
              bits[b >> 5] = wb | (1u << (b & 31u));
            }
            claims[nclaim] = kk;
          }
          ++nclaim;
          wave_lds_sync();
        }
      }
    }
  }
  wave_lds_sync();
  for (uint32_t i0 = 0; i0 < nclaim; i0 += 64u) {
    const uint32_t i = i0 + lane;
    if (i < nclaim) {
      const uint32_t k = claims[i];
      uint32_t a, b;
      pair_of_index64(k, n, a, b);
      const Words4 w = philox10(k, cv.c, cv.t, 1u, pa.key0, pa.key1);
      const size_t ia = cv.at_spill(perm[a]), ib = cv.at_spill(perm[b]);
      double ax, ay, az, bx, by, bz;
      load_momentum(st, ia, ax, ay, az);
      load_momentum(st, ib, bx, by, bz);
      scatter_pair(ax, ay, az, bx, by, bz, uniform53(w.w0, w.w1), uniform53(w.w2, w.w3));
      put_momentum(st, ia, ax, ay, az);
      put_momentum(st, ib, bx, by, bz);
      if (kTrace && tr.claim) {
        const uint32_t slot = atomicAdd(&tr.counts[1], 1u);
        if (slot < tr.claim_cap) {
          tr.claim[3 * (size_t)slot + 0] = cv.c;
          tr.claim[3 * (size_t)slot + 1] = a;
          tr.claim[3 * (size_t)slot + 2] = b;
        } else {
          atomicOr(&status->err, kErrTrace);
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n_acc += __shfl_down(n_acc, o);
  if (lane == 0) {
    const uint32_t slot = cv.c % kCounterSlots;
    atomicAdd(&status->pairs[slot], (unsigned long long)npairs);
    atomicAdd(&status->cand[slot], (unsigned long long)n_acc);
    atomicAdd(&status->claims[slot], (unsigned long long)nclaim);
  }
  wave_lds_sync();  // new momenta visible to the binning lanes
  double se = 0.0, sp = 0.0, sxx = 0.0;
  if (kFused) {
    const Geometry g_l = g;
    for (uint32_t j0 = 0; j0 < n; j0 += 64u) {
      const uint32_t j = j0 + lane;
      const bool active = j < n;
      Particle q{};
      uint32_t c2 = 0;
      if (active) {
        q = load_particle(st, cv.at_spill(j));
        if (obs) obs_add(q.px, q.py, q.pz, se, sp, sxx);
        advance<true>(g_l, q.x, q.y, q.z, q.px, q.py, q.pz);
        c2 = cell_id(g_l, q.x, q.y, q.z);
      }
      append(dst, c2, active, q, status);
    }
    if (lane == 0) src.count[cv.c] = 0u;
  } else if (obs) {
    for (uint32_t j = lane; j < n; j += 64u) {
      const size_t o = cv.at_spill(j);
      double px, py, pz;
      load_momentum(st, o, px, py, pz);
      obs_add(px, py, pz, se, sp, sxx);
    }
  }
  if (obs) obs_write_wave(obs, cv.c, n, se, sp, sxx);
}

// A fused step of a cell whose members are all in its block keeps the new
// momenta of up to kMax claims in LDS (where the rank sorted its ids; claim
// i's two members at 2i, 2i + 1, and by member a byte map to them, in the
// rank's buckets) for its binning, instead of writing them back to the
// source block, whose lines would then be written to memory once more though
// no one reads them again.
template <uint32_t kCap>
struct ClaimLds {
  static constexpr uint32_t kMax = kCap / 12u;  // 6 doubles a claim in sorted[]
  static_assert(6u * kMax * sizeof(double) <= kCap * sizeof(uint32_t), "claim momenta");
  static_assert(2u * kMax + 2u <= 255u && kCap <= 4u * (kRankBuckets + 4u), "claim map");
  double *mx, *my, *mz;
  uint8_t *map;
  template <bool kFused>
  __device__ __forceinline__ explicit ClaimLds(CellLds<kFused, kCap> &lds)
      : mx(reinterpret_cast<double *>(lds.sorted)), my(mx + 2u * kMax), mz(my + 2u * kMax),
        map(reinterpret_cast<uint8_t *>(lds.bkt)) {}
  // claim i's new momenta, of members ja and jb
  __device__ __forceinline__ void put(uint32_t i, uint32_t ja, uint32_t jb, double ax, double ay,
                                      double az, double bx, double by, double bz) const {
    mx[2u * i] = ax;
    my[2u * i] = ay;
    mz[2u * i] = az;
    mx[2u * i + 1u] = bx;
    my[2u * i + 1u] = by;
    mz[2u * i + 1u] = bz;
    map[ja] = (uint8_t)(2u * i + 1u);
    map[jb] = (uint8_t)(2u * i + 2u);
  }
  // member j's new momentum, if it has one
  __device__ __forceinline__ void take(uint32_t j, Particle &q) const {
    const uint32_t m = map[j];
    if (m != 0u) {
      q.px = mx[m - 1u];
      q.py = my[m - 1u];
      q.pz = mz[m - 1u];
    }
  }
};

// A cell's step by one wave runs in three parts: cell_open (canonical order),
// cell_pairs (pair tests, claims, kinematics) and cell_close (observation
// sums, streaming and binning).
struct CellWork {
  CellView cv;
  bool live;     // the later parts are still to do
  bool mid;      // instead of live: a cell that mid_open took
  bool mom_lds;  // new momenta are in LDS, not written back
};

// A cell of kCap < n <= kCellCap members in the LDS laid out for kCap: the
// words of CellLds up to its scratch fields hold kCellCap ids (then half as many
// filtered pairs and as many claims) and kCellCap canonical positions, which
// leaves no room for the rank's buckets (each lane counts the smaller ids
// instead, 5 % of the instructions of 700 members), for the claims' momenta
// (written back to the block) or for an overflowing cell's slots.  So a box
// whose cells rarely pass kCap keeps the occupancy of kCap's kernels: 24 576
// cells of 350, half of which hold 700 after every other step, 2.3 ms a step
// (3.5 with those cells in global scratch, 2.6 in a wave per cell with the LDS
// for kCellCap); 12 800 such cells of 160 000, the rest empty, 1.40 ms (1.90,
// 1.34).
template <uint32_t kCap>
struct MidLds {
  uint32_t *id;
  uint16_t *perm;
  template <bool kFused>
  __device__ __forceinline__ explicit MidLds(CellLds<kFused, kCap> &lds)
      : id(reinterpret_cast<uint32_t *>(&lds)), perm(reinterpret_cast<uint16_t *>(id + kCellCap)) {
    using Lds = CellLds<kFused, kCap>;
    static_assert(offsetof(Lds, buf) == 0 && offsetof(Lds, ov_pool_lo) >= kCellCap * 6u,
                  "ids and positions");
  }
};

// Its part 1: the canonical order.
template <bool kFused, bool kTrace, uint32_t kCap, bool kBlk>
__device__ __forceinline__ void mid_open(CellWork &w, const GCells &src, const TraceArgs &tr,
                                         CellLds<kFused, kCap> &lds) {
  w.mid = true;
  uint32_t *const s_id = MidLds<kCap>(lds).id;
  uint16_t *const s_perm = MidLds<kCap>(lds).perm;
  CellView &cv = w.cv;
  const uint32_t lane = lane_id(), n = cv.n, n4 = (n + 3u) & ~3u;
  const GState &st = src.st;
  cv.unlisted = true;
  cell_sync<kBlk>();
  for (uint32_t j = lane; j < n4; j += 64u)
    s_id[j] = j < n ? st.id[cv.at_spill(j)] : 0xFFFFFFFFu;
  cell_sync<kBlk>();
  constexpr uint32_t kRows = 4;  // members of a lane ranked together
  const uint4 *const s_id4 = reinterpret_cast<const uint4 *>(s_id);
  for (uint32_t j0 = 0; j0 < n; j0 += 64u * kRows) {
    uint32_t me[kRows], r[kRows];
#pragma unroll
    for (uint32_t u = 0; u < kRows; ++u) {
      const uint32_t j = j0 + 64u * u + lane;
      me[u] = j < n ? s_id[j] : 0u;
      r[u] = 0u;
    }
    for (uint32_t m = 0; m < n4 / 4u; ++m) {
      const uint4 v = s_id4[m];
#pragma unroll
      for (uint32_t u = 0; u < kRows; ++u)
        r[u] += (v.x < me[u]) + (v.y < me[u]) + (v.z < me[u]) + (v.w < me[u]);
    }
#pragma unroll
    for (uint32_t u = 0; u < kRows; ++u) {
      const uint32_t j = j0 + 64u * u + lane;
      if (j < n) {
        s_perm[r[u]] = (uint16_t)j;
        if (kTrace && tr.perm) tr.perm[tr.offsets[cv.c] + r[u]] = me[u];
      }
    }
  }
  cell_sync<kBlk>();
}

// Part 1: the cell's view, and its canonical order in lds.perm.  A cell of
// more than kCap particles is opened by mid_open up to kCellCap (kMid: kernels
// of boxes whose blocks exceed kCap; the longer kernels take up to 1 % more),
// else stepped here altogether.  Starts with a barrier, so a wave may call it
// for several cells.
// kBlk: the workgroup is this one wave; else the wave shares it with others
// and synchronises with itself only.
template <bool kFused, bool kTrace, uint32_t kCap, bool kBlk, bool kMid>
__device__ __forceinline__ void cell_open(CellWork &w, const GCells &src, const GCells &dst,
                                          uint32_t c, uint32_t t, const PairArgs &pa,
                                          const Geometry &g, DevStatus *status,
                                          const TraceArgs &tr, CellLds<kFused, kCap> &lds,
                                          double *obs) {
  w.live = w.mid = false;
  w.mom_lds = false;
  uint32_t *const s_id = lds.buf;
  uint16_t *const s_perm = lds.perm;
  cell_sync<kBlk>();
  const uint32_t lane = lane_id();
  CellView &cv = w.cv;
  cv.c = c;
  cv.t = t;
  cv.base = (size_t)cv.c * src.cap;
  cv.cap = src.cap;
  cv.n = src.count[cv.c];
  cv.ov = cv.n > src.cap;
  cv.unlisted = false;
  cv.sbase = 0;
  cv.sidx = nullptr;
  cv.slots = lds.sorted;
  if (cv.c == 0 && lane == 0) clear_idle_scratch(src, t);
  // Wave priority: the phases that are chains of dependent loads, LDS
  // atomics and barriers (ids and rank; claims, kinematics and binning)
  // issue ahead of the other waves' pair-test loops, which keep the VALU
  // busy meanwhile; the pair tests run at the base priority.
  __builtin_amdgcn_s_setprio(1);
  if (kMid ? __builtin_expect(cv.ov, 0) : cv.ov || cv.n > kCap) {
    // an overflowing cell: find its spilled members, then step it like any
    // other cell, or if it is too large for that with the global-memory method
    constexpr uint32_t kHeld = kMid ? kCellCap : kCap;
    find_spilled<kHeld>(src, cv, lds, status);
    cell_sync<kBlk>();
    if (lds.ov_ok == 0u) return;  // internal error, flagged
    const SpillDesc *const sd = src.sp;
    cv.sbase = sd->base;
    cv.sidx = sd->pool->buf + (((uint64_t)lds.ov_pool_hi << 32) | lds.ov_pool_lo);
    if (cv.n > kHeld) {
      large_cell_step<kFused, kTrace, kCap>(src, dst, cv, pa, g, status, tr, lds, obs);
      return;
    }
  }
  if constexpr (kMid) {
    if (__builtin_expect(cv.n > kCap, 0)) {
      mid_open<kFused, kTrace, kCap, kBlk>(w, src, tr, lds);
      return;
    }
  }
  const uint32_t n = cv.n;
  const GState &st = src.st;
  w.live = true;
  if (n >= 2) {
    // ids to LDS, padded to a multiple of 4 with an id no particle has
    const uint32_t n4 = (n + 3u) & ~3u;
    for (uint32_t j = lane; j < n4; j += 64u)
      s_id[j] = j < n ? st.id[cv.at_spill(j)] : 0xFFFFFFFFu;
    cell_sync<kBlk>();

    // canonical order: the rank of each id among the cell's ids
    if (n > kBucketRankMin) {
      // Counting by buckets of the id value (monotone in the id, so the
      // rank is exact whatever the ids): the bucket's start plus the number
      // of smaller ids in the same bucket.  Bucket b holds the ids with
      // (id - lo) >> shift == b, shift chosen so that b < kRankBuckets.
      uint32_t lo = 0xFFFFFFFFu, hi = 0u;
      for (uint32_t j = lane; j < n; j += 64) {
        const uint32_t v = s_id[j];
        lo = min(lo, v);
        hi = max(hi, v);
      }
      lo = wave_min(lo);
      hi = wave_max(hi);
      const uint32_t bits = 32u - (uint32_t)__builtin_clz(hi - lo);  // hi > lo: ids differ
      const uint32_t shift = bits > 8u ? bits - 8u : 0u;
      uint32_t *const s_bkt = lds.bkt;
      uint32_t *const s_sorted = lds.sorted;
      for (uint32_t b = lane; b < kRankBuckets; b += 64u) s_bkt[b] = 0u;
      if (lane == 0) s_bkt[kRankBuckets] = n;
      cell_sync<kBlk>();
      for (uint32_t j = lane; j < n; j += 64u) atomicAdd(&s_bkt[(s_id[j] - lo) >> shift], 1u);
      cell_sync<kBlk>();
      {  // inclusive scan of the counts: s_bkt[b] = end of bucket b
        uint4 q = reinterpret_cast<uint4 *>(s_bkt)[lane];
        q.y += q.x;
        q.z += q.y;
        q.w += q.z;
        const uint32_t incl = wave_inclusive_sum(q.w);
        const uint32_t excl = incl - q.w;
        q.x += excl;
        q.y += excl;
        q.z += excl;
        q.w += excl;
        reinterpret_cast<uint4 *>(s_bkt)[lane] = q;
      }
      cell_sync<kBlk>();
      // each bucket filled from its end: afterwards s_bkt[b] is its start
      for (uint32_t j = lane; j < n; j += 64u) {
        const uint32_t v = s_id[j];
        const uint32_t pos = atomicSub(&s_bkt[(v - lo) >> shift], 1u) - 1u;
        s_sorted[pos] = v;
      }
      cell_sync<kBlk>();
      for (uint32_t j = lane; j < n; j += 64u) {
        const uint32_t me = s_id[j], b = (me - lo) >> shift;
        const uint32_t p1 = s_bkt[b + 1];
        uint32_t r = s_bkt[b];
        for (uint32_t p = r; p < p1; ++p) r += s_sorted[p] < me ? 1u : 0u;
        s_perm[r] = (uint16_t)j;
        if (kTrace && tr.perm) tr.perm[tr.offsets[cv.c] + r] = me;
      }
    } else {
      // at most kBucketRankMin < 64 particles: one per lane, counting all ids
      const uint4 *s_id4 = reinterpret_cast<const uint4 *>(s_id);
      static_assert(kBucketRankMin < 64, "one particle per lane");
      if (lane < n) {
        const uint32_t me = s_id[lane];
        uint32_t r = 0;
        for (uint32_t m = 0; m < n4 / 4; ++m) {
          const uint4 q = s_id4[m];
          r += (q.x < me) + (q.y < me) + (q.z < me) + (q.w < me);
        }
        s_perm[r] = (uint16_t)lane;
        if (kTrace && tr.perm) tr.perm[tr.offsets[cv.c] + r] = me;
      }
    }
    cell_sync<kBlk>();
    if (cv.ov) {  // the members' slots, in LDS (the rank no longer needs it)
      for (uint32_t j = lane; j < n; j += 64u) lds.sorted[j] = (uint32_t)cv.at_spill(j);
      cell_sync<kBlk>();
    } else if (!kTrace) {
      // the claim map (one byte a member, zero: not scattered), in the
      // rank's buckets; the barrier after the pair tests orders it
      for (uint32_t j = lane * 4u; j < n; j += 256u)
        *reinterpret_cast<uint32_t *>(ClaimLds<kCap>(lds).map + j) = 0u;
    }
  } else if (kTrace && n == 1 && lane == 0 && tr.perm) {
    tr.perm[tr.offsets[cv.c]] = st.id[cv.at_spill(0)];
  }
}

// Part 2, on a cell's scratch: its canonical order in s_perm, kFilt filtered
// pairs in s_filt (filtered: nf of them there already, in increasing k; else
// they are found here) and its claims, at most n / 2, in s_claim.  kMomCap:
// claims whose new momenta fit cl.
template <bool kFused, bool kTrace, bool kBlk, uint32_t kFilt, uint32_t kMomCap, uint32_t kCap>
__device__ __forceinline__ void pairs_step(CellWork &w, const GCells &src, const PairArgs &pa,
                                           DevStatus *status, const TraceArgs &tr,
                                           const uint16_t *s_perm, uint32_t *s_filt,
                                           uint32_t *s_claim, const ClaimLds<kCap> &cl,
                                           const double *obs, bool filtered, uint32_t nf) {
  const CellView &cv = w.cv;
  const uint32_t lane = lane_id(), n = cv.n;
  const GState &st = src.st;
  uint32_t nclaim = 0;
  // every pair k = 0 .. n(n-1)/2 - 1 (test_pairs), then the exact test
  // and the claims of the filtered ones in increasing k
  const uint32_t npairs = n * (n - 1u) / 2u;
  uint32_t claimed_bits = 0, n_acc = 0;
  __builtin_amdgcn_s_setprio(0);
  if (!filtered && pa.any)
    test_pairs<true, kTrace, kBlk, kFilt>(0u, npairs, cv, pa, st, s_perm, s_filt, nf, s_claim,
                                          nclaim, claimed_bits, n_acc, tr, status);
  if (nf != 0)
    resolve_filtered<kTrace, kBlk>(nf, cv, pa, st, s_perm, s_filt, s_claim, nclaim,
                                   claimed_bits, n_acc, tr, status);
  cell_sync<kBlk>();

  __builtin_amdgcn_s_setprio(1);
  // work counters (spread over slots by cell against contention)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n_acc += __shfl_down(n_acc, o);
  if (lane == 0) {
    const uint32_t slot = cv.c % kCounterSlots;
    atomicAdd(&status->pairs[slot], (unsigned long long)npairs);
    atomicAdd(&status->cand[slot], (unsigned long long)n_acc);
    atomicAdd(&status->claims[slot], (unsigned long long)nclaim);
  }

  // kinematics of the claimed pairs (disjoint: one writer per particle),
  // written back in place, or for the binning below into LDS; a fused
  // step then bins every particle
  w.mom_lds = kFused && kMomCap != 0u && !cv.ov && nclaim <= kMomCap;
  for (uint32_t i0 = 0; i0 < nclaim; i0 += 64u) {
    const uint32_t i = i0 + lane;
    const bool active = i < nclaim;
    double ax = 0, ay = 0, az = 0, bx = 0, by = 0, bz = 0;
    uint32_t ja = 0, jb = 0;
    if (active) {
      const uint32_t v = s_claim[i];
      const uint32_t a = (v >> 10) & 1023u, b = v & 1023u;
      const uint32_t k = row_start(a, n) + (b - a - 1u);
      const Words4 u = philox10(k, cv.c, cv.t, 1u, pa.key0, pa.key1);
      ja = s_perm[a];
      jb = s_perm[b];
      const size_t ia = cv.at(ja), ib = cv.at(jb);
      load_momentum(st, ia, ax, ay, az);
      load_momentum(st, ib, bx, by, bz);
      scatter_pair(ax, ay, az, bx, by, bz, uniform53(u.w0, u.w1), uniform53(u.w2, u.w3));
      if (w.mom_lds) {
        cl.put(i, ja, jb, ax, ay, az, bx, by, bz);
      } else {
        put_momentum(st, ia, ax, ay, az);
        put_momentum(st, ib, bx, by, bz);
      }
      if (kTrace && tr.claim) {
        const uint32_t slot = atomicAdd(&tr.counts[1], 1u);
        if (slot < tr.claim_cap) {
          tr.claim[3 * (size_t)slot + 0] = cv.c;
          tr.claim[3 * (size_t)slot + 1] = a;
          tr.claim[3 * (size_t)slot + 2] = b;
        } else {
          atomicOr(&status->err, kErrTrace);
        }
      }
    }
  }
  if (kFused || obs) cell_sync<kBlk>();
}

// Part 2 of a cell that the LDS holds.
template <bool kFused, bool kTrace, uint32_t kCap, bool kBlk, bool kFiltered = false>
__device__ __forceinline__ void cell_pairs(CellWork &w, const GCells &src, const PairArgs &pa,
                                           DevStatus *status, const TraceArgs &tr,
                                           CellLds<kFused, kCap> &lds, const double *obs,
                                           uint32_t nf = 0) {
  // filtered pairs and claimed pairs share the id buffer, kCap / 2 each
  constexpr uint32_t kFilt = kCap / 2;
  static_assert(kCap <= kCellCap && kFilt >= 256, "cell capacity");
  if (w.cv.n < 2u) return;
  pairs_step<kFused, kTrace, kBlk, kFilt, ClaimLds<kCap>::kMax, kCap>(
      w, src, pa, status, tr, lds.perm, lds.buf, lds.buf + kFilt, ClaimLds<kCap>(lds), obs,
      kFiltered, nf);
}

// Part 3 (with kFused clears src's count).
template <bool kFused, uint32_t kCap>
__device__ __forceinline__ void cell_close(const CellWork &w, const GCells &src,
                                           const GCells &dst, const Geometry &g,
                                           DevStatus *status, CellLds<kFused, kCap> &lds,
                                           double *obs) {
  const CellView &cv = w.cv;
  const uint32_t lane = lane_id(), n = cv.n;
  const GState &st = src.st;
  const ClaimLds<kCap> cl(lds);
  if (kFused) {
    // stream and bin every particle (scattered momenta are in LDS or were
    // written back in place; the barrier above makes them visible to all
    // lanes).  The geometry is copied to registers once: read through a
    // reference it would be reloaded after every store.
    const Geometry g_l = g;
    double se = 0.0, sp = 0.0, sxx = 0.0;
    // the source cell's axis indices, for the direction of each move
    const uint32_t sy = (uint32_t)g_l.n[2], sx = (uint32_t)g_l.n[1] * sy;
    const int32_t cx = (int32_t)(cv.c / sx), cy = (int32_t)(cv.c % sx / sy),
                  cz = (int32_t)(cv.c % sy);
    uint32_t *const s_dir = lds.buf;  // the ids' dead buffer
    for (uint32_t j0 = 0; j0 < n; j0 += 64u) {
      const uint32_t j = j0 + lane;
      const bool active = j < n;
      Particle q{};
      uint32_t c2 = 0, dir = 13u;
      bool near = true;
      if (active) {
        q = load_particle(st, cv.at(j));
        if (w.mom_lds) {
          cl.take(j, q);
        }
        if (obs) obs_add(q.px, q.py, q.pz, se, sp, sxx);
        advance<true>(g_l, q.x, q.y, q.z, q.px, q.py, q.pz);
        int32_t ix, iy, iz;
        cell_axes(g_l, q.x, q.y, q.z, ix, iy, iz);
        c2 = (uint32_t)((ix * g_l.n[1] + iy) * g_l.n[2] + iz);
        const int32_t dx = ix - cx, dy = iy - cy, dz = iz - cz;
        // a move of less than a cell edge crosses at most one face per axis
        near = dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1;
        dir = near ? (uint32_t)(9 * (dx + 1) + 3 * (dy + 1) + (dz + 1)) : 13u;
      }
      if (__ballot(!near) == 0ull) {
        const uint32_t slot = neighbour_fetch_add(dst.count, cv.c, sx, sy, dir, active, s_dir);
        if (active) store_particle(dst, c2, slot, q, status);
      } else {
        append(dst, c2, active, q, status);
      }
    }
    if (lane == 0) src.count[cv.c] = 0u;
    if (obs) obs_write_wave(obs, cv.c, n, se, sp, sxx);
  } else if (obs) {
    double se = 0.0, sp = 0.0, sxx = 0.0;
    for (uint32_t j = lane; j < n; j += 64u) {
      const size_t o = cv.at(j);
      double px, py, pz;
      load_momentum(st, o, px, py, pz);
      obs_add(px, py, pz, se, sp, sxx);
    }
    obs_write_wave(obs, cv.c, n, se, sp, sxx);
  }
}

// Parts 2 and 3 of a cell that mid_open took.
template <bool kFused, bool kTrace, uint32_t kCap, bool kBlk>
__device__ __forceinline__ void mid_close(CellWork &w, const GCells &src, const GCells &dst,
                                          const PairArgs &pa, const Geometry &g,
                                          DevStatus *status, const TraceArgs &tr,
                                          CellLds<kFused, kCap> &lds, double *obs,
                                          bool filtered = false, uint32_t nf = 0) {
  constexpr uint32_t kFilt = kCellCap / 2;
  const MidLds<kCap> ml(lds);
  pairs_step<kFused, kTrace, kBlk, kFilt, 0u, kCap>(w, src, pa, status, tr, ml.perm, ml.id,
                                                    ml.id + kFilt, ClaimLds<kCap>(lds), obs,
                                                    filtered, nf);
  cell_close<kFused, kCap>(w, src, dst, g, status, lds, obs);
}

// Collisions of cell c of src at step t by one wave.  kFused: afterwards
// stream and bin the cell's particles into dst for step t+1 and clear src's
// count.
template <bool kFused, bool kTrace, uint32_t kCap, bool kBlk = true, bool kMid = false>
__device__ __forceinline__ void cell_step(const GCells &src, const GCells &dst, uint32_t c,
                                          uint32_t t, const PairArgs &pa,
                                          const Geometry &g, DevStatus *status,
                                          const TraceArgs &tr, CellLds<kFused, kCap> &lds,
                                          double *obs = nullptr) {
  CellWork w;
  cell_open<kFused, kTrace, kCap, kBlk, kMid>(w, src, dst, c, t, pa, g, status, tr, lds, obs);
  if constexpr (kMid)
    if (__builtin_expect(w.mid, 0))
      mid_close<kFused, kTrace, kCap, kBlk>(w, src, dst, pa, g, status, tr, lds, obs);
  if (!w.live) return;
  cell_pairs<kFused, kTrace, kCap, kBlk>(w, src, pa, status, tr, lds, obs);
  cell_close<kFused, kCap>(w, src, dst, g, status, lds, obs);
}

// ---------------------------------------------------------------------------
// Four cells by a workgroup of four waves (boxes of many dense cells).  Wave
// w opens and closes cell c0 + w as above; in between the waves share the
// four cells' pairs:
//   filter      the waves take the rows of 64 pair indices in turn, each
//               testing its indices in all four cells: what rounds 1 to 3 of
//               Philox owe to the index alone (three of a test's 16
//               multiplies, two of its 15 XORs) is computed once for the
//               four.  Passing pairs go to their cell's list in any order;
//   the rest    where no list holds more than kListMax, the waves test the
//               lists exactly in common rows and one wave claims and computes
//               the kinematics, a pair a lane: the ~40 filtered pairs of the
//               four cells fill a row where each cell alone fills a few of
//               its lanes.  Longer lists go to their cell's own wave, sorted.
// A cell whose list would exceed kListAll (or that overflows its block, or
// that holds no pair) is left out and taken by its own wave alone.
// Bound by VALU issue on the full tube (93 % busy; a wave per cell: all the
// time).  Against one wave per cell: 727 -> 578 M VALU instructions a launch
// there, 1.23 -> 1.11 ms; 3-D tube's 50 steps 4.82 -> 4.33 ms (96 -> 87 us a step).  Two
// cells to a workgroup gained half of that, and one LDS atomic a row for all
// four lists, instead of one a list, less than four.
// ---------------------------------------------------------------------------
constexpr uint32_t kListMax = 40;   // of the shared rows; <= ClaimLds::kMax: every claim fits
constexpr uint32_t kListAll = 256;  // of a cell's list
template <uint32_t kG>
struct GroupLds {
  uint32_t n[kG];    // members of the cells that share their pairs, else 0
  uint32_t cnt[kG];  // filtered pairs, listed in the cell's lds.buf
  uint32_t sorted[kG * kListMax];  // the exact test's results, by cell and index
};

template <bool kFused, uint32_t kCap, uint32_t kG>
__device__ __forceinline__ void group_filter(uint32_t c0, uint32_t t, const uint32_t *np,
                                             const PairArgs &pa, GroupLds<kG> &q,
                                             CellLds<kFused, kCap> *lds, uint32_t wv) {
  const uint32_t lane = lane_id(), lim = pa.w1_max;
  const uint64_t tb = (uint64_t)t * kMulB;
  uint32_t s2[kG], s3[kG];  // what the cell adds to word 2 in rounds 2 and 3
#pragma unroll
  for (uint32_t i = 0; i < kG; ++i) {
    const uint64_t ca = (uint64_t)((uint32_t)(tb >> 32) ^ (c0 + i) ^ pa.key0) * kMulA;
    s2[i] = (uint32_t)(ca >> 32) ^ (pa.key1 + kWeylB);
    s3[i] = (uint32_t)ca ^ (pa.key1 + 2u * kWeylB);
  }
  const uint32_t e2 = (uint32_t)tb ^ (pa.key0 + kWeylA), e3 = pa.key0 + 2u * kWeylA;
  const auto uniform = [](uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  };
  uint32_t most = np[0], least = np[0];
#pragma unroll
  for (uint32_t i = 1; i < kG; ++i) {
    most = max(most, np[i]);
    least = min(least, np[i]);
  }
  most = uniform(most);
  least = uniform(least);
  // word w1 of index k in cell i, from the shared products
  const auto word = [&](uint32_t i, uint64_t ka, uint64_t kb, uint64_t kc) {
    const uint64_t kd = (uint64_t)((uint32_t)ka ^ s2[i]) * kMulB;  // round 3
    return philox_w1_from<3>(xor3((uint32_t)(kd >> 32), (uint32_t)kb, e3), (uint32_t)kd,
                             (uint32_t)(kc >> 32) ^ s3[i], (uint32_t)kc, pa.key0, pa.key1);
  };
  const auto put = [&](uint32_t i, uint32_t k, bool pass) {
    if (__ballot(pass) != 0ull && pass) {
      const uint32_t at = atomicAdd(&q.cnt[i], 1u);
      if (at < kListAll) lds[i].buf[at] = k;
    }
  };
  uint32_t k0 = wv * 64u;
  for (; k0 + 64u <= least; k0 += 64u * kG) {  // whole rows of every cell
    const uint32_t k = k0 + lane;
    const uint64_t ka = (uint64_t)k * kMulA;                                 // round 1
    const uint64_t kb = (uint64_t)((uint32_t)(ka >> 32) ^ pa.key1) * kMulB;  // round 2
    const uint64_t kc = (uint64_t)((uint32_t)(kb >> 32) ^ e2) * kMulA;       // round 3
    uint32_t w[kG], low = 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t i = 0; i < kG; ++i) {
      w[i] = word(i, ka, kb, kc);
      low = min(low, w[i]);
    }
    if (__ballot(low <= lim) != 0ull) {
#pragma unroll
      for (uint32_t i = 0; i < kG; ++i) put(i, k, w[i] <= lim);
    }
  }
  for (; k0 < most; k0 += 64u * kG) {
    const uint32_t k = k0 + lane;
    const uint64_t ka = (uint64_t)k * kMulA;
    const uint64_t kb = (uint64_t)((uint32_t)(ka >> 32) ^ pa.key1) * kMulB;
    const uint64_t kc = (uint64_t)((uint32_t)(kb >> 32) ^ e2) * kMulA;
#pragma unroll
    for (uint32_t i = 0; i < kG; ++i)
      if (k0 < np[i]) put(i, k, word(i, ka, kb, kc) <= lim && k < np[i]);
  }
}

// The cells' parts of GroupLds::sorted: off[i] is the first entry of cell i;
// a cell that its own wave takes has none.
template <uint32_t kG>
__device__ __forceinline__ void group_offsets(const GroupLds<kG> &q, uint32_t *off) {
  off[0] = 0;
#pragma unroll
  for (uint32_t i = 0; i < kG; ++i) {
    const uint32_t f = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.cnt[i]);
    off[i + 1] = off[i] + (f <= kListMax ? f : 0u);
  }
}

// Exact tests of the filtered pairs, wave wv the rows wv, wv + kG, ... of 64:
// each pair ranks its index in its cell's list and leaves flag | cell << 20 |
// a << 10 | b at its place.
template <bool kFused, uint32_t kCap, uint32_t kG>
__device__ __forceinline__ void group_exact(uint32_t c0, uint32_t t, const uint32_t *n,
                                            const PairArgs &pa, const GCells &src,
                                            GroupLds<kG> &q, const CellLds<kFused, kCap> *lds,
                                            uint32_t wv) {
  uint32_t off[kG + 1];
  group_offsets<kG>(q, off);
  for (uint32_t e = wv * 64u + lane_id(); e < off[kG]; e += 64u * kG) {
    uint32_t i = 0, first = 0, f = off[1], nn = n[0];
#pragma unroll
    for (uint32_t u = 1; u < kG; ++u)
      if (e >= off[u]) {
        i = u;
        first = off[u];
        f = off[u + 1] - off[u];
        nn = n[u];
      }
    const uint32_t k = lds[i].buf[e - first];
    const uint4 *const list = reinterpret_cast<const uint4 *>(lds[i].buf);
    uint32_t r = first;
#pragma unroll 2
    for (uint32_t m = 0; 4u * m < f; ++m) {
      const uint4 v = list[m];
      r += (v.x < k) + (v.y < k) + (v.z < k) + (v.w < k);
    }
    const Words4 w = philox10(k, c0 + i, t, 0u, pa.key0, pa.key1);
    uint32_t a, b;
    pair_of_index(k, nn, a, b);
    const size_t base = (size_t)(c0 + i) * src.cap;
    double ax, ay, az, bx, by, bz;
    load_momentum(src.st, base + lds[i].perm[a], ax, ay, az);
    load_momentum(src.st, base + lds[i].perm[b], bx, by, bz);
    const bool acc = uniform53(w.w0, w.w1) < p22(ax, ay, az, bx, by, bz, pa.kfac);
    q.sorted[r] = (acc ? 0x80000000u : 0u) | i << 20 | a << 10 | b;
  }
}

// Claims and kinematics (one wave): the accepted pairs move together, in
// order; each row of 64 is claimed in order and its claims scattered, a pair
// a lane.
template <bool kFused, uint32_t kCap, uint32_t kG>
__device__ __forceinline__ void group_claim(uint32_t c0, uint32_t t, const uint32_t *n,
                                            const PairArgs &pa, const GCells &src,
                                            DevStatus *status, GroupLds<kG> &q,
                                            CellLds<kFused, kCap> *lds) {
  static_assert(kListMax <= ClaimLds<kCap>::kMax, "claim momenta");
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t off[kG + 1], pairs = 0;
  group_offsets<kG>(q, off);
#pragma unroll
  for (uint32_t i = 0; i < kG; ++i)
    if (n[i] > 1u && (uint32_t)__builtin_amdgcn_readfirstlane((int)q.cnt[i]) <= kListMax)
      pairs += n[i] * (n[i] - 1u) / 2u;
  uint32_t total = 0;  // accepted pairs
  for (uint32_t e0 = 0; e0 < off[kG]; e0 += 64u) {
    const uint32_t v = e0 + lane < off[kG] ? q.sorted[e0 + lane] : 0u;
    wave_lds_sync();
    const uint64_t m = __ballot((v & 0x80000000u) != 0u);
    if (v & 0x80000000u) q.sorted[total + (uint32_t)__popcll(m & below)] = v & 0x7FFFFFFFu;
    total += (uint32_t)__popcll(m);
  }
  wave_lds_sync();
  uint32_t got[kG] = {}, n_claims = 0;  // claims of each cell, and of all
  for (uint32_t e0 = 0; e0 < total; e0 += 64u) {
    const bool have = e0 + lane < total;
    const uint32_t v = have ? q.sorted[e0 + lane] : 0u;
    const uint32_t i = v >> 20, a = (v >> 10) & 1023u, b = v & 1023u;
    const uint32_t ma = i << 10 | a, mb = i << 10 | b;
    const uint32_t ja = lds[i].perm[a], jb = lds[i].perm[b];
    const ClaimLds<kCap> cl(lds[i]);
    // free of an earlier row's claims
    bool open = have && cl.map[ja] == 0 && cl.map[jb] == 0;
    uint64_t won = 0;
    for (uint64_t m = __ballot(open); m != 0; m = __ballot(open)) {
      const uint32_t l = (uint32_t)__builtin_ctzll(m);
      const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
      const uint32_t li = vl >> 10 & ~1023u, la = li | (vl >> 10 & 1023u), lb = li | (vl & 1023u);
      won |= 1ull << l;
      open = open && ma != la && ma != lb && mb != la && mb != lb;
    }
    const bool mine = ((won >> lane) & 1ull) != 0ull;
    uint32_t at = 0, nn = n[0];  // the claim's number in its cell; members
#pragma unroll
    for (uint32_t u = 0; u < kG; ++u) {
      const uint64_t m = __ballot(mine && i == u);
      if (i == u) {
        at = got[u] + (uint32_t)__popcll(m & below);
        nn = n[u];
      }
      got[u] += (uint32_t)__popcll(m);
    }
    n_claims += (uint32_t)__popcll(won);
    if (mine) {
      const Words4 w = philox10(row_start(a, nn) + (b - a - 1u), c0 + i, t, 1u, pa.key0, pa.key1);
      const size_t base = (size_t)(c0 + i) * src.cap;
      double ax, ay, az, bx, by, bz;
      load_momentum(src.st, base + ja, ax, ay, az);
      load_momentum(src.st, base + jb, bx, by, bz);
      scatter_pair(ax, ay, az, bx, by, bz, uniform53(w.w0, w.w1), uniform53(w.w2, w.w3));
      cl.put(at, ja, jb, ax, ay, az, bx, by, bz);
      if (!kFused) {
        put_momentum(src.st, base + ja, ax, ay, az);
        put_momentum(src.st, base + jb, bx, by, bz);
      }
    }
    wave_lds_sync();
  }
  if (lane == 0) {
    const uint32_t slot = c0 % kCounterSlots;
    atomicAdd(&status->pairs[slot], (unsigned long long)pairs);
    atomicAdd(&status->cand[slot], (unsigned long long)total);
    atomicAdd(&status->claims[slot], (unsigned long long)n_claims);
  }
}

// Sorts a list of nf <= kListAll filtered pairs, padded with all ones (one
// wave): each entry counts the smaller ones.
__device__ __forceinline__ void group_sort(uint32_t nf, uint32_t *list) {
  const uint32_t lane = lane_id();
  constexpr uint32_t kRows = kListAll / 64u;
  uint32_t k[kRows], r[kRows];
#pragma unroll
  for (uint32_t u = 0; u < kRows; ++u) {
    k[u] = list[64u * u + lane];
    r[u] = 0;
    if (64u * u < nf)
      for (uint32_t m = 0; 4u * m < nf; ++m) {
        const uint4 v = reinterpret_cast<const uint4 *>(list)[m];
        r[u] += (v.x < k[u]) + (v.y < k[u]) + (v.z < k[u]) + (v.w < k[u]);
      }
  }
  wave_lds_sync();
#pragma unroll
  for (uint32_t u = 0; u < kRows; ++u)
    if (64u * u + lane < nf) list[r[u]] = k[u];
  wave_lds_sync();
}

// Cells c0 .. c0 + 3 (those below n_cells) by a workgroup of four waves.
template <bool kFused, uint32_t kCap, uint32_t kG, bool kMid>
__device__ __forceinline__ void group_cells_step(const GCells &src, const GCells &dst, uint32_t c0,
                                                uint32_t n_cells, uint32_t t, const PairArgs &pa,
                                                const Geometry &g, DevStatus *status,
                                                GroupLds<kG> &q, CellLds<kFused, kCap> *lds,
                                                double *obs) {
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64u));
  const TraceArgs none{};
  CellWork w;
  w.live = w.mid = false;
  w.cv.n = 0u;
  if (c0 + wv < n_cells)
    cell_open<kFused, false, kCap, false, kMid>(w, src, dst, c0 + wv, t, pa, g, status, none,
                                                lds[wv], obs);
  if (lane_id() == 0) {
    q.n[wv] = (w.live || w.mid) && !w.cv.ov && w.cv.n > 1u ? w.cv.n : 0u;
    // (a mid cell's group never goes together: its canonical positions lie
    // elsewhere; the first kListMax + 1 entries of its list stay unused)
    q.cnt[wv] = w.mid ? kListMax + 1u : 0u;
  }
  // (the ids' buffer becomes the list of filtered pairs, unused entries all ones)
  static_assert(kListAll == 4u * 64u && kListAll <= kCap / 2u, "list");
  reinterpret_cast<uint4 *>(lds[wv].buf)[lane_id()] =
      uint4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  __syncthreads();
  uint32_t n[kG], np[kG];
#pragma unroll
  for (uint32_t i = 0; i < kG; ++i) {
    n[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.n[i]);
    np[i] = n[i] > 1u ? n[i] * (n[i] - 1u) / 2u : 0u;
  }
  __builtin_amdgcn_s_setprio(0);
  if (pa.any) group_filter<kFused, kCap, kG>(c0, t, np, pa, q, lds, wv);
  __builtin_amdgcn_s_setprio(1);
  __syncthreads();
  bool together = true;  // every list short enough for the shared rows
#pragma unroll
  for (uint32_t i = 0; i < kG; ++i)
    together = together && (uint32_t)__builtin_amdgcn_readfirstlane((int)q.cnt[i]) <= kListMax;
  if (together) {
    group_exact<kFused, kCap, kG>(c0, t, n, pa, src, q, lds, wv);
    __syncthreads();
    if (wv == 0) group_claim<kFused, kCap, kG>(c0, t, n, pa, src, status, q, lds);
    __syncthreads();
  }
  if constexpr (kMid) {
    if (__builtin_expect(w.mid, 0)) {
      const uint32_t entries = q.cnt[wv];
      const bool filtered = q.n[wv] != 0u && entries <= kListAll;
      if (filtered) group_sort(entries, lds[wv].buf);  // (unused ones last)
      mid_close<kFused, false, kCap, false>(w, src, dst, pa, g, status, none, lds[wv], obs,
                                            filtered, filtered ? entries - (kListMax + 1u) : 0u);
    }
  }
  if (!w.live) return;
  const uint32_t nf = q.cnt[wv];
  if (together && q.n[wv] != 0u) {
    w.mom_lds = kFused;
  } else if (q.n[wv] != 0u && nf <= kListAll) {
    group_sort(nf, lds[wv].buf);
    cell_pairs<kFused, false, kCap, false, true>(w, src, pa, status, none, lds[wv], obs, nf);
  } else {
    cell_pairs<kFused, false, kCap, false>(w, src, pa, status, none, lds[wv], obs);
  }
  cell_close<kFused, kCap>(w, src, dst, g, status, lds[wv], obs);
}

constexpr uint32_t kPackedMax = 64;  // particles of a packed unit, and of a cell it takes

// The cells among c0 .. c_end - 1 (at most 64) that a packed launch left
// alone (more than kPackedMax particles, or overflowing), stepped one after
// another by the whole wave.
template <bool kFused, bool kTrace, uint32_t kCap, bool kMid = false>
__device__ __forceinline__ void large_cells_step(const GCells &src, const GCells &dst,
                                                 uint32_t c0, uint32_t c_end, uint32_t t,
                                                 const PairArgs &pa,
                                                 const Geometry &g, DevStatus *status,
                                                 const TraceArgs &tr,
                                                 CellLds<kFused, kCap> &lds,
                                                 double *obs = nullptr) {
  const uint32_t c = c0 + lane_id();
  const uint32_t n = c < c_end ? src.count[c] : 0u;
  uint64_t big = __ballot(n > kPackedMax || n > src.cap);
  while (big != 0) {
    const uint32_t l = (uint32_t)__builtin_ctzll(big);
    big &= big - 1ull;
    cell_step<kFused, kTrace, kCap, true, kMid>(src, dst, c0 + l, t, pa, g, status, tr, lds, obs);
  }
}

// ---------------------------------------------------------------------------
// Packed cells: a workgroup of four waves takes a tile of up to 64
// consecutive cells and packs whole cells, in cell order, into units of at
// most 64 particles, one wave a unit, one particle per lane (a unit ends
// before the cell that would not fit).  So a sparse box
// steps with few idle lanes whatever its mix of occupancies, where a fixed
// number of lanes per cell idles most of them in its emptier cells.  Each
// unit:
//   1. loads its particles (a lane each), ids and positions into LDS;
//   2. ranks each id among its cell's ids and stores the momentum at the
//      canonical position (cell start + rank);
//   3. tests each cell's pairs k = i, i + n, i + 2n, ... in its n lanes with
//      the Philox w1 filter, appending the passing ones to an LDS list (in
//      increasing k per cell);
//   4. in rows of 64 list entries: the exact Eq. (3) test, one entry a
//      lane, then the greedy claims of the row's accepted pairs in list
//      order, with the claimed flags of all canonical positions in one
//      wave-uniform mask (a row is resolved early when the list nears full,
//      which keeps each cell's claims in increasing k);
//   5. computes the kinematics of each claimed pair in both of its lanes
//      (same inputs and code, so the same result) and keeps its half;
//   6. fused: streams and bins every particle; else writes the scattered
//      momenta back.
// Cells holding more than 64 particles, or more than their block holds,
// take a wave each after the units (a launch of their own cost 5-12 us a
// step), or are left to the kernels for larger cells.
// What bounds it: VALU issue (~80 % busy on the 32^3 fm^3 set, ~1 400
// instructions a unit, two fifths of them pair tests) where waves fill the
// chip, the chain of a unit's loads, LDS exchanges, slot atomics and stores
// (~10 us) where they do not.  Four waves a tile, not one: 24 units of a
// dense tile one after another kept its wave for 350 us, the last ones
// nearly alone.  160 000 cells, 50 steps: 12 a cell 8.85 -> 5.49 ms (32
// lanes a cell before, one particle a lane, half the lanes idle), 2 a cell
// 1.83 -> 1.79 ms; 128 batched events of 5 100 particles, 100 steps: 30.1 ->
// 7.1 ms (a wave per cell before); 24 ensemble events, 25 steps: 15.4 ->
// 13.0 ms; 32^3 fm^3 set, 10 steps: 20.1 -> 19.5 ms.  Each lane's cell by
// marks at the cells' first lanes and a prefix maximum, where a binary search
// of the counts' prefix in LDS took six dependent reads (and the counters
// summed once a wave): 5.56 -> 5.42 ms, 1.80 -> 1.78, 19.6 -> 19.4 on the set.
// ---------------------------------------------------------------------------
constexpr uint32_t kPackedFilt = 256;  // filtered pairs held before a row is resolved

struct PackedLds {
  __align__(16) uint32_t id[64];   // by lane: the unit's particles, cell by cell
  double x[64], y[64], z[64];      // by lane
  double px[64], py[64], pz[64];   // by canonical position
  uint32_t filt[kPackedFilt];      // filtered pairs: tile cell << 16 | k
  uint32_t start[64], cnt[64];     // by tile cell: first lane, particles
  uint32_t partner[64];            // by canonical position: the claimed partner's
  SlotTable tab;
};

// A wave's LDS: its units, then (after them) its larger cells.
constexpr uint32_t kPackedWaves = 4;
template <bool kFused>
union PackedWaveLds {
  PackedLds unit;
  CellLds<kFused, kSmallCap> cell;
};

// Exact test and claims of filt[i0 .. i0 + 63] (< nf), in list order.
template <bool kTrace>
__device__ __forceinline__ void packed_resolve_row(
    uint32_t i0, uint32_t nf, uint32_t c0, uint32_t t, const PairArgs &pa, PackedLds &lds,
    uint64_t &claimed, uint32_t &nclaim, uint32_t &n_acc, const TraceArgs &tr,
    DevStatus *status) {
  const uint32_t lane = lane_id();
  const uint32_t i = i0 + lane;
  bool acc = false;
  uint32_t v = 0;
  if (i < nf) {
    const uint32_t e = lds.filt[i];
    const uint32_t cl = e >> 16, k = e & 0xFFFFu;
    const uint32_t n = lds.cnt[cl], st = lds.start[cl];
    const Words4 w = philox10(k, c0 + cl, t, 0u, pa.key0, pa.key1);
    uint32_t a, b;
    pair_of_index(k, n, a, b);
    acc = uniform53(w.w0, w.w1) < p22(lds.px[st + a], lds.py[st + a], lds.pz[st + a],
                                      lds.px[st + b], lds.py[st + b], lds.pz[st + b],
                                      pa.kfac);
    v = (st + a) << 8 | (st + b);
    if (kTrace && acc && tr.cand) {
      const uint32_t slot = atomicAdd(&tr.counts[0], 1u);
      if (slot < tr.cand_cap) {
        tr.cand[3 * (size_t)slot + 0] = c0 + cl;
        tr.cand[3 * (size_t)slot + 1] = a;
        tr.cand[3 * (size_t)slot + 2] = b;
      } else {
        atomicOr(&status->err, kErrTrace);
      }
    }
  }
  n_acc += (uint32_t)__popcll(__ballot(acc));
  for (uint64_t m = __ballot(acc); m != 0; m &= m - 1ull) {
    const uint32_t l = (uint32_t)__builtin_ctzll(m);
    const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
    const uint32_t pa_ = vl >> 8, pb_ = vl & 0xFFu;
    const uint64_t ab = (1ull << pa_) | (1ull << pb_);
    if ((claimed & ab) == 0) {
      claimed |= ab;
      if (lane == 0) {
        lds.partner[pa_] = pb_;
        lds.partner[pb_] = pa_;
      }
      ++nclaim;
      if (kTrace && tr.claim && lane == l) {
        const uint32_t e = lds.filt[i];
        const uint32_t cl = e >> 16, st = lds.start[cl];
        const uint32_t slot = atomicAdd(&tr.counts[1], 1u);
        if (slot < tr.claim_cap) {
          tr.claim[3 * (size_t)slot + 0] = c0 + cl;
          tr.claim[3 * (size_t)slot + 1] = pa_ - st;
          tr.claim[3 * (size_t)slot + 2] = pb_ - st;
        } else {
          atomicOr(&status->err, kErrTrace);
        }
      }
    }
  }
}

// One wave's share of the tile of cells c0 .. c_end - 1 (at most 64), by a workgroup of
// kPackedWaves waves: the units are numbered in cell order and wave w takes
// units w, w + kPackedWaves, ...; with kLarge, the cells left out of the
// units (more than 64 particles, or overflowing) follow in the same count,
// each stepped by one wave as in cell_step (if `large`).  The waves meet once, after all
// have read the tile's counts and before those are cleared.
template <bool kFused, bool kTrace, bool kLarge, bool kMid>
__device__ __forceinline__ void packed_cells_step(const GCells &src, const GCells &dst,
                                                  uint32_t c0, uint32_t c_end, uint32_t t,
                                                  const PairArgs &pa, const Geometry &g,
                                                  DevStatus *status, const TraceArgs &tr,
                                                  PackedWaveLds<kFused> &wlds, uint32_t wave,
                                                  bool large, double *obs = nullptr) {
  // wave priority as in cell_step: the filter loop at the base priority,
  // the latency-bound rest of a unit above it
  __builtin_amdgcn_s_setprio(1);
  PackedLds &lds = wlds.unit;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  const uint32_t lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  if (c0 == 0 && wave == 0 && lane == 0) clear_idle_scratch(src, t);
  // the tile's cells, one a lane; overflowing and larger cells are left out
  const uint32_t cc = c0 + lane;
  const uint32_t ccnt = cc < c_end ? src.count[cc] : 0u;
  const bool packed = cc < c_end && ccnt <= kPackedMax && ccnt <= src.cap;
  __syncthreads();
  if (kFused && wave == 0 && packed) src.count[cc] = 0u;  // for the buffer's next use
  if (obs && wave == 0 && packed && ccnt == 0u) {
    double *const out = obs + kCellSums * (size_t)cc;
    out[0] = out[1] = out[2] = out[3] = 0.0;
  }
  const uint64_t left_out = __ballot(ccnt > kPackedMax || ccnt > src.cap);
  const uint32_t nl = packed ? ccnt : 0u;
  const uint32_t incl = wave_inclusive_sum(nl);  // inclusive prefix of the packed counts
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  if (kFused) clear_slot_table(lds.tab);
  uint32_t cnt_pairs = 0, n_acc = 0, n_claims = 0, unit = 0;
  for (uint32_t base = 0; base < total;) {
    // the unit: the cells whose particles end within base + 64 (a prefix of
    // the tile's lanes beyond the previous unit; each cell fits alone)
    const uint64_t fit = __ballot(incl <= base + kPackedMax);
    const uint32_t e = 63u - (uint32_t)__builtin_clzll(fit);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)e);
    if (unit++ % kPackedWaves != wave) {
      base = end;
      continue;
    }
    const uint32_t p = end - base;  // particles of the unit
    const bool in_unit = nl > 0 && incl - nl >= base && lane <= e;
    wave_lds_sync();  // the previous unit's readers of lds are done
    // each lane's cell: the unit's cells mark their first lanes, and the
    // largest mark up to a lane is its cell
    lds.partner[lane] = 0u;
    wave_lds_sync();
    if (in_unit) {
      lds.start[lane] = incl - nl - base;
      lds.cnt[lane] = nl;
      lds.partner[incl - nl - base] = lane;
      cnt_pairs += nl * (nl - 1u) / 2u;
    }
    wave_lds_sync();
    const bool mine = lane < p;
    const uint32_t mark = wave_inclusive_max(lds.partner[lane]);
    const uint32_t cl = mine ? mark : 0u;
    const uint32_t st = mine ? lds.start[cl] : 0u;
    const uint32_t n = mine ? lds.cnt[cl] : 0u;
    const uint32_t gl = lane - st;
    const uint32_t c = c0 + cl;
    {
      uint32_t id = kNone;
      if (mine) {
        const size_t o = (size_t)c * src.cap + gl;
        const Particle q = load_particle(src.st, o);
        lds.x[lane] = q.x;
        lds.y[lane] = q.y;
        lds.z[lane] = q.z;
        lds.px[lane] = q.px;  // by lane until ranked
        lds.py[lane] = q.py;
        lds.pz[lane] = q.pz;
        id = q.id;
      }
      lds.id[lane] = id;
    }
    // canonical rank among the cell's ids; the momenta move to their
    // canonical positions
    uint32_t pos;
    {
      const uint32_t id = lds.id[lane];
      const uint32_t maxn = wave_max(n);
      uint32_t r = 0;
      wave_lds_sync();
      for (uint32_t m = 0; m < maxn; ++m)
        if (m < n) r += lds.id[st + m] < id ? 1u : 0u;
      pos = st + r;
      const double qx = lds.px[lane], qy = lds.py[lane], qz = lds.pz[lane];
      wave_lds_sync();
      if (mine) {
        lds.px[pos] = qx;
        lds.py[pos] = qy;
        lds.pz[pos] = qz;
        if (kTrace && tr.perm) tr.perm[tr.offsets[c] + r] = id;
      }
    }
    wave_lds_sync();

    // pair tests, the w1 filter first, in passes that fill the list; then
    // the exact test and claims of the list by rows
    uint64_t claimed = 0;
    uint32_t nclaim = 0;
    if (pa.any) {
      const uint32_t npairs = n * (n - 1u) / 2u;
      uint32_t k = gl;
      while (__ballot(k < npairs) != 0) {
        uint32_t nf = 0;
        __builtin_amdgcn_s_setprio(0);
        do {
          const bool pass = k < npairs &&
                            philox10_w1(k, c, t, 0u, pa.key0, pa.key1) <= pa.w1_max;
          const uint64_t mk = __ballot(pass);
          if (pass) lds.filt[nf + (uint32_t)__popcll(mk & below)] = cl << 16 | k;
          nf += (uint32_t)__popcll(mk);
          k += n;
        } while (nf <= kPackedFilt - 64u && __ballot(k < npairs) != 0);
        __builtin_amdgcn_s_setprio(1);
        wave_lds_sync();
        for (uint32_t i0 = 0; i0 < nf; i0 += 64u)
          packed_resolve_row<kTrace>(i0, nf, c0, t, pa, lds, claimed, nclaim, n_acc, tr,
                                     status);
        wave_lds_sync();
      }
    }
    n_claims += nclaim;

    // kinematics of the claimed pairs, in both lanes of each
    double px = lds.px[pos], py = lds.py[pos], pz = lds.pz[pos];
    const bool scat = mine && ((claimed >> pos) & 1ull) != 0;
    if (scat) {
      const uint32_t other = lds.partner[pos];
      const bool lo = pos < other;
      const uint32_t A = lo ? pos : other, B = lo ? other : pos;
      const uint32_t ra = A - st, rb = B - st;
      const uint32_t k = row_start(ra, n) + (rb - ra - 1u);
      const Words4 w = philox10(k, c, t, 1u, pa.key0, pa.key1);
      double ax = lds.px[A], ay = lds.py[A], az = lds.pz[A];
      double bx = lds.px[B], by = lds.py[B], bz = lds.pz[B];
      scatter_pair(ax, ay, az, bx, by, bz, uniform53(w.w0, w.w1), uniform53(w.w2, w.w3));
      px = lo ? ax : bx;
      py = lo ? ay : by;
      pz = lo ? az : bz;
      if (!kFused) {
        put_momentum(src.st, (size_t)c * src.cap + gl, px, py, pz);
      }
    }
    if (obs) {
      // the cells' sums (kCellSums), one cell a lane, from the terms of its
      // particles, which take the momenta's place in LDS
      wave_lds_sync();
      if (mine) {
        double se = 0.0, sp = 0.0, sxx = 0.0;
        obs_add(px, py, pz, se, sp, sxx);
        lds.px[lane] = se;
        lds.py[lane] = sp;
        lds.pz[lane] = sxx;
      }
      wave_lds_sync();
      if (in_unit) {
        double se = 0.0, sp = 0.0, sxx = 0.0;
        const uint32_t first = incl - nl - base;
        for (uint32_t j = first; j < first + nl; ++j) {
          se += lds.px[j];
          sp += lds.py[j];
          sxx += lds.pz[j];
        }
        double *const out = obs + kCellSums * (size_t)cc;
        out[0] = se;
        out[1] = sp;
        out[2] = sxx;
        out[3] = (double)nl;
      }
    }
    if (kFused) {
      double x = 0, y = 0, z = 0;
      uint32_t c2 = 0, id = 0;
      if (mine) {
        const Geometry g_l = g;
        x = lds.x[lane];
        y = lds.y[lane];
        z = lds.z[lane];
        id = lds.id[lane];
        advance<true>(g_l, x, y, z, px, py, pz);
        c2 = cell_id(g_l, x, y, z);
      }
      append_table(dst, c2, mine, Particle{x, y, z, px, py, pz, id}, status, lds.tab);
    }
    base = end;
  }
  // work counters of the wave's units, in one slot
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) cnt_pairs += __shfl_down(cnt_pairs, s);
  if (lane == 0 && cnt_pairs != 0) {
    const uint32_t slot = c0 % kCounterSlots;
    atomicAdd(&status->pairs[slot], (unsigned long long)cnt_pairs);
    atomicAdd(&status->cand[slot], (unsigned long long)n_acc);
    atomicAdd(&status->claims[slot], (unsigned long long)n_claims);
  }
  if (kLarge && large) {
    for (uint64_t big = left_out; big != 0; big &= big - 1ull)
      if (unit++ % kPackedWaves == wave)
        cell_step<kFused, kTrace, kSmallCap, false, kMid>(src, dst,
                                                          c0 + (uint32_t)__builtin_ctzll(big), t,
                                                          pa, g, status, tr, wlds.cell, obs);
  }
}

// dst is src shifted by dst_shift bytes and g is read from device memory
// where the binning uses it (as for k_step: fewer values held through the
// loops).  Five waves per SIMD: the compiler's choice (4, 101-104 VGPRs)
// made the 32^3 fm^3 set's fused step 5 % slower, six (80 VGPRs, 12
// spilled) 4 %.
template <bool kFused, bool kTrace, bool kLarge, bool kMid>
__global__ __launch_bounds__(64 * kPackedWaves) __attribute__((amdgpu_waves_per_eu(5))) void k_step_packed(
    Cells src_arg, int64_t dst_shift, uint32_t n_cells, uint32_t tile, uint32_t t, PairArgs pa,
    const Geometry *__restrict__ gp, DevStatus *status, TraceArgs tr) {
  const GCells src = binning(to_global(src_arg), t);
  __shared__ PackedWaveLds<kFused> lds[kPackedWaves];
  const uint32_t c0 = xcd_runs<8>(blockIdx.x, gridDim.x) * tile;
  const uint32_t c_end = min(c0 + tile, n_cells);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64u));
  packed_cells_step<kFused, kTrace, kLarge, kMid>(src, dst_of(src, dst_shift, t), c0, c_end, t, pa,
                                            *gp, status, tr, lds[wave], wave, true);
}

// One wave per 64 consecutive cells: the cells that the packed launch left.
template <bool kFused, bool kTrace, uint32_t kCap, bool kMid>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_step_large(
    Cells src_arg, Cells dst_arg, uint32_t n_cells,
                                                   uint32_t t, PairArgs pa,
                                                   Geometry g, DevStatus *status,
                                                   TraceArgs tr) {
  const GCells src = binning(to_global(src_arg), t);
  const GCells dst = binning(to_global(dst_arg), t + 1u);
  __shared__ CellLds<kFused, kCap> lds;
  const uint32_t c0 = blockIdx.x * 64u;
  const uint32_t c_end = c0 + 64u < n_cells ? c0 + 64u : n_cells;
  large_cells_step<kFused, kTrace, kCap, kMid>(src, dst, c0, c_end, t, pa, g, status, tr, lds);
}

// One wave per cell, for the cells that the packed launch left when they are
// common (a wave that scans 64 of them would step them one after another).
template <bool kFused, bool kTrace, uint32_t kCap, bool kMid>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(cell_waves<kCap>()))) void k_step_over(
    Cells src_arg, int64_t dst_shift,
                                                  uint32_t t, PairArgs pa,
                                                  const Geometry *__restrict__ gp,
                                                  DevStatus *status, TraceArgs tr) {
  const GCells src = binning(to_global(src_arg), t);
  __shared__ CellLds<kFused, kCap> lds;
  const uint32_t c = xcd_runs<8>(blockIdx.x, gridDim.x);
  const uint32_t cnt = src.count[c];
  if (cnt <= kPackedMax && cnt <= src.cap) return;
  cell_step<kFused, kTrace, kCap, true, kMid>(src, dst_of(src, dst_shift, t), c, t, pa, *gp, status, tr,
                                  lds);
}

// dst is src shifted by dst_shift bytes (the two buffers of a context are
// laid out alike), and g is read from device memory where the binning uses
// it: as kernel arguments both would be loaded at entry and held through the
// pair loop, which spills scalar registers into vector lanes and reloads them
// in the loop.  Derived from src, the dst pointers stay known to address
// global memory.
template <bool kFused, uint32_t kCap, bool kMid>
__global__ __launch_bounds__(64 * kGroup) __attribute__((amdgpu_waves_per_eu(cell_waves<kCap>()))) void k_step_group(
    Cells src_arg, int64_t dst_shift, uint32_t n_cells, uint32_t t, PairArgs pa,
    const Geometry *__restrict__ gp, DevStatus *status) {
  const GCells src = binning(to_global(src_arg), t);
  __shared__ CellLds<kFused, kCap> lds[kGroup];
  __shared__ GroupLds<kGroup> q;
  group_cells_step<kFused, kCap, kGroup, kMid>(src, dst_of(src, dst_shift, t),
                                         xcd_runs<2>(blockIdx.x, gridDim.x) * kGroup, n_cells, t,
                                         pa, *gp, status, q, lds, nullptr);
}

template <bool kFused, bool kTrace, uint32_t kCap, bool kMid>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(cell_waves<kCap>()))) void k_step(
    Cells src_arg, int64_t dst_shift, uint32_t t,
                                             PairArgs pa, const Geometry *__restrict__ gp,
                                             DevStatus *status, TraceArgs tr) {
  const GCells src = binning(to_global(src_arg), t);
  __shared__ CellLds<kFused, kCap> lds;
  cell_step<kFused, kTrace, kCap, true, kMid>(src, dst_of(src, dst_shift, t),
                                  xcd_runs<8>(blockIdx.x, gridDim.x), t, pa, *gp, status, tr,
                                  lds);
}

// ---------------------------------------------------------------------------
// Several waves per cell, for boxes of few dense cells, where one wave per
// cell leaves most SIMDs idle and the step is one cell's chain of phases.
// A workgroup of kW waves:
//   1. loads every particle into registers (kCap / 64 kW per thread; the
//      slots' loads do not wait for the count, with kSome only those of the
//      first `ahead` slots), ids into LDS;
//   2. ranks the ids and stores the momenta in canonical order in LDS, where
//      the later phases read them: no further global load;
//   3. tests the pairs in rounds: wave w filters the w-th of kW consecutive
//      ranges (Philox w1) into its own list and keeps in it those that the
//      exact test accepts; then the first wave claims from the lists in
//      order, so that the claims run in increasing pair order as with one
//      wave.  A range is half as long as fills its list on average; should a
//      list fill all the same, the first wave tests the rest of that range
//      itself;
//   4. with each row of claims the first wave computes their kinematics, in
//      the lanes that hold them, in place (a member is claimed once, but a
//      later round still tests with its momentum from before: so where there
//      are several rounds, or a list filled, the claims are listed and the
//      kinematics follow the last one);
//   5. fused: streams and bins each particle from its registers; else writes
//      the scattered momenta back.
// Cells whose members are not all in their block go to the one-wave path.
// ---------------------------------------------------------------------------
constexpr uint32_t kWideFilt = 256;  // filtered pairs of a wave's list
template <bool kFused, uint32_t kCap, uint32_t kW>
struct WideLds {
  CellLds<kFused, kCap> cell;  // ids, rank scratch, claims (and the one-wave path)
  double px[kCap], py[kCap], pz[kCap];  // by canonical position
  uint32_t filt[kW][kWideFilt];
  uint32_t n_filt[kW], k_resume[kW];
  uint32_t claimed[kCap / 32];  // flags by canonical position
  uint32_t dir[54];
  uint32_t n_claim;
};

// Exact test of the nf pairs in filt (one wave): the accepted ones, as
// a << 10 | b, move to its front in order; returns their number.
template <typename Lds>
__device__ __forceinline__ uint32_t wide_exact(uint32_t nf, uint32_t *filt, const Lds &lds,
                                               uint32_t c, uint32_t n, uint32_t t,
                                               const PairArgs &pa) {
  uint32_t kept = 0;
  for (uint32_t i0 = 0; i0 < nf; i0 += 64u) {
    const uint32_t i = i0 + lane_id();
    bool acc = false;
    uint32_t a = 0, b = 0;
    if (i < nf) {
      const uint32_t k = filt[i];
      const Words4 w = philox10(k, c, t, 0u, pa.key0, pa.key1);
      pair_of_index(k, n, a, b);
      acc = uniform53(w.w0, w.w1) < p22(lds.px[a], lds.py[a], lds.pz[a], lds.px[b], lds.py[b],
                                        lds.pz[b], pa.kfac);
    }
    wave_lds_sync();
    const uint64_t m = __ballot(acc);
    if (acc) filt[kept + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1ull))] = a << 10 | b;
    kept += (uint32_t)__popcll(m);
  }
  wave_lds_sync();
  return kept;
}

// New momenta of the pair (a, b) of cell c, in place.
template <typename Lds>
__device__ __forceinline__ void wide_scatter(uint32_t a, uint32_t b, Lds &lds, uint32_t c,
                                             uint32_t n, uint32_t t, const PairArgs &pa) {
  const Words4 w = philox10(row_start(a, n) + (b - a - 1u), c, t, 1u, pa.key0, pa.key1);
  double ax = lds.px[a], ay = lds.py[a], az = lds.pz[a];
  double bx = lds.px[b], by = lds.py[b], bz = lds.pz[b];
  scatter_pair(ax, ay, az, bx, by, bz, uniform53(w.w0, w.w1), uniform53(w.w2, w.w3));
  lds.px[a] = ax;
  lds.py[a] = ay;
  lds.pz[a] = az;
  lds.px[b] = bx;
  lds.py[b] = by;
  lds.pz[b] = bz;
}

// Claims of a row of accepted pairs, one a lane (a << 10 | b; `have`: the
// lane holds one), in lane order, by one wave: of those whose members are
// free the first is taken and its members' others dropped, until none is
// left.  Returns the lanes that won.
template <typename Lds>
__device__ __forceinline__ uint64_t wide_claim_row(uint32_t v, bool have, Lds &lds) {
  const uint32_t a = v >> 10, b = v & 1023u;
  bool open = have && ((lds.claimed[a >> 5] >> (a & 31u)) & 1u) == 0u &&
              ((lds.claimed[b >> 5] >> (b & 31u)) & 1u) == 0u;
  uint64_t won = 0;
  for (uint64_t m = __ballot(open); m != 0; m = __ballot(open)) {
    const uint32_t l = (uint32_t)__builtin_ctzll(m);
    const uint32_t vl = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
    const uint32_t la = vl >> 10, lb = vl & 1023u;
    won |= 1ull << l;
    open = open && a != la && a != lb && b != la && b != lb;
  }
  if ((won >> lane_id()) & 1ull) {
    atomicOr(&lds.claimed[a >> 5], 1u << (a & 31u));
    atomicOr(&lds.claimed[b >> 5], 1u << (b & 31u));
  }
  wave_lds_sync();
  return won;
}

// Claims of a whole list, appended to claims.
template <typename Lds>
__device__ __forceinline__ void wide_claim(uint32_t na, const uint32_t *list, Lds &lds,
                                           uint32_t *claims, uint32_t &nclaim) {
  const uint32_t lane = lane_id();
  for (uint32_t i0 = 0; i0 < na; i0 += 64u) {
    const uint32_t v = i0 + lane < na ? list[i0 + lane] : 0u;
    const uint64_t won = wide_claim_row(v, i0 + lane < na, lds);
    if ((won >> lane) & 1ull)
      claims[nclaim + (uint32_t)__popcll(won & ((1ull << lane) - 1ull))] = v;
    nclaim += (uint32_t)__popcll(won);
  }
}

template <bool kFused, uint32_t kCap, uint32_t kW, bool kSome>
__device__ __forceinline__ void wide_cell_step(const GCells &src, const GCells &dst, uint32_t c,
                                               uint32_t ahead, uint32_t t, const PairArgs &pa,
                                               const Geometry &g, DevStatus *status,
                                               WideLds<kFused, kCap, kW> &lds) {
  constexpr uint32_t kT = 64u * kW, kPer = kCap / kT;
  static_assert(kPer * kT == kCap && kCap <= kCellCap, "whole particles per thread");
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / 64u));
  const size_t base = (size_t)c * src.cap;
  Particle q[kPer];
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    q[i] = Particle{};
    if (tid + i * kT < (kSome ? ahead : src.cap)) q[i] = load_particle(src.st, base + tid + i * kT);
  }
  const uint32_t n = src.count[c];
  if (n > src.cap) {
    if (wv == 0)
      cell_step<kFused, false, kCap, false>(src, dst, c, t, pa, g, status, TraceArgs{}, lds.cell);
    return;
  }
  if (c == 0 && tid == 0) clear_idle_scratch(src, t);
  if (kSome && __builtin_expect(n > ahead, 0)) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t j = tid + i * kT;
      if (j >= ahead && j < n) q[i] = load_particle(src.st, base + j);
    }
  }

  // ids to LDS, padded to a multiple of 4 with an id no particle has
  uint32_t *const s_id = lds.cell.buf;
  const uint32_t n4 = (n + 3u) & ~3u;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    const uint32_t j = tid + i * kT;
    if (j < n4) s_id[j] = j < n ? q[i].id : 0xFFFFFFFFu;
  }
  for (uint32_t w = tid; w < kCap / 32u; w += kT) lds.claimed[w] = 0u;
  if (tid < 27u) lds.dir[tid] = 0u;
  __syncthreads();
  // canonical position: every thread counts the smaller ids (up to kCountMax
  // members), else by buckets of the id as in cell_step
  constexpr uint32_t kCountMax = 256;
  uint32_t rank[kPer];
  if (n <= kCountMax) {
    const uint4 *const s_id4 = reinterpret_cast<const uint4 *>(s_id);
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t me = q[i].id;
      uint32_t r = 0;
      if (tid + i * kT < n)
#pragma unroll 4
        for (uint32_t m = 0; m < n4 / 4u; ++m) {
          const uint4 v = s_id4[m];
          r += (v.x < me) + (v.y < me) + (v.z < me) + (v.w < me);
        }
      rank[i] = r;
    }
  } else {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (uint32_t j = lane; j < n; j += 64u) {
      lo = min(lo, s_id[j]);
      hi = max(hi, s_id[j]);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    const uint32_t bits = 32u - (uint32_t)__builtin_clz(hi - lo);
    const uint32_t shift = bits > 8u ? bits - 8u : 0u;
    uint32_t *const s_bkt = lds.cell.bkt;
    for (uint32_t b = tid; b < kRankBuckets; b += kT) s_bkt[b] = 0u;
    if (tid == 0) s_bkt[kRankBuckets] = n;
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i)
      if (tid + i * kT < n) atomicAdd(&s_bkt[(q[i].id - lo) >> shift], 1u);
    __syncthreads();
    if (wv == 0) {  // ends of the buckets
      uint4 v = reinterpret_cast<uint4 *>(s_bkt)[lane];
      v.y += v.x;
      v.z += v.y;
      v.w += v.z;
      const uint32_t excl = wave_inclusive_sum(v.w) - v.w;
      v.x += excl;
      v.y += excl;
      v.z += excl;
      v.w += excl;
      reinterpret_cast<uint4 *>(s_bkt)[lane] = v;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i)
      if (tid + i * kT < n)
        lds.cell.sorted[atomicSub(&s_bkt[(q[i].id - lo) >> shift], 1u) - 1u] = q[i].id;
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      rank[i] = 0;
      if (tid + i * kT < n) {
        const uint32_t b = (q[i].id - lo) >> shift, p1 = s_bkt[b + 1u];
        uint32_t r = s_bkt[b];
        for (uint32_t p = r; p < p1; ++p) r += lds.cell.sorted[p] < q[i].id ? 1u : 0u;
        rank[i] = r;
      }
    }
  }
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i)
    if (tid + i * kT < n) {
      lds.px[rank[i]] = q[i].px;
      lds.py[rank[i]] = q[i].py;
      lds.pz[rank[i]] = q[i].pz;
    }
  __syncthreads();

  uint32_t *const claims = lds.cell.buf;  // the ids' buffer; at most n / 2 claims
  const uint32_t npairs = n > 1u ? n * (n - 1u) / 2u : 0u;
  uint32_t nclaim = 0, n_acc = 0, listed = 0;
  if (pa.any && npairs != 0u) {
    CellView cv{};
    cv.c = c;
    cv.n = n;
    cv.t = t;
    // pairs of a wave's range: an equal share, at most what fills half its
    // list on average, whole rows of two
    const float full = 0.5f * (float)kWideFilt * 0x1p32f / ((float)pa.w1_max + 1.0f);
    const uint32_t room = max(128u, (uint32_t)min(full, 1e6f) & ~127u);
    const uint32_t range = min(room, (npairs + 128u * kW - 1u) / (128u * kW) * 128u);
    for (uint32_t k0 = 0; k0 < npairs; k0 += kW * range) {
      const uint32_t kb = min(k0 + wv * range, npairs), ke = min(kb + range, npairs);
      uint32_t nf = 0, none = 0, no_bits = 0, unused = 0;
      const uint32_t stop = test_pairs<false, false, false, kWideFilt>(
          kb, ke, cv, pa, src.st, nullptr, lds.filt[wv], nf, nullptr, none, no_bits, unused,
          TraceArgs{}, status);
      wave_lds_sync();
      const uint32_t na = wide_exact(nf, lds.filt[wv], lds, c, n, t, pa);
      n_acc += na;
      if (lane == 0) {
        lds.n_filt[wv] = na;
        lds.k_resume[wv] = stop;
      }
      __syncthreads();
      if (wv == 0) {
        const uint32_t cnt = lane < kW ? lds.n_filt[lane] : 0u;
        const uint32_t end = min(k0 + (lane + 1u) * range, npairs);
        const bool whole = __ballot(lane < kW && lds.k_resume[lane] < end) == 0ull;
        if (whole && npairs <= kW * range) {
          // the only round: rows of 64 over all the lists
          const uint32_t incl = wave_inclusive_sum(cnt);
          const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
          for (uint32_t i0 = 0; i0 < total; i0 += 64u) {
            const uint32_t i = i0 + lane;
            uint32_t w = 0, first = 0;  // the list holding entry i, its first entry
#pragma unroll
            for (uint32_t u = 0; u + 1u < kW; ++u) {
              const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)u);
              if (i >= e) {
                w = u + 1u;
                first = e;
              }
            }
            const uint32_t v = i < total ? lds.filt[w][i - first] : 0u;
            const uint64_t won = wide_claim_row(v, i < total, lds);
            nclaim += (uint32_t)__popcll(won);
            if ((won >> lane) & 1ull) wide_scatter(v >> 10, v & 1023u, lds, c, n, t, pa);
          }
        } else {
          for (uint32_t w = 0; w < kW; ++w) {
            wide_claim(lds.n_filt[w], lds.filt[w], lds, claims, listed);
            // a list that filled: the rest of its range
            const uint32_t to = min(k0 + (w + 1u) * range, npairs);
            for (uint32_t k = lds.k_resume[w]; k < to;) {
              uint32_t more = 0;
              k = test_pairs<false, false, false, kWideFilt>(k, to, cv, pa, src.st, nullptr,
                                                             lds.filt[w], more, nullptr, none,
                                                             no_bits, unused, TraceArgs{}, status);
              wave_lds_sync();
              more = wide_exact(more, lds.filt[w], lds, c, n, t, pa);
              n_acc += more;
              wide_claim(more, lds.filt[w], lds, claims, listed);
            }
          }
        }
        if (lane == 0) lds.n_claim = listed;
      }
      __syncthreads();
    }
    listed = lds.n_claim;
  }
  if (lane == 0) {
    const uint32_t slot = c % kCounterSlots;
    if (n_acc != 0u) atomicAdd(&status->cand[slot], (unsigned long long)n_acc);
    if (wv == 0) {
      atomicAdd(&status->pairs[slot], (unsigned long long)npairs);
      atomicAdd(&status->claims[slot], (unsigned long long)(nclaim + listed));
    }
  }
  if (listed != 0u) {
    for (uint32_t i = tid; i < listed; i += kT)
      wide_scatter(claims[i] >> 10, claims[i] & 1023u, lds, c, n, t, pa);
    __syncthreads();
  }
  if (!kFused) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t r = rank[i];
      if (tid + i * kT < n && ((lds.claimed[r >> 5] >> (r & 31u)) & 1u))
        put_momentum(src.st, base + tid + i * kT, lds.px[r], lds.py[r], lds.pz[r]);
    }
    return;
  }
  // streaming and binning: slots by direction of move, numbered over the
  // whole workgroup (as neighbour_fetch_add does for a wave)
  const uint32_t sy = (uint32_t)g.n[2], sx = (uint32_t)g.n[1] * sy;
  const int32_t cx = (int32_t)(c / sx), cy = (int32_t)(c % sx / sy), cz = (int32_t)(c % sy);
  uint32_t c2[kPer], dir[kPer], order[kPer];
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    dir[i] = 27u;  // none
    c2[i] = order[i] = 0u;
    if (tid + i * kT < n) {
      const uint32_t r = rank[i];
      q[i].px = lds.px[r];
      q[i].py = lds.py[r];
      q[i].pz = lds.pz[r];
      advance<true>(g, q[i].x, q[i].y, q[i].z, q[i].px, q[i].py, q[i].pz);
      int32_t ix, iy, iz;
      cell_axes(g, q[i].x, q[i].y, q[i].z, ix, iy, iz);
      c2[i] = (uint32_t)((ix * g.n[1] + iy) * g.n[2] + iz);
      const int32_t dx = ix - cx, dy = iy - cy, dz = iz - cz;
      dir[i] = 28u;  // not a neighbour
      if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1) {
        dir[i] = (uint32_t)(9 * (dx + 1) + 3 * (dy + 1) + (dz + 1));
        order[i] = atomicAdd(&lds.dir[dir[i]], 1u);
      }
    }
  }
  __syncthreads();
  if (tid < 27u && lds.dir[tid] != 0u) {
    const int32_t dx = (int32_t)(tid / 9u) - 1, dy = (int32_t)(tid / 3u % 3u) - 1,
                  dz = (int32_t)(tid % 3u) - 1;
    const uint32_t key = (uint32_t)((int32_t)c + dx * (int32_t)sx + dy * (int32_t)sy + dz);
    lds.dir[27u + tid] = atomic_add(dst.count + key, lds.dir[tid]);
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    if (dir[i] < 27u) store_particle(dst, c2[i], lds.dir[27u + dir[i]] + order[i], q[i], status);
    if (__ballot(dir[i] == 28u) != 0ull) append(dst, c2[i], dir[i] == 28u, q[i], status);
  }
  if (tid == 0) src.count[c] = 0u;
}

// Waves per SIMD: four waves a cell with four particles a thread would take
// 133 VGPRs and three waves, which leaves the last of 900 cells for a second
// round (900 cells of 40 in blocks of 600: 15.8 -> 12.5 us a step).
template <uint32_t kCap, uint32_t kW>
constexpr int wide_min_waves() {
  return kCap / (64u * kW) == 4u ? 4 : (int)(kW / 4u);
}

template <bool kFused, uint32_t kCap, uint32_t kW, bool kSome>
__global__ __launch_bounds__(64 * kW) __attribute__((amdgpu_waves_per_eu(wide_min_waves<kCap, kW>()))) void k_step_wide(Cells src_arg, int64_t dst_shift,
                                                       uint32_t ahead, uint32_t t, PairArgs pa,
                                                       const Geometry *__restrict__ gp,
                                                       DevStatus *status) {
  const GCells src = binning(to_global(src_arg), t);
  __shared__ WideLds<kFused, kCap, kW> lds;
  const Geometry g = *gp;
  wide_cell_step<kFused, kCap, kW, kSome>(src, dst_of(src, dst_shift, t),
                                   xcd_runs<8>(blockIdx.x, gridDim.x), ahead, t, pa, g,
                                   status, lds);
}

// ---------------------------------------------------------------------------
// Batched steps: all live events of a batch advance together.  Each kernel
// has a work space in which the events are laid out one after another
// (space_begin[e] = the first unit of event e, ascending from 0):
//   items   cpi consecutive cells, for the binning (every event); a wave
//           takes items with a grid stride, so a grid smaller than the item
//           count is a persistent launch;
//   tiles   `tile` cells, a workgroup each, for the events with lanes per
//           cell > 0, which are stepped in packed units;
//   scans   64 cells, one wave each, stepping the cells that the units leave
//           out, for those of these events whose blocks exceed the small LDS;
//   cells   one cell per wave, for events stepped one wave per cell;
//   groups  kGroup cells, a workgroup each, for those of these events whose
//           waves share their cells' pairs.
// The step kernels have no loop over units: a loop keeps the descriptor and
// lane constants live across iterations, which costs registers and with
// them the occupancy that hides memory latency.  Within a run of k steps,
// launch j (0: stream + bin, 1..k-1: fused, k: collisions only) reads buffer
// cur ^ (j & 1) of each event and uses step index t + j - 1; the run ends
// with k_batch_advance.
// ---------------------------------------------------------------------------
// The event of `unit` in a work space: the number of entries of begin[]
// that are <= unit, minus one (begin[] is ascending from 0; an event with
// no units has the begin of the next one, so it is never the answer).  Each
// lane counts the entries lane, lane + 64, ... (independent loads, no
// cross-lane step inside the loop, so they are all in flight together),
// then the wave sums the counts.  `unit` must be the same in every lane of
// the wave; so is the result.
__device__ __forceinline__ uint32_t find_event(const uint32_t *__restrict__ begin,
                                               uint32_t n_events, uint32_t unit) {
  uint32_t count = 0;
#pragma unroll 4
  for (uint32_t e = lane_id(); e < n_events; e += 64) count += begin[e] <= unit ? 1u : 0u;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) count += (uint32_t)__shfl_xor((int)count, o);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)count) - 1u;
}

// The event's fields for launch j of a run, loaded once into registers (the
// kernels store to global memory, so fields read through the table would
// be reloaded after every store).
struct EventView {
  GCells src, dst;
  Geometry g;
  PairArgs pa;
  DevStatus *status;
  uint32_t t, n_cells;
};

__device__ __forceinline__ EventView event_view(const BatchEvent *__restrict__ E, uint32_t j) {
  EventView v;
  if ((E->cur ^ (j & 1u)) == 0u) {
    v.src = to_global(E->buf[0]);
    v.dst = to_global(E->buf[1]);
  } else {
    v.src = to_global(E->buf[1]);
    v.dst = to_global(E->buf[0]);
  }
  v.g = E->g;
  v.pa = E->pa;
  v.status = E->status;
  v.t = E->t + j - 1u;
  v.src = binning(v.src, v.t);
  v.dst = binning(v.dst, v.t + 1u);
  v.n_cells = E->n_cells;
  return v;
}

// Where launch j of a run writes the event's observation sums: its per-cell
// sums array if the step the launch collides (t + j - 1) ends an
// observation interval, else nowhere.
__device__ __forceinline__ double *obs_target(const BatchEvent *__restrict__ E, uint32_t j) {
  const uint32_t every = E->obs_every;
  return every != 0u && (E->t + j) % every == 0u ? E->obs_sums : nullptr;
}

__global__ __launch_bounds__(kBlock) void k_batch_bin(const BatchEvent *__restrict__ ev,
                                                      const uint32_t *__restrict__ item_begin,
                                                      uint32_t n_events, uint32_t n_items) {
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // wave-uniform
  __shared__ SlotTable tab[kCellsPerBlock];
  for (uint32_t item = blockIdx.x * kCellsPerBlock + w; item < n_items;
       item += gridDim.x * kCellsPerBlock) {
    const BatchEvent *__restrict__ E = ev + find_event(item_begin, n_events, item);
    GCells src, dst;
    if (E->cur == 0u) {
      src = to_global(E->buf[0]);
      dst = to_global(E->buf[1]);
    } else {
      src = to_global(E->buf[1]);
      dst = to_global(E->buf[0]);
    }
    src = binning(src, E->t - 1u);
    dst = binning(dst, E->t);
    if (item == E->item_begin && lane_id() == 0) clear_idle_spill_set(src);
    const Geometry g = E->g;
    DevStatus *const status = E->status;
    const uint32_t cpi = E->cpi, n_cells = E->n_cells, lanes = E->lanes;
    const uint32_t c0 = (item - E->item_begin) * cpi;
    const uint32_t c1 = c0 + cpi < n_cells ? c0 + cpi : n_cells;
    switch (lanes) {
      case 8:
        for (uint32_t c = c0; c < c1; c += 8) cells_stream_bin<8>(src, dst, c, c1, g, status, nullptr, tab[w]);
        break;
      case 16:
        for (uint32_t c = c0; c < c1; c += 4) cells_stream_bin<16>(src, dst, c, c1, g, status, nullptr, tab[w]);
        break;
      case 32:
        for (uint32_t c = c0; c < c1; c += 2) cells_stream_bin<32>(src, dst, c, c1, g, status, nullptr, tab[w]);
        break;
      default:
        for (uint32_t c = c0; c < c1; ++c) cells_stream_bin<64>(src, dst, c, c + 1, g, status, nullptr, tab[w]);
    }
  }
}

// Packed cells: a workgroup per tile of the event's `tile` cells.  The cells
// that the units leave out are stepped here too where their blocks fit the
// small LDS, else by k_batch_step_scan.
template <bool kFused>
__global__ __launch_bounds__(64 * kPackedWaves) __attribute__((amdgpu_waves_per_eu(5))) void k_batch_step_packed(
    const BatchEvent *__restrict__ ev, const uint32_t *__restrict__ tile_begin,
    uint32_t n_events, uint32_t j) {
  __shared__ PackedWaveLds<kFused> lds[kPackedWaves];
  const uint32_t unit = xcd_runs<8>(blockIdx.x, gridDim.x);
  const BatchEvent *__restrict__ E = ev + find_event(tile_begin, n_events, unit);
  const uint32_t s = (E->cur ^ (j & 1u)) & 1u;
  const uint32_t t = E->t + j - 1u;
  const GCells src = binning(to_global(E->buf[s]), t);
  const int64_t shift = (const char *)E->buf[s ^ 1u].st.rec - (const char *)E->buf[s].st.rec;
  const PairArgs pa = E->pa;
  const uint32_t c0 = (unit - E->tile_begin) * E->tile;
  const uint32_t c_end = min(c0 + E->tile, E->n_cells);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64u));
  packed_cells_step<kFused, false, true, false>(src, dst_of(src, shift, t), c0, c_end, t, pa, E->g,
                                         E->status, TraceArgs{}, lds[wave], wave,
                                         src.cap <= kSmallCap, obs_target(E, j));
}

// The cells of 64 consecutive cells of a packed event with blocks of more
// than kSmallCap slots that its units left out, by the whole wave.
template <bool kFused>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_batch_step_scan(
    const BatchEvent *__restrict__ ev, const uint32_t *__restrict__ scan_begin,
    uint32_t n_events, uint32_t j) {
  __shared__ CellLds<kFused, kCellCap> lds;
  const uint32_t unit = blockIdx.x;
  const BatchEvent *__restrict__ E = ev + find_event(scan_begin, n_events, unit);
  const EventView v = event_view(E, j);
  const uint32_t c0 = (unit - E->scan_begin) * 64u;
  const uint32_t c1 = c0 + 64u < v.n_cells ? c0 + 64u : v.n_cells;
  large_cells_step<kFused, false, kCellCap>(v.src, v.dst, c0, c1, v.t, v.pa, v.g, v.status,
                                            TraceArgs{}, lds, obs_target(E, j));
}

// One wave per cell of the events stepped one wave per cell, held to the
// register budget of the plain kernel (cell_waves).
template <bool kFused, uint32_t kCap>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(cell_waves<kCap>()))) void k_batch_step_cells(
    const BatchEvent *__restrict__ ev,
                                                         const uint32_t *__restrict__ cell_begin,
                                                         uint32_t n_events, uint32_t j) {
  __shared__ CellLds<kFused, kCap> lds;
  const uint32_t unit = xcd_runs<8>(blockIdx.x, gridDim.x);
  const BatchEvent *__restrict__ E = ev + find_event(cell_begin, n_events, unit);
  // dst is src shifted by the distance between the event's two buffers
  // (laid out alike), g is read by reference from the table where the
  // binning uses it (see k_step)
  const uint32_t s = (E->cur ^ (j & 1u)) & 1u;
  const uint32_t t = E->t + j - 1u;
  const GCells src = binning(to_global(E->buf[s]), t);
  const int64_t shift = (const char *)E->buf[s ^ 1u].st.rec - (const char *)E->buf[s].st.rec;
  const PairArgs pa = E->pa;
  cell_step<kFused, false, kCap>(src, dst_of(src, shift, t), unit - E->cell_begin, t,
                                 pa, E->g, E->status, TraceArgs{}, lds, obs_target(E, j));
}

// Groups of kGroup consecutive cells of the events whose waves share their
// cells' pairs.
template <bool kFused>
__global__ __launch_bounds__(64 * kGroup) __attribute__((amdgpu_waves_per_eu(cell_waves<kSmallCap>()))) void k_batch_step_group(
    const BatchEvent *__restrict__ ev, const uint32_t *__restrict__ group_begin,
    uint32_t n_events, uint32_t j) {
  __shared__ CellLds<kFused, kSmallCap> lds[kGroup];
  __shared__ GroupLds<kGroup> q;
  const uint32_t unit = xcd_runs<2>(blockIdx.x, gridDim.x);
  const BatchEvent *__restrict__ E = ev + find_event(group_begin, n_events, unit);
  const uint32_t s = (E->cur ^ (j & 1u)) & 1u;
  const uint32_t t = E->t + j - 1u;
  const GCells src = binning(to_global(E->buf[s]), t);
  const int64_t shift = (const char *)E->buf[s ^ 1u].st.rec - (const char *)E->buf[s].st.rec;
  const PairArgs pa = E->pa;
  group_cells_step<kFused, kSmallCap, kGroup, false>(src, dst_of(src, shift, t),
                                              (unit - E->cell_begin) * kGroup, E->n_cells, t, pa,
                                              E->g, E->status, q, lds, obs_target(E, j));
}

// End of a run of k steps: every event moved k buffers and k step indices.
__global__ void k_batch_advance(BatchEvent *ev, uint32_t n_events, uint32_t k) {
  const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n_events) {
    ev[e].cur ^= (k & 1u);
    ev[e].t += k;
  }
}

// ---------------------------------------------------------------------------
// Observe: per-cell sums of E and p_x, then per-slab sums over the slab's
// cells in cell order.  Slab ix is the contiguous cell range
// [ix ny nz, (ix+1) ny nz).
// ---------------------------------------------------------------------------
// G lanes per cell (8, 16, 32 or 64, by the mean occupancy: with a wave per
// cell the 2.1 M cells of the 32^3 fm^3 set took 746 us, now 285).
template <uint32_t G>
__global__ __launch_bounds__(kBlock) void k_observe_cells(Cells cur_arg, uint32_t n_cells,
                                                          double *cell_sums,
                                                          uint32_t binning_step) {
  const GCells cur = binning(to_global(cur_arg), binning_step);
  constexpr uint32_t kWaveCells = 64u / G;
  const uint32_t gl = lane_id() % G;
  const uint32_t c = (blockIdx.x * kBlock + threadIdx.x) / G;
  const uint32_t cnt = c < n_cells ? cur.count[c] : 0u;
  const uint32_t n = cnt < cur.cap ? cnt : cur.cap;
  const size_t base = (size_t)c * cur.cap;
  double se = 0.0, sp = 0.0, sxx = 0.0;
  for (uint32_t j = gl; j < n; j += G) {
    double px, py, pz;
    load_momentum(cur.st, base + j, px, py, pz);
    obs_add(px, py, pz, se, sp, sxx);
  }
  // overflowing cells: one scan of the spill slots by the whole wave, each hit
  // added in its cell's first lane (a scan by each cell's own G lanes: 357 us
  // for 321 538 particles, 8 689 of 160 000 cells overflowing, now 113)
  if (__ballot(cnt > cur.cap) != 0ull) {
    const SpillDesc *const spl = cur.sp;
    const uint32_t ns = min(spl->hdr[2u * cur.q], spl->capacity);
    const uint32_t first = c - lane_id() / G;  // the wave's first cell
    for (uint32_t i0 = 0; i0 < ns; i0 += 64u) {
      const uint32_t i = i0 + lane_id();
      const uint32_t at = i < ns ? spl->cell[i] - first : kWaveCells;
      double ve = 0.0, vp = 0.0, vxx = 0.0;
      if (at < kWaveCells) {
        double px, py, pz;
        load_momentum(cur.st, spl->base + i, px, py, pz);
        obs_add(px, py, pz, ve, vp, vxx);
      }
      for (uint64_t m = __ballot(at < kWaveCells); m != 0; m &= m - 1ull) {
        const int l = (int)__builtin_ctzll(m);
        const double te = __shfl(ve, l), tp = __shfl(vp, l), txx = __shfl(vxx, l);
        if (lane_id() == G * (uint32_t)__builtin_amdgcn_readlane((int)at, l)) {
          se += te;
          sp += tp;
          sxx += txx;
        }
      }
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    se += __shfl_xor(se, o);
    sp += __shfl_xor(sp, o);
    sxx += __shfl_xor(sxx, o);
  }
  if (gl == 0 && c < n_cells) {
    double *const out = cell_sums + kCellSums * (size_t)c;
    out[0] = se;
    out[1] = sp;
    out[2] = sxx;
    out[3] = (double)cnt;
  }
}

// The rest frame (Landau frame of the t-x block of T^{mu nu}) of a slab:
// T^mu_nu u^nu = e u^mu, u = gamma (1, v), in the order the determinism
// contract fixes (a product of two factors under the square root).
__device__ __forceinline__ void rest_frame(double t00, double t0x, double txx, double &e,
                                           double &v) {
  const double a = t00 + txx;
  const double b = 2.0 * __builtin_fabs(t0x);
  double disc = (a - b) * (a + b);
  if (disc < 0.0) disc = 0.0;
  e = ((t00 - txx) + __builtin_sqrt(disc)) / 2.0;
  const double den = e + txx;
  v = den > 0.0 ? t0x / den : 0.0;
}

// Slab ix's sums over its cells in cell order, then the moments (a
// workgroup of kBlock threads).
__device__ __forceinline__ void slab_moments(const double *cell_sums, uint32_t cells_per_slab,
                                             double vol, uint32_t ix, const SlabOut &out) {
  __shared__ double s_sum[kCellSums][kBlock / 64];
  const size_t c0 = (size_t)ix * cells_per_slab;
  double acc[kCellSums] = {0.0, 0.0, 0.0, 0.0};
  for (uint32_t j = threadIdx.x; j < cells_per_slab; j += kBlock)
#pragma unroll
    for (uint32_t k = 0; k < kCellSums; ++k) acc[k] += cell_sums[kCellSums * (c0 + j) + k];
#pragma unroll
  for (uint32_t k = 0; k < kCellSums; ++k)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_down(acc[k], o);
  const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
  if (lane == 0)
#pragma unroll
    for (uint32_t k = 0; k < kCellSums; ++k) s_sum[k][wave] = acc[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot[kCellSums];
#pragma unroll
    for (uint32_t k = 0; k < kCellSums; ++k) {
      tot[k] = 0.0;
      for (int w = 0; w < kBlock / 64; ++w) tot[k] += s_sum[k][w];
    }
    const double t00 = tot[0] / vol, t0x = tot[1] / vol, txx = tot[2] / vol;
    if (out.T00) out.T00[ix] = t00;
    if (out.T0x) out.T0x[ix] = t0x;
    if (out.Txx) out.Txx[ix] = txx;
    if (out.n) out.n[ix] = tot[3] / vol;
    if (out.e || out.v) {
      double e, v;
      rest_frame(t00, t0x, txx, e, v);
      if (out.e) out.e[ix] = e;
      if (out.v) out.v[ix] = v;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_observe_slabs(const double *cell_sums,
                                                          uint32_t cells_per_slab,
                                                          double vol, SlabOut out) {
  slab_moments(cell_sums, cells_per_slab, vol, blockIdx.x, out);
}

// The slabs of the events observed after launch j of a run: block (ix,
// event) sums slab ix of an event due for an observation (its cells' sums,
// written by the launch) into T00 and T0x of the observation's row.
__global__ __launch_bounds__(kBlock) void k_batch_observe(const BatchEvent *__restrict__ ev,
                                                          uint32_t n_events, uint32_t j) {
  const uint32_t e = blockIdx.y;
  if (e >= n_events) return;
  const BatchEvent *__restrict__ E = ev + e;
  const uint32_t every = E->obs_every;
  if (every == 0u || (E->t + j) % every != 0u) return;
  const uint32_t nx = (uint32_t)E->g.n[0];
  if (blockIdx.x >= nx) return;
  const uint32_t row = ((E->t + j) / every) % E->obs_rows;
  double *const out = E->obs_out + (size_t)row * 2u * nx;
  SlabOut o{};
  o.T00 = out;
  o.T0x = out + nx;
  slab_moments(E->obs_sums, (uint32_t)(E->g.n[1] * E->g.n[2]), E->obs_vol, blockIdx.x, o);
}

// State export in one launch, one wave per cell (small states, whose outputs
// stay in the caches).
__global__ __launch_bounds__(kBlock) void k_gather_by_id(Cells cur_arg, uint32_t n_cells,
                                                         double *x, double *y, double *z,
                                                         double *px, double *py,
                                                         double *pz, uint32_t binning_step) {
  const GCells cur = binning(to_global(cur_arg), binning_step);
  const uint32_t lane = lane_id();
  const uint32_t c = blockIdx.x * kCellsPerBlock + threadIdx.x / 64;
  if (c >= n_cells) return;
  const auto put = [&](size_t o) {
    const Particle q = load_particle(cur.st, o);
    x[q.id] = q.x;
    y[q.id] = q.y;
    z[q.id] = q.z;
    px[q.id] = q.px;
    py[q.id] = q.py;
    pz[q.id] = q.pz;
  };
  const uint32_t n = occupancy(cur, c);
  const size_t base = (size_t)c * cur.cap;
  for (uint32_t j = lane; j < n; j += 64) put(base + j);
  if (cur.count[c] > cur.cap) {  // overflowing: its spilled members
    const SpillDesc *const spl = cur.sp;
    const uint32_t ns = min(spl->hdr[2u * cur.q], spl->capacity);
    for (uint32_t i = lane; i < ns; i += 64)
      if (spl->cell[i] == c) put(spl->base + i);
  }
}

// State export of larger states, first of two launches: slot_of[id] for
// every particle, G lanes per cell; the second reads the records in id
// order.  What is scattered is then 4 bytes written and one record read a
// particle, not six 8-byte writes (each a partial line): 16.3 M particles
// 3.42 -> 0.96 ms, 24.9 M in 2.1 M cells 5.99 -> 1.46 ms, 0.33 M 46 -> 20
// us; below some 10^5 particles the second launch costs more than it saves
// (10 000: 6 us in one launch, 8 in two).  The second takes only slots of the
// buffer: a particle that no cell holds was not listed, as when a captured
// export is replayed while the other buffer holds the state.  (Filling slot_of
// first, to tell those apart, took 3 us of 0.33 M particles' 36, 30 of 9.6 M's
// 535.)
constexpr int64_t kIndexedExportMin = 1 << 17;
template <uint32_t G>
__global__ __launch_bounds__(kBlock) void k_index_by_id(Cells cur_arg, uint32_t n_cells,
                                                        uint32_t *slot_of,
                                                        uint32_t binning_step) {
  const GCells cur = binning(to_global(cur_arg), binning_step);
  const uint32_t gl = lane_id() % G;
  const uint32_t c = (blockIdx.x * kBlock + threadIdx.x) / G;
  // the spilled particles, a thread each, by the first kSpillBlocks blocks (a
  // search of the spill slots by each overflowing cell: 402 us for 321 538
  // particles, 8 689 of 160 000 cells overflowing, now 36)
  constexpr uint32_t kSpillBlocks = 256;
  if (blockIdx.x < kSpillBlocks) {
    const SpillDesc *const spl = cur.sp;
    const uint32_t ns = min(spl->hdr[2u * cur.q], spl->capacity);
    const uint32_t stride = min(gridDim.x, kSpillBlocks) * kBlock;
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < ns; i += stride) {
      const size_t o = spl->base + i;
      slot_of[cur.st.id[o]] = (uint32_t)o;
    }
  }
  if (c >= n_cells) return;
  const uint32_t n = occupancy(cur, c);
  const size_t base = (size_t)c * cur.cap;
  for (uint32_t j = gl; j < n; j += G) slot_of[cur.st.id[base + j]] = (uint32_t)(base + j);
}

// Second launch: the records in id order.
__global__ __launch_bounds__(kBlock) void k_export_by_id(Cells cur_arg, int64_t n,
                                                         uint32_t n_slots,
                                                         const uint32_t *slot_of, double *x,
                                                         double *y, double *z, double *px,
                                                         double *py, double *pz) {
  const GCells cur = to_global(cur_arg);
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t o = slot_of[i];
  if (o >= n_slots) return;
  const gptr<Double2> r = record(cur.st, o);
  const Double2 a = r[0], b = r[1], c = r[2];
  px[i] = a.x;
  py[i] = a.y;
  pz[i] = b.x;
  x[i] = b.y;
  y[i] = c.x;
  z[i] = c.y;
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }
// Lanes per cell of the kernels that walk the cells of a state of n
// particles: the mean occupancy, rounded up to a power of two within 8 .. 64.
inline uint32_t walk_lanes(int64_t n, int64_t n_cells) {
  uint32_t g = 8;
  while (g < 64 && (int64_t)g * n_cells < n) g *= 2;
  return g;
}
template <typename F>
void with_walk_lanes(uint32_t g, F &&f) {
  switch (g) {
    case 8: f(std::integral_constant<uint32_t, 8>{}); break;
    case 16: f(std::integral_constant<uint32_t, 16>{}); break;
    case 32: f(std::integral_constant<uint32_t, 32>{}); break;
    default: f(std::integral_constant<uint32_t, 64>{});
  }
}
inline unsigned cell_blocks(int64_t n_cells) {
  return (unsigned)((n_cells + kCellsPerBlock - 1) / kCellsPerBlock);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
void launch_fill_u32(uint32_t *p, uint32_t v, int64_t count, hipStream_t s) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(count)), dim3(kBlock), 0, s, p, v, count);
}

void launch_store_f64(double *p, double v, hipStream_t s) {
  hipLaunchKernelGGL(k_store_f64, dim3(1), dim3(64), 0, s, p, v);
}

bool launch_write_bytes(void *dst, const void *src, size_t bytes, hipStream_t s) {
  if (bytes % 4 != 0 || bytes > sizeof(WriteWords) || ((uintptr_t)dst & 3u) != 0) return false;
  WriteWords v{};
  __builtin_memcpy(v.w, src, bytes);
  hipLaunchKernelGGL(k_write_words, dim3(1), dim3(64), 0, s, (uint32_t *)dst, v,
                     (uint32_t)(bytes / 4));
  return true;
}

namespace {

// A kernel launch that records the stage-timing events ev_start / ev_stop on
// its own dispatch when given (no event packets between launches, and the
// events read the kernel's duration), else a plain launch.
template <typename K, typename... Args>
void launch_timed(K kernel, dim3 grid, dim3 block, hipStream_t s, hipEvent_t ev_start,
                  hipEvent_t ev_stop, Args... args) {
  if (ev_start)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev_start, ev_stop, 0u, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
}

// A timed stage that launches nothing still records its events.
void record_empty(hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s) {
  if (ev_start) (void)hipEventRecord(ev_start, s);
  if (ev_stop) (void)hipEventRecord(ev_stop, s);
}

}  // namespace

void launch_init_bin(const double *x, const double *y, const double *z,
                     const double *px, const double *py, const double *pz,
                     const Cells &dst, int64_t n, const Geometry &g, DevStatus *st,
                     uint32_t binning_step, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_init_bin, dim3(grid_for(n)), dim3(kBlock), 0, s, x, y, z, px, py,
                     pz, dst, n, g, st, binning_step);
}

void launch_stream_bin(const Cells &src, const Cells &dst, int64_t n_cells, uint32_t lanes,
                       const Geometry &g, DevStatus *status, uint32_t *trace_cell,
                       uint32_t t, hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (n_cells <= 0) {
    record_empty(ev_start, ev_stop, s);
    return;
  }
  // (packed cells: 16 lanes a cell; a stream-bin that packs 64 particles
  // a round whatever their cells measured the same on the 32^3 fm^3 set,
  // whose sparse cells' cost is their partly used cache lines)
  const uint32_t G = lanes == 0 || lanes == kWideCells ? 64u
                     : lanes == kPackedCells                 ? 16u
                                                             : lanes;
  const int64_t waves = (n_cells + 64 / G - 1) / (64 / G);
  const dim3 grid(cell_blocks(waves)), block(kBlock);
  const uint32_t nc = (uint32_t)n_cells;
  switch (G) {
    case 8:
      launch_timed(k_stream_bin<8>, grid, block, s, ev_start, ev_stop, src, dst, nc, g, status,
                   trace_cell, t);
      break;
    case 16:
      launch_timed(k_stream_bin<16>, grid, block, s, ev_start, ev_stop, src, dst, nc, g, status,
                   trace_cell, t);
      break;
    case 32:
      launch_timed(k_stream_bin<32>, grid, block, s, ev_start, ev_stop, src, dst, nc, g, status,
                   trace_cell, t);
      break;
    default:
      launch_timed(k_stream_bin<64>, grid, block, s, ev_start, ev_stop, src, dst, nc, g, status,
                   trace_cell, t);
  }
}

void launch_offsets(const Cells &cur, uint32_t *offsets, uint32_t *tile_sums,
                    int64_t n_cells, hipStream_t s) {
  const unsigned tiles = (unsigned)((n_cells + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(kBlock), 0, s, cur, offsets,
                     tile_sums, n_cells);
  hipLaunchKernelGGL(k_scan_carry, dim3(tiles), dim3(kBlock), 0, s, offsets,
                     (const uint32_t *)tile_sums, n_cells);
}

namespace {

// fork: work queued on s so far precedes the work then queued on side
void fork(hipStream_t s, const SideStream *side) {
  if (!side) return;
  (void)hipEventRecord(side->fork, s);
  (void)hipStreamWaitEvent(side->stream, side->fork, 0);
}

// join: the work queued on side precedes the work then queued on s
void join(hipStream_t s, const SideStream *side) {
  if (!side) return;
  (void)hipEventRecord(side->join, side->stream);
  (void)hipStreamWaitEvent(s, side->join, 0);
}

// kMid: blocks larger than kCap (see cell_open).
template <bool kFused, bool kTrace, uint32_t kCap, bool kMid>
void launch_step_cap(const Cells &src, const Cells &dst, uint32_t n_cells, uint32_t lanes,
                     uint32_t t, const PairArgs &pa, const Geometry &g, DevStatus *status,
                     const TraceArgs &tr, hipStream_t s, const SideStream *side,
                     const StepDevice &dev) {
  const dim3 block(64);
  const int64_t shift = (int64_t)((const char *)dst.st.rec - (const char *)src.st.rec);
  // one kernel: timing events ride on its dispatch (no packets of their own
  // between launches)
  if (lanes == kWideCells && !kTrace) {
    const auto wide = [&](auto waves) {
      constexpr uint32_t kW = decltype(waves)::value;
      const auto launch = [&](auto kernel) {
        launch_timed(kernel, dim3(n_cells), dim3(64 * kW), s, dev.ev_start, dev.ev_stop, src,
                     shift, dev.ahead, t, pa, dev.g, status);
      };
      if (dev.ahead < src.cap)
        launch(k_step_wide<kFused, kCap, kW, true>);
      else
        launch(k_step_wide<kFused, kCap, kW, false>);
    };
    if (dev.waves == 4)
      wide(std::integral_constant<uint32_t, 4>{});
    else if (dev.waves == 8)
      wide(std::integral_constant<uint32_t, 8>{});
    else
      wide(std::integral_constant<uint32_t, kCap == kSmallCap ? 8 : 16>{});
    return;
  }
  if constexpr (!kTrace) {
    if (kCap == kSmallCap && lanes == 0 && dev.group) {
      launch_timed(k_step_group<kFused, kSmallCap, kMid>, dim3((n_cells + kGroup - 1) / kGroup),
                   dim3(64 * kGroup), s, dev.ev_start, dev.ev_stop, src, shift, n_cells, t, pa,
                   dev.g, status);
      return;
    }
  }
  if (lanes == 0 || lanes == kWideCells) {
    launch_timed(k_step<kFused, kTrace, kCap, kMid>, dim3(n_cells), block, s, dev.ev_start,
                 dev.ev_stop, src, shift, t, pa, dev.g, status, tr);
    return;
  }
  const dim3 grid((n_cells + dev.tile - 1) / dev.tile), wide(64 * kPackedWaves);
  // few larger cells, in blocks that the small LDS holds: the packed kernel
  // steps them itself
  if constexpr (!kTrace && kCap == kSmallCap) {
    if (dev.over_span != 1) {
      launch_timed(k_step_packed<kFused, kTrace, true, kMid>, grid, wide, s, dev.ev_start, dev.ev_stop,
                   src, shift, n_cells, dev.tile, t, pa, dev.g, status, tr);
      return;
    }
  }
  // the packed cells and, concurrently, the cells that the packed kernel
  // leaves alone (disjoint cells; both append to dst through atomics); timed
  // by events recorded around the whole launch
  if (dev.ev_start) (void)hipEventRecord(dev.ev_start, s);
  fork(s, side);
  hipLaunchKernelGGL((k_step_packed<kFused, kTrace, false, false>), grid, wide, 0, s, src, shift,
                     n_cells, dev.tile, t, pa, dev.g, status, tr);
  hipStream_t so = side ? side->stream : s;
  if (dev.over_span == 1)
    hipLaunchKernelGGL((k_step_over<kFused, kTrace, kCap, kMid>), dim3(n_cells), block, 0, so, src,
                       shift, t, pa, dev.g, status, tr);
  else
    hipLaunchKernelGGL((k_step_large<kFused, kTrace, kCap, kMid>), dim3((n_cells + 63) / 64), block,
                       0, so, src, dst, n_cells, t, pa, g, status, tr);
  join(s, side);
  if (dev.ev_stop) (void)hipEventRecord(dev.ev_stop, s);
}

template <uint32_t kCap, bool kMid>
void launch_step_any(const Cells &src, const Cells &dst, bool fused, uint32_t n_cells,
                     uint32_t lanes, uint32_t t, const PairArgs &pa, const Geometry &g,
                     DevStatus *status, const TraceArgs *trace, hipStream_t s,
                     const SideStream *side, const StepDevice &dev) {
  if (trace)
    launch_step_cap<false, true, kCap, false>(src, dst, n_cells, lanes, t, pa, g, status, *trace, s,
                                       side, dev);
  else if (fused)
    launch_step_cap<true, false, kCap, kMid>(src, dst, n_cells, lanes, t, pa, g, status,
                                       TraceArgs{}, s, side, dev);
  else
    launch_step_cap<false, false, kCap, kMid>(src, dst, n_cells, lanes, t, pa, g, status,
                                        TraceArgs{}, s, side, dev);
}

}  // namespace

void launch_step(const Cells &src, const Cells &dst, bool fused, int64_t n_cells,
                 uint32_t lanes, uint32_t t, const PairArgs &pa, const Geometry &g,
                 DevStatus *status, const TraceArgs *trace, hipStream_t s,
                 const SideStream *side, const StepDevice &dev) {
  if (n_cells <= 0) {
    record_empty(dev.ev_start, dev.ev_stop, s);
    return;
  }
  // cells of at most 512 slots, or particles, use the kernels with half the
  // LDS (the wide kernel by slots alone)
  if (src.cap <= kSmallCap)
    launch_step_any<kSmallCap, false>(src, dst, fused, (uint32_t)n_cells, lanes, t, pa, g, status,
                                      trace, s, side, dev);
  else if (dev.fits_small && lanes != kWideCells && !trace)
    launch_step_any<kSmallCap, true>(src, dst, fused, (uint32_t)n_cells, lanes, t, pa, g, status,
                                     trace, s, side, dev);
  else
    launch_step_any<kCellCap, false>(src, dst, fused, (uint32_t)n_cells, lanes, t, pa, g, status,
                                     trace, s, side, dev);
}

namespace {

__global__ __launch_bounds__(kBlock) void k_count_cells(const double *__restrict__ x,
                                                        const double *__restrict__ y,
                                                        const double *__restrict__ z,
                                                        int64_t n, Geometry g,
                                                        uint32_t *count) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double a = x[i], b = y[i], c = z[i];
    if (__builtin_isfinite(a) && __builtin_isfinite(b) && __builtin_isfinite(c))
      atomicAdd(&count[cell_id(g, a, b, c)], 1u);
  }
}

__global__ __launch_bounds__(kBlock) void k_max_u32(const uint32_t *__restrict__ v, int64_t n,
                                                    uint32_t *out) {
  uint32_t m = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    m = max(m, v[i]);
  m = wave_max(m);
  __shared__ uint32_t part[kBlock / 64];
  if (lane_id() == 0) part[threadIdx.x / 64] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t w = 1; w < kBlock / 64; ++w) m = max(m, part[w]);
    atomicMax(out, m);
  }
}

}  // namespace

void launch_count_cells(const double *x, const double *y, const double *z, int64_t n,
                        const Geometry &g, int64_t n_cells, uint32_t *count,
                        uint32_t *max_count, hipStream_t s) {
  launch_fill_u32(count, 0u, n_cells, s);
  launch_fill_u32(max_count, 0u, 1, s);
  if (n > 0) {
    const unsigned grid = grid_for(n) < 4096u ? grid_for(n) : 4096u;
    hipLaunchKernelGGL(k_count_cells, dim3(grid), dim3(kBlock), 0, s, x, y, z, n, g, count);
  }
  // few blocks, one atomic each: atomics on the one word run one after the
  // other (160 000 cells: 31 us with 2 500 of them)
  const unsigned grid = grid_for(n_cells) < 256u ? grid_for(n_cells) : 256u;
  hipLaunchKernelGGL(k_max_u32, dim3(grid), dim3(kBlock), 0, s, (const uint32_t *)count,
                     n_cells, max_count);
}

void launch_occupancy_over(const Cells &cur, int64_t n_cells, DevStatus *status,
                           hipStream_t s) {
  if (n_cells <= 0) return;
  const unsigned grid = grid_for(n_cells) < 1024u ? grid_for(n_cells) : 1024u;
  hipLaunchKernelGGL(k_occupancy_over, dim3(grid), dim3(kBlock), 0, s, cur,
                     (uint32_t)n_cells, status->over);
}

void launch_observe(const Cells &cur, const Geometry &g, int64_t n, double vol,
                    double *cell_sums, const SlabOut &out, uint32_t binning_step,
                    hipStream_t s) {
  const int64_t n_cells = (int64_t)g.n[0] * g.n[1] * g.n[2];
  const uint32_t G = walk_lanes(n, n_cells);
  with_walk_lanes(G, [&](auto lanes) {
    hipLaunchKernelGGL((k_observe_cells<lanes.value>), dim3(grid_for(n_cells * G)),
                       dim3(kBlock), 0, s, cur, (uint32_t)n_cells, cell_sums, binning_step);
  });
  hipLaunchKernelGGL(k_observe_slabs, dim3((unsigned)g.n[0]), dim3(kBlock), 0, s,
                     (const double *)cell_sums, (uint32_t)(g.n[1] * g.n[2]), vol, out);
}

void launch_batch_run(BatchEvent *ev, const BatchSpaces &sp, uint32_t n_events, int32_t k,
                      uint32_t persistent_waves, hipStream_t s, const SideStream *side,
                      void (*between)(void *, int), void *ctx, const uint8_t *obs_at) {
  if (n_events == 0 || sp.n_items == 0 || k <= 0) return;
  const uint32_t bin_waves =
      persistent_waves > 0 && persistent_waves < sp.n_items ? persistent_waves : sp.n_items;
  const uint32_t bin_grid = (bin_waves + kCellsPerBlock - 1) / kCellsPerBlock;
  const BatchEvent *cev = ev;
  const dim3 wave(64);
  if (between) between(ctx, 0);
  hipLaunchKernelGGL(k_batch_bin, dim3(bin_grid), dim3(kBlock), 0, s, cev, sp.item_begin,
                     n_events, sp.n_items);
  // launch j: the packed events on s; concurrently on the side stream the
  // cells of events stepped one wave per cell, then the larger cells of
  // packed events with large blocks (all disjoint cells; appends go through
  // atomics)
  auto step = [&](auto fused, uint32_t j) {
    constexpr bool kF = decltype(fused)::value;
    // the events due for an observation after this launch
    const bool observe = sp.obs_nx > 0 && (!obs_at || obs_at[j]);
    // (an observing launch steps the scans behind the tiles: a scan clears the
    // counts of the cells that it steps, and a tile that read one of those as
    // empty would write zeros over the sums of the cell)
    const bool scan_aside = sp.n_scans > 0 && !observe;
    const bool both =
        sp.n_tiles > 0 &&
        (sp.n_cells[0] > 0 || sp.n_cells[1] > 0 || sp.n_groups > 0 || scan_aside);
    const SideStream *sd = both ? side : nullptr;
    const hipStream_t s2 = sd ? sd->stream : s;
    fork(s, sd);
    if (sp.n_tiles > 0)
      hipLaunchKernelGGL((k_batch_step_packed<kF>), dim3(sp.n_tiles), dim3(64 * kPackedWaves), 0,
                         s, cev, sp.tile_begin, n_events, j);
    if (sp.n_groups > 0)
      hipLaunchKernelGGL((k_batch_step_group<kF>), dim3(sp.n_groups), dim3(64 * kGroup), 0, s2,
                         cev, sp.group_begin, n_events, j);
    if (sp.n_cells[0] > 0)
      hipLaunchKernelGGL((k_batch_step_cells<kF, kSmallCap>), dim3(sp.n_cells[0]), wave, 0, s2,
                         cev, sp.cell_begin[0], n_events, j);
    if (sp.n_cells[1] > 0)
      hipLaunchKernelGGL((k_batch_step_cells<kF, kCellCap>), dim3(sp.n_cells[1]), wave, 0, s2,
                         cev, sp.cell_begin[1], n_events, j);
    if (sp.n_scans > 0)
      hipLaunchKernelGGL((k_batch_step_scan<kF>), dim3(sp.n_scans), wave, 0,
                         scan_aside ? s2 : s, cev, sp.scan_begin, n_events, j);
    join(s, sd);
    if (observe)
      hipLaunchKernelGGL(k_batch_observe, dim3(sp.obs_nx, n_events), dim3(kBlock), 0, s, cev,
                         n_events, j);
  };
  using Fused = std::integral_constant<bool, true>;
  using Last = std::integral_constant<bool, false>;
  for (int32_t j = 1; j < k; ++j) {
    if (between) between(ctx, 1);
    step(Fused{}, (uint32_t)j);
  }
  if (between) between(ctx, 2);
  step(Last{}, (uint32_t)k);
  if (between) between(ctx, -1);
  hipLaunchKernelGGL(k_batch_advance, dim3((n_events + 63) / 64), dim3(64), 0, s, ev,
                     n_events, (uint32_t)k);
}

void launch_export(const Cells &cur, int64_t n_cells, int64_t n, uint32_t *slot_of, double *x,
                   double *y, double *z, double *px, double *py, double *pz,
                   uint32_t binning_step, hipStream_t s) {
  if (n_cells <= 0 || n <= 0) return;
  if (n < kIndexedExportMin) {
    hipLaunchKernelGGL(k_gather_by_id, dim3(cell_blocks(n_cells)), dim3(kBlock), 0, s, cur,
                       (uint32_t)n_cells, x, y, z, px, py, pz, binning_step);
    return;
  }
  const uint32_t G = walk_lanes(n, n_cells);
  with_walk_lanes(G, [&](auto lanes) {
    hipLaunchKernelGGL((k_index_by_id<lanes.value>), dim3(grid_for(n_cells * G)), dim3(kBlock),
                       0, s, cur, (uint32_t)n_cells, slot_of, binning_step);
  });
  const uint32_t n_slots = (uint32_t)(n_cells * (int64_t)cur.cap + n);  // blocks, spill slots
  hipLaunchKernelGGL(k_export_by_id, dim3(grid_for(n)), dim3(kBlock), 0, s, cur, n, n_slots,
                     (const uint32_t *)slot_of, x, y, z, px, py, pz);
}

}  // namespace cuba
