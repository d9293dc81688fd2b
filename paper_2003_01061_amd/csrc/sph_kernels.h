// sph_kernels.h -- the gfx950 kernels of one relaxation step.
//
// Per step (Algorithm 1's loop body, every feature at once, all reading x^n);
// h_i = h_t(x_i), the cell of x_i and its rank inside the cell are already
// known from the previous step's integration (or the set-up hash):
//   k_scan           single-pass exclusive scan of the cell counts (decoupled
//                    look-back) -> cell start table
//   k_scatter        position of every particle in cell order
//   k_rank_gather    order inside a cell by caller id (canonical, history
//                    free), permute the particle records into it, and store
//                    the boundary normals of particles on holes
//   k_nbr_group      (or k_nbr_forces) ELL neighbour list (exact FP64 predicate +
//                    feature relation) fused with the Shepard gamma, V~, pressure
//                    force with the boundary term and its tangent projection
//                    -> a^p; striped minima of dt_1 and sums of V~
//   k_midpoint       3D: v~ and eta of every particle for the gathers
//   k_sweep_b        dt_1 from its stripes, mid-point velocity, viscous force
//                    -> a; striped minima of dt
//   k_integrate_hash dt from its stripes, v_{n+1/2}, x_{n+1}, projection /
//                    rejection, then h, cell and rank of every particle for the
//                    next step
// and the control of the step (E_sys, phases, resets, damping of every feature,
// a block per job) runs beside the next step's scan, or as k_control after the
// last step of a call.
// A launch covers every job of a batch: particles carry a global feature id
// (64 per job slot), every kernel reads its particle's job record, and a
// job's cells occupy their own range of the batch's cell ids, so jobs never
// interact and each job's result is the same alone or in any mix (with Verlet
// lists, whose rebuilds follow the whole batch, up to the order of its sums).
#pragma once
#include "sph_device.h"

namespace sph {

__device__ __forceinline__ unsigned long long umin64(unsigned long long a, unsigned long long b) {
  return a < b ? a : b;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// The particle's terms of Eq. (fa_time_step_size) from |a|^2 and |v|^2 (the
// third term can never be the smallest, so it is left out): min(0.25
// sqrt(r_c / |a|), r_c / (40 |v|)), infinite when both vanish.  F32: in
// FP32 (the FP32 modes hold the time steps to 1e-5), unless a square is
// beyond FP32's range, where FP32 would give a time step of 0.
template <bool F32>
__device__ __forceinline__ double step_terms(double rc, double a2, double v2) {
  if constexpr (F32) {
    if (!(a2 < 1e36 && v2 < 1e36)) return step_terms<false>(rc, a2, v2);
    const float rcf = (float)rc, am = __builtin_amdgcn_sqrtf((float)a2),
                vm = __builtin_amdgcn_sqrtf((float)v2);
    float dt = __builtin_inff();
    if (am > 0.0f) dt = 0.25f * __builtin_amdgcn_sqrtf(rcf * __builtin_amdgcn_rcpf(am));
    if (vm > 0.0f) {
      const float t = rcf * __builtin_amdgcn_rcpf(40.0f * vm);
      dt = t < dt ? t : dt;
    }
    return (double)dt;
  } else {
    double dt = __builtin_inf();
    const double am = __builtin_sqrt(a2);
    if (am > 0.0) dt = 0.25 * __builtin_sqrt(rc / am);
    const double vm = __builtin_sqrt(v2);
    if (vm > 0.0) {
      const double t = rc / (40.0 * vm);
      dt = t < dt ? t : dt;
    }
    return dt;
  }
}

// Per-feature reduction of one wave: the valid lanes of each distinct feature
// are reduced with xor shuffles and committed by one lane with device atomics
// into one of NSTRIPE copies of the feature's accumulators (chosen by wave).
// Minima of non-negative double bit patterns and integer sums are exact and
// order independent, so the result does not depend on scheduling or on which
// other jobs share the launch.  Atomics on one cache line follow each other
// wherever on the line they fall, so the copies of a feature lie 512 bytes apart:
// k_sweep_b of 1,000,000 particles in 2D, by two lanes, took 59 us with 32 copies
// so, 91 with 32 copies in 2 lines (59 with 64 in 4), and as a feature's row of copies is
// also the row of its neighbours', a block folds them all with a few loads.
__device__ __forceinline__ size_t stripe_at(int q, int copies, int stripe) {
  return ((size_t)(q / MAXF) * copies + stripe) * MAXF + q % MAXF;
}
__device__ __forceinline__ int wave_stripe(int waves) {   // waves: of a block that commit
  return (int)((blockIdx.x * waves + (threadIdx.x >> 6)) & (NSTRIPE - 1));
}
// which: DT1 or DT; ssum null: no sums
constexpr int DT1 = 0, DT = NSTRIPE;   // a feature's copies of either time step in smin
__device__ __forceinline__ void wave_commit(bool valid, int key, unsigned long long vmin,
                                            unsigned long long vadd, unsigned long long *smin, int which,
                                            unsigned long long *ssum, int waves = BLOCK / 64) {
  const int stripe = wave_stripe(waves);
  unsigned long long mask = __ballot(valid);
  const int lane = __lane_id();
  while (mask) {
    const int leader = __ffsll((long long)mask) - 1;
    const int kl = __shfl(key, leader);
    const bool mine = valid && key == kl;
    const unsigned long long mm = __ballot(mine);
    unsigned long long mn = mine ? vmin : ~0ull;
    unsigned long long sm = mine ? vadd : 0ull;
    for (int o = 32; o > 0; o >>= 1) {
      mn = umin64(mn, __shfl_xor(mn, o));
      if (ssum) sm += __shfl_xor(sm, o);
    }
    if (lane == leader) {
      atomicMin(&smin[stripe_at(kl, 2 * NSTRIPE, which + stripe)], mn);
      if (ssum && sm) atomicAdd(&ssum[stripe_at(kl, NSTRIPE, stripe)], sm);
    }
    mask &= ~mm;
  }
}

// the same for a counter of each job (word: SC_PAIRS or SC_ESCAPED)
__device__ __forceinline__ void wave_count(bool valid, int job, unsigned long long add,
                                           unsigned long long *scnt, int word, int waves = BLOCK / 64) {
  const int stripe = wave_stripe(waves);
  unsigned long long mask = __ballot(valid);
  const int lane = __lane_id();
  while (mask) {
    const int leader = __ffsll((long long)mask) - 1;
    const int jl = __shfl(job, leader);
    const bool mine = valid && job == jl;
    const unsigned long long sm = wave_sum_u64(mine ? add : 0ull);
    if (lane == leader) atomicAdd(&scnt[((size_t)jl * NSTRIPE + stripe) * SC_ROW + word], sm);
    mask &= ~__ballot(mine);
  }
}

// read a striped accumulator word (filled by the previous launch) and reset it
__device__ __forceinline__ unsigned long long take(unsigned long long *p, unsigned long long reset) {
  const unsigned long long v = *p;
  *p = reset;
  return v;
}

// Folding the copies is the consumer's: each block of the next kernel does it in
// the shadow of its own loads, which costs it 0.5 to 2 us (the control beside the
// scan 1 to 3), where a launch costs 3 to 4 (4,352 particles: 44.0 us a step with two such launches
// and the control's, 39.3 without; 3D, 66,000: 151 and 143; 2,000,000: no
// difference).
// The copies of a job's features, a lane per feature and a share of the copies
// per wave, as one round of independent row loads; the block's waves leave their
// minima in `part` and meet at a barrier.
constexpr int FOLD = NSTRIPE / (BLOCK / 64);
static_assert(NSTRIPE % (BLOCK / 64) == 0 && MAXF == 64, "a lane per feature, whole shares");
using FoldParts = unsigned long long[BLOCK / 64][MAXF];
__device__ __forceinline__ void fold_rows(const Batch &B, int which, int job, FoldParts &part) {
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  unsigned long long v = ~0ull;
  if (lane < B.jobs[job].nf) {
    const unsigned long long *row = B.smin + stripe_at(job * MAXF + lane, 2 * NSTRIPE, which + wave * FOLD);
#pragma unroll
    for (int r = 0; r < FOLD; ++r) v = umin64(v, row[r * MAXF]);
  }
  part[wave][lane] = v;
}
// The time step of feature f (a global id) from the folded copies: the minimum
// of the particle terms and the job's dt_max.
__device__ __forceinline__ unsigned long long step_bits(const Batch &B, const FoldParts &part, int f) {
  unsigned long long v = dbits(B.jobs[f / MAXF].ctl.dt_max);
#pragma unroll
  for (int w = 0; w < BLOCK / 64; ++w) v = umin64(v, part[w][f % MAXF]);
  return v;
}

// ---------------------------------------------------------------------------
// control of every feature of one job after a step, by one block; folds and
// clears the step's stripes and prepares the next step
// ---------------------------------------------------------------------------
__device__ __forceinline__ void control_job(const Batch &B, int job) {
  __shared__ FoldParts p1, p2, pv;
  __shared__ int moving;
  if (threadIdx.x == 0) moving = 0;
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  Group &G = B.grp[(size_t)job * MAXF + lane];
  unsigned long long c = 0ull;   // pairs in the lower half wave, escapes in the upper
  if (wave == BLOCK / 64 - 1)
    c = take(B.scnt + ((size_t)job * NSTRIPE + lane % NSTRIPE) * SC_ROW + (lane < NSTRIPE ? SC_PAIRS : SC_ESCAPED),
             0ull);
  fold_rows(B, DT1, job, p1);
  fold_rows(B, DT, job, p2);
  const bool tracked = G.tracked != 0;
  unsigned long long sum = 0ull;
  if (tracked) {
    const int q = job * MAXF + lane;
#pragma unroll
    for (int r = 0; r < FOLD; ++r) {
      const int k = wave * FOLD + r;
      sum += take(B.ssum + stripe_at(q, NSTRIPE, k), 0ull);
      B.smin[stripe_at(q, 2 * NSTRIPE, DT1 + k)] = ~0ull;
      B.smin[stripe_at(q, 2 * NSTRIPE, DT + k)] = ~0ull;
    }
  }
  pv[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && tracked) {
    const Ctl &P = B.jobs[job].ctl;
    if (G.phase != PH_FROZEN) {
      unsigned long long vsum = 0ull;
      for (int w = 0; w < BLOCK / 64; ++w) vsum += pv[w][lane];
      const double dt1 = bitsd(step_bits(B, p1, job * MAXF + lane)), dt = bitsd(step_bits(B, p2, job * MAXF + lane));
      const double vbar = (double)vsum / G.vscale;
      G.dt1 = dt1;
      G.dt = dt;
      control_law(P, G, vbar, dt);
    }
    G.active = G.phase != PH_FROZEN;
    G.reset_now = G.reset_next;
    G.eps = damping(P, G);
    if (G.active) atomicOr(&moving, 1);
  }
  __syncthreads();
  if (wave == BLOCK / 64 - 1) {
    for (int o = NSTRIPE / 2; o > 0; o >>= 1) c += __shfl_xor(c, o);
    const unsigned long long e = __shfl(c, NSTRIPE);
    JobStat &S = B.st[job];
    if (lane == 0 && S.live) {
      if (!S.converged) S.steps += 1ull;     // a converged job stops counting
      S.inter_last = c;
      S.inter_total += c;
      S.escaped += e;
      S.converged = moving ? 0 : 1;
    }
  }
}

// after the last step of a call: a block per job slot
__global__ __launch_bounds__(BLOCK) void k_control(Batch B) { control_job(B, (int)blockIdx.x); }

// ---------------------------------------------------------------------------
// cell hashing and counting sort
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void hash_one(const Geom &g, const Grid &G, double4 &xh, uint32_t &cell) {
  double p[3] = {xh.x, xh.y, xh.z};
  xh.w = h_target<D>(g, p);
  const int l = h_level(G, xh.w);
  int c0 = cell_coord(G, l, 0, p[0]);
  int c1 = cell_coord(G, l, 1, p[1]);
  int c2 = D == 3 ? cell_coord(G, l, 2, p[2]) : 0;
  cell = G.cbase + G.lbase[l] +
         cell_row<D>(G, l, (uint32_t)c1, (uint32_t)c2) * (uint32_t)G.nc[l][0] + (uint32_t)c0;
}

// Rank of a particle inside its cell.  Lanes of a wave that hold the same
// cell in consecutive lanes form a run (particles are in cell order, and most
// stay in their cell from one step to the next); the run's first lane
// reserves the whole run with one atomic and the others take consecutive
// ranks, so a wave issues one atomic per distinct run instead of one per
// particle.  Valid lanes are a prefix of the wave.  Ranks only need to be
// distinct: k_rank_gather puts each cell in caller-id order afterwards.
__device__ __forceinline__ uint32_t rank_in_cell(uint32_t c, bool valid, uint32_t *cnt) {
  const int lane = __lane_id();
  const uint32_t prev = __shfl_up(c, 1);
  const bool head = valid && (lane == 0 || prev != c);
  const unsigned long long heads = __ballot(head);
  const int nvalid = __popcll(__ballot(valid));
  const unsigned long long below_eq = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  const unsigned long long above = heads & ~below_eq;
  const int next = above ? __ffsll((long long)above) - 1 : 64;
  uint32_t base = 0;
  if (head) base = atomicAdd(&cnt[c], (uint32_t)((next < nvalid ? next : nvalid) - lane));
  const unsigned long long mine = heads & below_eq;
  const int my_head = mine ? 63 - __clzll((long long)mine) : 0;
  return __shfl(base, my_head) + (uint32_t)(lane - my_head);
}

// h, cell and rank inside the cell of the particles [i0, i1) (set-up and
// test paths; a step gets them from k_integrate_hash)
template <int D>
__global__ __launch_bounds__(BLOCK) void k_hash(Batch B, Parts s, int i0, int i1,
                                                uint32_t *__restrict__ cell,
                                                uint32_t *__restrict__ rank,
                                                uint32_t *__restrict__ cnt) {
  const int i = i0 + (int)(blockIdx.x * BLOCK + threadIdx.x);
  const bool valid = i < i1;
  uint32_t c = 0;
  if (valid) {
    const uint32_t f = s.f[i];
    const JobDev &J = B.jobs[f / MAXF];
    double4 xh = s.xh[i];
    hash_one<D>(J.g, J.G, xh, c);
    s.xh[i] = xh;
    s.xf[i] = scan_record<D>(xh, f);
    cell[i] = c;
  }
  const uint32_t r = rank_in_cell(c, valid, cnt);
  if (valid) rank[i] = r;
}

constexpr int SCAN_PER = 16;
constexpr int SCAN_TILE = BLOCK * SCAN_PER;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *lds, uint32_t &total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds[wid] = x;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int w = 0; w < BLOCK / 64; ++w) {
    uint32_t t = lds[w];
    if (w < wid) pre += t;
    tot += t;
  }
  __syncthreads();
  total = tot;
  return pre + x - v;
}

// Single-pass exclusive scan (decoupled look-back).  Tiles take ids from a
// ticket in dispatch order, so a tile only ever waits for tiles that have
// already started; each tile publishes {flag, value} in one 64-bit word:
// flag 1 = tile aggregate, flag 2 = inclusive prefix.  Flag and value travel
// in the same atomic word and nothing else is communicated between tiles, so
// relaxed device-scope atomics suffice (a release would write back the L2 of
// the XCD on every tile).  A tile's counts are loaded coalesced and
// transposed through LDS so that each thread scans SCAN_PER consecutive
// cells.  status[] and the ticket are cleared by k_scatter, which runs after
// the scan has finished.  The first
// ctl_jobs blocks do the control of the step before instead (control_job): it
// needs nothing of the scan, and the scan nothing of it.
__global__ __launch_bounds__(BLOCK) void k_scan(Batch B, int ctl_jobs, const uint32_t *__restrict__ in,
                                                uint32_t *__restrict__ out, uint32_t n,
                                                unsigned long long *status, uint32_t *ticket,
                                                uint32_t ntiles, unsigned int *gflags,
                                                const unsigned long long *__restrict__ vstate) {
  if ((int)blockIdx.x < ctl_jobs) {
    control_job(B, (int)blockIdx.x);
    return;
  }
  // with Verlet candidate lists, particles are re-sorted only when the lists
  // are rebuilt
  if (vstate && !vstate[VS_REBUILD]) return;
  __shared__ uint32_t lds[BLOCK / 64];
  __shared__ uint32_t s_tile, s_prefix;
  // tile in LDS, one padding word per SCAN_PER so that the per-thread reads
  // of SCAN_PER consecutive words hit distinct banks
  __shared__ uint32_t tbuf[SCAN_TILE + SCAN_TILE / SCAN_PER];
  if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
  __syncthreads();
  const uint32_t tile = s_tile;
  if (tile >= ntiles) {            // stale ticket: report, never wait
    if (threadIdx.x == 0) atomicExch(&gflags[0], 1u);
    return;
  }
  const size_t tbase = (size_t)tile * SCAN_TILE;
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    const uint32_t t = (uint32_t)k * BLOCK + threadIdx.x;
    const size_t idx = tbase + t;
    tbuf[t + t / SCAN_PER] = idx < n ? in[idx] : 0u;
  }
  __syncthreads();
  uint32_t v[SCAN_PER];
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    v[k] = tbuf[threadIdx.x * (SCAN_PER + 1) + k];
    sum += v[k];
  }
  uint32_t tot;
  uint32_t ex = block_exclusive_scan(sum, lds, tot);
  if (threadIdx.x < 64) {
    // publish the tile aggregate, then look back with the whole wave: lane l
    // reads tile (base - l); tiles before 0 count as an inclusive prefix 0.
    // Predecessors took their tickets earlier and publish without waiting on
    // later tiles, so the loop ends; the spin bound only turns a broken
    // invariant into an error instead of a hang.
    const int lane = threadIdx.x;
    if (lane == 0)
      __hip_atomic_store(&status[tile], ((tile == 0 ? 2ull : 1ull) << 32) | tot, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    uint32_t prefix = 0;
    int base = (int)tile - 1;
    unsigned spins = 0;
    while (base >= 0) {
      const int p = base - lane;
      unsigned long long w = p >= 0 ? __hip_atomic_load(&status[p], __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)
                                    : (2ull << 32);
      const unsigned flag = (unsigned)(w >> 32);
      const unsigned long long m2 = __ballot(flag == 2u);
      const unsigned long long m0 = __ballot(flag == 0u);
      const int first2 = m2 ? __ffsll((long long)m2) - 1 : 64;
      const unsigned long long upto = first2 >= 63 ? ~0ull : ((2ull << first2) - 1ull);
      if (m0 & upto) {
        if (++spins > (1u << 22)) {
          if (lane == 0) atomicExch(&gflags[0], 1u);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      unsigned long long part = lane <= first2 ? (unsigned long long)(uint32_t)w : 0ull;
      part = wave_sum_u64(part);
      prefix += (uint32_t)part;
      if (first2 < 64) break;
      base -= 64;
    }
    if (lane == 0) {
      if (tile != 0)
        __hip_atomic_store(&status[tile], (2ull << 32) | (uint32_t)(prefix + tot), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      s_prefix = prefix;
      if ((size_t)(tile + 1) * SCAN_TILE >= n) out[n] = prefix + tot;
    }
  }
  __syncthreads();
  ex += s_prefix;
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {   // back through LDS for coalesced stores
    tbuf[threadIdx.x * (SCAN_PER + 1) + k] = ex;
    ex += v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < SCAN_PER; ++k) {
    const uint32_t t = (uint32_t)k * BLOCK + threadIdx.x;
    const size_t idx = tbase + t;
    if (idx < n) out[idx] = tbuf[t + t / SCAN_PER];
  }
}

__global__ __launch_bounds__(BLOCK) void k_scatter(int n, const uint32_t *__restrict__ cell,
                                                   const uint32_t *__restrict__ rank,
                                                   const uint32_t *__restrict__ cstart,
                                                   const uint32_t *__restrict__ oid,
                                                   uint32_t *__restrict__ psrc,
                                                   uint32_t *__restrict__ pkey,
                                                   unsigned long long *__restrict__ status,
                                                   uint32_t ntiles, uint32_t *__restrict__ ticket,
                                                   const unsigned long long *__restrict__ vstate) {
  if (vstate && !vstate[VS_REBUILD]) return;   // no sort between list builds
  const int i = blockIdx.x * BLOCK + threadIdx.x;
  for (uint32_t t = (uint32_t)i; t < ntiles; t += gridDim.x * BLOCK) status[t] = 0ull;
  if (i == 0) *ticket = 0u;
  if (i >= n) return;
  uint32_t pos = cstart[cell[i]] + rank[i];
  if (pos >= (uint32_t)n) return;   // counts are consistent by construction
  psrc[pos] = (uint32_t)i;
  pkey[pos] = oid[i];
}

// Entry u of a cell (filled in atomic order) finds its rank among the cell's
// caller ids and copies its particle to that slot; the first entry of a cell
// clears the cell's count for the next hash.  With Verlet candidate lists the
// particles live in buffer a between rebuilds: with no rebuild due, every
// particle keeps its slot, clears its cell's count and refreshes its boundary
// normal; at a rebuild the sorted copy goes to b (whose slot also records x
// and h), and the list build copies it back into a.
// Bound by memory and its latency.  The bound on the registers keeps the
// closest-point search, which only curve particles run, from costing the others
// their waves: of 2,000,000 particles in 3D 83.1 us with 73 registers (6 waves a
// SIMD), 76.0 with 58 (8).
template <int D>
__global__ __launch_bounds__(BLOCK, 8) void k_rank_gather(Batch B, int n, const uint32_t *__restrict__ psrc,
                                                       const uint32_t *__restrict__ pkey,
                                                       const uint32_t *__restrict__ cell,
                                                       const uint32_t *__restrict__ cstart,
                                                       uint32_t *__restrict__ cnt, Parts a,
                                                       Parts b) {
  const int u = blockIdx.x * BLOCK + threadIdx.x;
  if (u >= n) return;
  const bool sorted = !B.skin_on || B.vstate[VS_REBUILD] != 0ull;
  uint32_t src = (uint32_t)u, dst = (uint32_t)u;
  if (sorted) {
    src = psrc[u];
    if (src >= (uint32_t)n) return;
    const uint32_t c = cell[src];
    const uint32_t lo = cstart[c], hi = cstart[c + 1];
    const uint32_t key = pkey[u];
    uint32_t r = 0;
    for (uint32_t v = lo; v < hi; ++v) r += pkey[v] < key ? 1u : 0u;
    if ((uint32_t)u == lo) cnt[c] = 0u;
    dst = lo + r;
    if (dst >= (uint32_t)n) return;
    b.oid[dst] = key;
  } else {
    cnt[cell[u]] = 0u;
  }
  const double4 xh = a.xh[src];
  const uint32_t f = a.f[src];
  if (sorted) {   // without a re-sort the particle stays where it is, in a
    b.f[dst] = (uint16_t)f;
    b.xh[dst] = xh;
    b.v[dst] = a.v[src];
    b.xf[dst] = scan_record<D>(xh, f);
    if (B.skin_on) B.xref[dst] = xh;
  }
  // the domain's outward normal at a particle of a feature of lower dimension
  // than the domain, for the pressure sweep of the volume particles beside it
  // (computed there, it would hold registers inside the neighbour loop):
  // towards the centre of a disc or ball, against the level set's gradient for
  // an ellipse or ellipsoid, the closest segment's for an imported curve, and
  // for a box face, edge or corner the constant normal of the volume's table
  const Feat F = B.feat[f];
  if (F.k < D) {
    if (F.kind == K_POLY && D == 2) {   // an imported curve: the closest segment's right normal
      const Geom &gg = B.jobs[f / MAXF].g;
      const double x[3] = {xh.x, xh.y, xh.z};
      double q[2], t[2];
      seg_tangent<2>(gg, poly_closest<2>(gg, F.hole, x, q), t);
      B.enrm[dst] = make_double4(t[1], -t[0], 0.0, 0.0);
    } else if (F.kind == K_POLY) {   // a 3D curve on the zero set: towards decreasing
                                      // phi, and its closest segment in w
      const Geom &gg = B.jobs[f / MAXF].g;
      const double x[3] = {xh.x, xh.y, xh.z};
      double q[3], m[3];
      const int k = poly_closest<3>(gg, F.hole, x, q);
      ls_unit<3>(gg, x, m);
      B.enrm[dst] = make_double4(-m[0], -m[1], -m[2], (double)k);
    } else if (F.kind == K_LEVEL) {   // the zero level set: towards decreasing phi
      const double x[3] = {xh.x, xh.y, xh.z};
      double m[3];
      ls_unit<D>(B.jobs[f / MAXF].g, x, m);
      B.enrm[dst] = make_double4(-m[0], -m[1], -m[2], 0.0);
    } else if (F.kind == K_SHELL) {   // the ball domain's sphere: radially outwards
      const double *cc = B.jobs[f / MAXF].g.dc;
      const double d0 = xh.x - cc[0], d1 = xh.y - cc[1], d2 = D == 3 ? xh.z - cc[2] : 0.0;
      const double il = 1.0 / __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      B.enrm[dst] = make_double4(d0 * il, d1 * il, d2 * il, 0.0);
    } else if (F.kind == K_HOLE) {
      const Geom &g = B.jobs[f / MAXF].g;
      double4 e;
      if (g.hell[F.hole]) {
        const double x[3] = {xh.x, xh.y, xh.z};
        double m[3] = {0.0, 0.0, 0.0};
        ell_normal<D>(g, F.hole, x, m);
        e = make_double4(-m[0], -m[1], -m[2], 0.0);
      } else {
        const double *cc = g.hc[F.hole];
        const double d0 = cc[0] - xh.x, d1 = cc[1] - xh.y, d2 = D == 3 ? cc[2] - xh.z : 0.0;
        const double il = 1.0 / __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        e = make_double4(d0 * il, d1 * il, d2 * il, 0.0);
      }
      B.enrm[dst] = e;
    } else {   // a box face, edge or corner, an imported corner: the table's constant
      const int job = f / MAXF, vol = B.jobs[job].vol;
      if (vol >= 0) {
        const BNorm N = B.bn[(size_t)(job * MAXF + vol) * MAXF + (f & (MAXF - 1))];
        B.enrm[dst] = make_double4(N.n[0], N.n[1], N.n[2], 0.0);
      }
    }
  }
}

// how the kernels with one lane per particle add (2D): in list order, as four
// lanes would, or either by the job (JobDev::four)
enum { AS_ONE, AS_FOUR, AS_JOB };

// does v hold in a lane of the wave (on the host: a lane by itself)
__host__ __device__ __forceinline__ bool any_lane(bool v) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_ballot_w64(v) != 0ull;
#else
  return v;
#endif
}
#ifdef __HIP_DEVICE_COMPILE__
using LdsList = const __attribute__((address_space(3))) uint32_t *;
#else
using LdsList = const uint32_t *;
#endif

// ---------------------------------------------------------------------------
// Pair terms of sweep A (Eqs. (gamma_disc_renormSPH), (particle_volume),
// (sph_pressure_force_disc_weighted)) for a particle of intrinsic dimension K,
// evaluated in R and accumulated by Sum<CMP>: in FP64, or (CMP, R = float) in
// FP32 with Neumaier compensation.  What is fused into a multiply-add is written
// out, not left to the compiler, so that every kernel gets the same bits: group_sums
// by four lanes and four_sums, which add them in the same order, take each other's
// place.
// ---------------------------------------------------------------------------
template <int D, int K, typename R, bool CMP>
struct TermsA {
  // h enters rho_t = h^-k; the kernel is evaluated at the smoothing length
  // klen h (cut-off radius 2 klen h)
  R hi, kl, ihi, hik, hi2k, ihik, P0;
  __host__ __device__ __forceinline__ TermsA(double h, double klen, double p0) {
#pragma clang fp contract(off)
    hi = (R)h;
    kl = (R)klen;
    ihi = rcp_((R)(klen * h));
    hik = powK<K>(hi);
    hi2k = hik * hik;
    ihik = powK<K>(ihi);
    P0 = (R)p0;
  }
  // the self term, when `on`
  __host__ __device__ __forceinline__ void self(bool on, Sum<CMP> &aS, Sum<CMP> &aG) const {
#pragma clang fp contract(off)
    constexpr R alpha = kalphaK<K, R>();
    const R wself = alpha * ihik;
    aS.init(on ? (double)wself : 0.0);
    aG.init(on ? (double)(wself * hik) : 0.0);
  }
  // a neighbour of the same feature, with no weight unless `on`
  __host__ __device__ __forceinline__ void own(const double4 &xi, const double4 &xj, bool on, Sum<CMP> &aS,
                                               Sum<CMP> &aG, Sum<CMP> *aP) const {
#pragma clang fp contract(off)
    constexpr R alpha = kalphaK<K, R>();
    const double d0 = xi.x - xj.x, d1 = xi.y - xj.y, d2 = D == 3 ? xi.z - xj.z : 0.0;
    const R dx0 = (R)d0, dx1 = (R)d1, dx2 = D == 3 ? (R)d2 : R(0);
    const R rr = sqrt_(sum2<D>(dx0, dx1, dx2));
    const R hj = (R)xj.w;
    const R hjk = powK<K>(hj);
    const R hsum = fma_(hjk, hjk, hi2k);
    const R ihij = rcp_(kl * (R(0.5) * (hi + hj)));
    const R qij = rr * ihij;
    const R w = on ? alpha * wshapeK<K>(rr * ihi) * ihik : R(0);           // W(r, h_i)
    aS.add(w);
    aG.add_term(w, hjk);
    const R ih2 = ihij * ihij;
    const R ihk2 = K == 1 ? ih2 * ihij : (K == 2 ? ih2 * ih2 : ih2 * ih2 * ihij);
    const R c = on ? P0 * hsum * alpha * dwqK<K>(qij) * ihk2 : R(0);       // (dW/dr)/r at h_ij
    aP[0].add_product(c, d0);
    aP[1].add_product(c, d1);
    if (D == 3) aP[2].add_product(c, d2);
  }
  // the boundary particle b; false where the normal is the pair's own (3D
  // patches, modes 7 and 8), which is left to the pass for those
  __host__ __device__ __forceinline__ bool boundary(const Parts &s, const double4 *__restrict__ enrm,
                                                    const BNorm *__restrict__ bnrow, int bw, double bscale,
                                                    const double4 &xi, uint32_t b, Sum<CMP> &aS,
                                                    Sum<CMP> *aB) const {
#pragma clang fp contract(off)
    constexpr R alpha = kalphaK<K, R>();
    const double4 xj = s.xh[b];
    const R dx0 = (R)(xi.x - xj.x), dx1 = (R)(xi.y - xj.y);
    const R dx2 = D == 3 ? (R)(xi.z - xj.z) : R(0);
    const R rr = sqrt_(sum2<D>(dx0, dx1, dx2));
    // the particle volume (Eq. (particle_volume)) is the inverse of i's
    // number density: the boundary particles that act on i count too
    aS.add(alpha * wshapeK<K>(rr * ihi) * ihik);
    double nv[3];
    if constexpr (K == D) {   // the volume: the domain's normal k_rank_gather stored at b
      const double4 e4 = enrm[b];
      nv[0] = e4.x;
      nv[1] = e4.y;
      nv[2] = e4.z;
    } else {
      const BNorm N = bnrow[s.f[b] & (MAXF - 1)];
      if (D == 3 && N.mode >= 7) return false;
      if (N.mode >= 2) {   // a curved boundary: the normal k_rank_gather stored
        const double4 e4 = enrm[b];
        nv[0] = e4.x;
        nv[1] = e4.y;
        nv[2] = e4.z;
      } else {
        nv[0] = N.n[0];
        nv[1] = N.n[1];
        nv[2] = N.n[2];
      }
    }
    const R hj = (R)xj.w;
    const R hjk = powK<K>(hj);
    const R hsum = fma_(hjk, hjk, hi2k);
    const R ihij = rcp_(kl * (R(0.5) * (hi + hj)));
    const R om = (bw == 0 ? rcp_(hj) : (bw == 1 ? powK<K>(hj) * rcp_(hj) : R(0))) * (R)bscale;
    const R w = alpha * wshapeK<K>(rr * ihij) * powK<K>(ihij);          // W(r, h_ib)
    const R c = P0 * hsum * w * om;
    aB[0].add_product(c, nv[0]);
    aB[1].add_product(c, nv[1]);
    if (D == 3) aB[2].add_product(c, nv[2]);
    return true;
  }
};

// Pair sums of sweep A of particle i over its neighbour list, by G lanes: lane l
// takes the entries l, l + G, ..., NB of them at a time, and the caller adds the
// lanes' sums.
template <int D, int K, typename R, bool CMP, bool PN, int NB, int G>
__host__ __device__ __forceinline__ void group_sums(const Geom &g, const Parts &s,
                                             const double4 *__restrict__ enrm,
                                             const BNorm *__restrict__ bnrow, int bw, double p0,
                                             double klen, double bscale,
                                             const uint32_t *__restrict__ nbr, int n, int i,
                                             uint32_t cnt, const double4 &xi, bool pair_normals,
                                             double &S, double &gam, double Pi[3], double B[3],
                                             LdsList ring, uint32_t ring_len, uint32_t lane) {
  const TermsA<D, K, R, CMP> T(xi.w, klen, p0);
  Sum<CMP> aS, aG, aP[3], aB[3];
  T.self(lane == 0, aS, aG);   // the self term is lane 0's
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    aP[a].init(0.0);
    aB[a].init(0.0);
  }
  // The list is in the particle's LDS ring (entry e in slot e % ring_len) when
  // the lists of all the wave's particles fit it; else it is read from memory.
  // The ring is an LDS pointer, so that the two reads stay apart (one read
  // through a selected generic pointer would be a flat load).
  const bool in_ring = !any_lane(cnt > ring_len);
  auto entry = [&](uint32_t e) -> uint32_t {
    return in_ring ? ring[(e % ring_len)] : nbr[((size_t)(e / LB) * n + i) * LB + e % LB];
  };
  // The entries of the particle's own feature, e0 + q G + lane.  The
  // passes end with the longest list of the wave, so no lane leaves the loop
  // before the others: a place past a lane's own list takes the particle
  // itself, with no weight.  Boundary entries are few and most particles have
  // none: a pass of their own keeps their registers out of this loop.
  bool boundary = false;
  for (uint32_t e0 = 0; any_lane(e0 < cnt); e0 += NB * G) {
    uint32_t u[NB];
    if (in_ring) {
#pragma unroll
      for (int q = 0; q < NB; ++q) u[q] = ring[((e0 + q * G + lane) % ring_len)];
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const uint32_t e = e0 + q * G + lane;
        u[q] = e < cnt ? nbr[((size_t)(e / LB) * n + i) * LB + e % LB] : 0u;
      }
    }
    double4 xr[NB];
    bool own[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const bool have = e0 + q * G + lane < cnt;
      own[q] = have && !(u[q] >> 31);
      boundary = boundary || (have && (u[q] >> 31));
      xr[q] = s.xh[have ? u[q] & 0x7fffffffu : (uint32_t)i];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (q > 0 && !any_lane(e0 + q * G + lane < cnt)) break;   // no list of the wave goes on
      T.own(xi, xr[q], own[q], aS, aG, aP);
    }
  }
  if (boundary) {
    for (uint32_t e = lane; e < cnt; e += G) {
      const uint32_t v = entry(e);
      if (!(v >> 31)) continue;
      (void)T.boundary(s, enrm, bnrow, bw, bscale, xi, v & 0x7fffffffu, aS, aB);
    }
  }
  if constexpr (D == 3 && K == 2) {
    // A 3D surface patch at a curve (mode 7) or vertex (8) beside it: the
    // normal is the direction to b within i's tangent plane (i's stored
    // normal removed), at a curve also without the part along b's closest
    // segment, normalised.  Only patch particles of a geometry with imported
    // curves take this pass.
    if (PN && boundary && pair_normals) {
      const double4 ei = enrm[i];
      for (uint32_t e = lane; e < cnt; e += G) {
        const uint32_t v = entry(e);
        if (!(v >> 31)) continue;
        const uint32_t b = v & 0x7fffffffu;
        const int mode = bnrow[s.f[b] & (MAXF - 1)].mode;
        if (mode < 7) continue;
        const double4 xj = s.xh[b];
        const R dx0 = (R)(xi.x - xj.x), dx1 = (R)(xi.y - xj.y), dx2 = (R)(xi.z - xj.z);
        const R rr = sqrt_(dx0 * dx0 + dx1 * dx1 + dx2 * dx2);
        double d0 = xj.x - xi.x, d1 = xj.y - xi.y, d2 = xj.z - xi.z;
        const double dm = d0 * ei.x + d1 * ei.y + d2 * ei.z;
        d0 -= dm * ei.x;
        d1 -= dm * ei.y;
        d2 -= dm * ei.z;
        if (mode == 7) {
          double t[3];
          seg_tangent<3>(g, (int)enrm[b].w, t);
          const double dt = d0 * t[0] + d1 * t[1] + d2 * t[2];
          d0 -= dt * t[0];
          d1 -= dt * t[1];
          d2 -= dt * t[2];
        }
        const double l = __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        const double il = l > 0.0 ? 1.0 / l : 0.0;
        const R hj = (R)xj.w;
        const R hjk = powK<K>(hj);
        const R hsum = T.hi2k + hjk * hjk;
        const R ihij = rcp_(T.kl * (R(0.5) * (T.hi + hj)));
        const R om = (bw == 0 ? rcp_(hj) : (bw == 1 ? powK<K>(hj) * rcp_(hj) : R(0))) * (R)bscale;
        const R w = kalphaK<K, R>() * wshapeK<K>(rr * ihij) * powK<K>(ihij);      // W(r, h_ib)
        const R c = T.P0 * hsum * w * om;
        aB[0].add_product(c, d0 * il);
        aB[1].add_product(c, d1 * il);
        aB[2].add_product(c, d2 * il);
      }
    }
  }
  S = aS.get();
  gam = aG.get();
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    Pi[a] = aP[a].get();
    B[a] = aB[a].get();
  }
}

// The sums by one lane in list order, each entry's terms as they come (2D).  With
// nlanes > 1, and in 3D, which has no such kernel: those of lane `lane` of
// k_nbr_group (host callers).
template <int D, int K, typename R, bool CMP>
__host__ __device__ __forceinline__ void sweep_a_sums(const Geom &g, const Parts &s,
                                             const double4 *__restrict__ enrm,
                                             const BNorm *__restrict__ bnrow, int bw, double p0,
                                             double klen, double bscale,
                                             const uint32_t *__restrict__ nbr, int n, int i,
                                             uint32_t cnt, const double4 &xi, int fi, bool pair_normals,
                                             double &S, double &gam, double Pi[3], double B[3],
                                             const uint32_t *ring = nullptr, uint32_t ring_len = 0,
                                             uint32_t ring_stride = 0, uint32_t lane = 0,
                                             uint32_t nlanes = 1) {
  if (D == 3 || nlanes > 1) {
    auto split = [&](auto lanes) {
      group_sums<D, K, R, CMP, true, 4, decltype(lanes)::value>(g, s, enrm, bnrow, bw, p0, klen, bscale, nbr, n, i,
                                                                cnt, xi, pair_normals, S, gam, Pi, B, nullptr, 0,
                                                                lane);
    };
    if (nlanes <= 1) split(std::integral_constant<int, 1>());
    else if (nlanes == 2) split(std::integral_constant<int, 2>());
    else if (nlanes == 4) split(std::integral_constant<int, 4>());
    else split(std::integral_constant<int, 8>());
    return;
  }
  // h enters rho_t = h^-k; the kernel is evaluated at the smoothing length
  // klen h (cut-off radius 2 klen h)
  const R hi = (R)xi.w;
  const R kl = (R)klen;
  const R ihi = rcp_((R)(klen * xi.w));
  constexpr R alpha = kalphaK<K, R>();
  const R hik = powK<K>(hi), hi2k = hik * hik;
  const R ihik = powK<K>(ihi);
  const R P0 = (R)p0;
  const R wself = alpha * ihik;
  Sum<CMP> aS, aG, aP[2], aB[2];
  aS.init((double)wself);
  aG.init((double)(wself * hik));
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    aP[a].init(0.0);
    aB[a].init(0.0);
  }
  constexpr int NB = SPH_NBATCH;
  static_assert(NB == 4 || NB == LB, "record batches of 4 or 8 tile a list block");
  // records gathered together: GB of a batch's NB (fewer live registers)
  constexpr int GB = SPH_GBATCH < NB ? SPH_GBATCH : NB;
  static_assert(NB % GB == 0, "gather groups tile a batch");
  // The list's last entries may also sit in the caller's LDS ring (entry e
  // in slot e % ring_len, column stride ring_stride): entries from lbase on
  // are read there, the ones before from the list in memory (whole blocks,
  // as lbase is a multiple of LB).  Either way every entry is read in list
  // order, so the sums are the same.
  uint32_t lbase = cnt;
  if (ring != nullptr) lbase = cnt > ring_len ? (cnt - ring_len + LB - 1) / LB * LB : 0u;
  const uint4 *gl = reinterpret_cast<const uint4 *>(nbr) + (size_t)i * (LB / 4);
  for (uint32_t e0 = 0; e0 < cnt; e0 += NB) {
    {
      uint32_t u[NB];
      if (e0 < lbase) {   // NB entries of a block in memory: 16-byte loads
#pragma unroll
        for (int h = 0; h < NB / 4; ++h) {
          const uint4 w = gl[(size_t)(e0 / LB) * n * (LB / 4) + (e0 % LB) / 4 + h];
          u[4 * h] = w.x;
          u[4 * h + 1] = w.y;
          u[4 * h + 2] = w.z;
          u[4 * h + 3] = w.w;
        }
      } else {
#pragma unroll
        for (int q = 0; q < NB; ++q) u[q] = ring[((e0 + q) % ring_len) * ring_stride];
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) u[q] = e0 + q < cnt ? u[q] : 0u;
#pragma unroll
      for (int g0 = 0; g0 < NB; g0 += GB) {
      double4 xr[GB];
#pragma unroll
      for (int q = 0; q < GB; ++q) xr[q] = s.xh[u[g0 + q] & 0x7fffffffu];
#pragma unroll
      for (int qg = 0; qg < GB; ++qg) {
        const int q = g0 + qg;
        if (e0 + q >= cnt) break;
        const double4 xj = xr[qg];
        const R dx0 = (R)(xi.x - xj.x), dx1 = (R)(xi.y - xj.y);
        const R rr = sqrt_(dx0 * dx0 + dx1 * dx1);
        const R hj = (R)xj.w;
        const R hjk = powK<K>(hj);
        const R hsum = hi2k + hjk * hjk;
        const R ihij = rcp_(kl * (R(0.5) * (hi + hj)));
        const R qij = rr * ihij;
        if (!(u[q] >> 31)) {
          const R w = alpha * wshapeK<K>(rr * ihi) * ihik;           // W(r, h_i)
          aS.add(w);
          aG.add(w * hjk);
          const R ih2 = ihij * ihij;
          const R ihk2 = K == 1 ? ih2 * ihij : (K == 2 ? ih2 * ih2 : ih2 * ih2 * ihij);
          const R c = P0 * hsum * alpha * dwqK<K>(qij) * ihk2;       // (dW/dr)/r at h_ij
          aP[0].add(c * dx0);
          aP[1].add(c * dx1);
        } else {
          // the particle volume (Eq. (particle_volume)) is the inverse of i's
          // number density: the boundary particles that act on i count too
          aS.add(alpha * wshapeK<K>(rr * ihi) * ihik);
          double nv[2];
          if constexpr (K == D) {   // the volume: the domain's normal k_rank_gather stored at b
            const double4 e = enrm[u[q] & 0x7fffffffu];
            nv[0] = e.x;
            nv[1] = e.y;
          } else {
            const int fj = s.f[u[q] & 0x7fffffffu];
            const BNorm N = bnrow[fj & (MAXF - 1)];
            if (N.mode >= 2) {   // a curved boundary: the normal k_rank_gather stored
              const double4 e = enrm[u[q] & 0x7fffffffu];
              nv[0] = e.x;
              nv[1] = e.y;
              } else {
              nv[0] = N.n[0];
              nv[1] = N.n[1];
            }
          }
          const R om = (bw == 0 ? rcp_(hj) : (bw == 1 ? powK<K>(hj) * rcp_(hj) : R(0))) * (R)bscale;
          const R w = alpha * wshapeK<K>(qij) * powK<K>(ihij);          // W(r, h_ib)
          if constexpr (CMP) {   // FP32 terms: the normal rounded to FP32
            const float c = (float)(P0 * hsum * w * om);
            aB[0].add(c * (float)nv[0]);
            aB[1].add(c * (float)nv[1]);
          } else {
            const double c = (double)(P0 * hsum * w * om);
            aB[0].add(c * nv[0]);
            aB[1].add(c * nv[1]);
          }
        }
      }
      }
    }
  }
  S = aS.get();
  gam = aG.get();
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    Pi[a] = aP[a].get();
    B[a] = aB[a].get();
  }
  Pi[2] = B[2] = 0.0;
}

// The sums of group_sums by one lane for four (2D): entry e in sum e % 4, own
// entries first, then the boundary's, and the four added as group_sum adds the
// lanes'.  Same bits, in the registers of one lane.
template <int K, typename R, bool CMP>
__host__ __device__ __forceinline__ void four_sums(const Parts &s, const double4 *__restrict__ enrm,
                                                   const BNorm *__restrict__ bnrow, int bw, double p0, double klen,
                                                   double bscale, const uint32_t *__restrict__ nbr, int n, int i,
                                                   uint32_t cnt, const double4 &xi, double &S, double &gam,
                                                   double Pi[3], double B[3], const uint32_t *ring,
                                                   uint32_t ring_len, uint32_t ring_stride) {
  constexpr int D = 2, V = 4;
  auto total = [](const Sum<CMP> &a, const Sum<CMP> &b, const Sum<CMP> &c, const Sum<CMP> &d) {
    return (a.get() + b.get()) + (c.get() + d.get());
  };
  const TermsA<D, K, R, CMP> T(xi.w, klen, p0);
  Sum<CMP> aS[V], aG[V], aP[V][3];
#pragma unroll
  for (int l = 0; l < V; ++l) {
    T.self(l == 0, aS[l], aG[l]);
#pragma unroll
    for (int a = 0; a < 3; ++a) aP[l][a].init(0.0);
  }
  constexpr int NB = SPH_NBATCH;
  static_assert((NB == 4 || NB == LB) && NB % V == 0, "record batches of 4 or 8 tile a list block");
  // records gathered together: GB of a batch's NB (fewer live registers)
  constexpr int GB = SPH_GBATCH < NB ? SPH_GBATCH : NB;
  static_assert(NB % GB == 0, "gather groups tile a batch");
  // The list's last entries may also sit in the caller's LDS ring (entry e
  // in slot e % ring_len, column stride ring_stride): entries from lbase on
  // are read there, the ones before from the list in memory (whole blocks,
  // as lbase is a multiple of LB).  Either way every entry is read in list
  // order, so the sums are the same.
  uint32_t lbase = cnt;
  if (ring != nullptr) lbase = cnt > ring_len ? (cnt - ring_len + LB - 1) / LB * LB : 0u;
  const uint4 *gl = reinterpret_cast<const uint4 *>(nbr) + (size_t)i * (LB / 4);
  auto batch = [&](uint32_t e0, uint32_t (&u)[NB]) {
    if (e0 < lbase) {   // NB entries of a block in memory: 16-byte loads
#pragma unroll
      for (int h = 0; h < NB / 4; ++h) {
        const uint4 w = gl[(size_t)(e0 / LB) * n * (LB / 4) + (e0 % LB) / 4 + h];
        u[4 * h] = w.x;
        u[4 * h + 1] = w.y;
        u[4 * h + 2] = w.z;
        u[4 * h + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q) u[q] = ring[((e0 + q) % ring_len) * ring_stride];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) u[q] = e0 + q < cnt ? u[q] : 0u;
  };
  uint32_t boundary = 0u;   // its top bit: some entry is of the boundary
  for (uint32_t e0 = 0; e0 < cnt; e0 += NB) {
    uint32_t u[NB];
    batch(e0, u);
#pragma unroll
    for (int g0 = 0; g0 < NB; g0 += GB) {
      double4 xr[GB];
#pragma unroll
      for (int q = 0; q < GB; ++q) xr[q] = s.xh[u[g0 + q] & 0x7fffffffu];
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        if (e0 + g0 + q >= cnt) break;
        const uint32_t v = u[g0 + q];
        boundary |= v;
        T.own(xi, xr[q], !(v >> 31), aS[(g0 + q) % V], aG[(g0 + q) % V], aP[(g0 + q) % V]);
      }
    }
  }
  gam = total(aG[0], aG[1], aG[2], aG[3]);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    Pi[a] = total(aP[0][a], aP[1][a], aP[2][a], aP[3][a]);
    B[a] = 0.0;
  }
  if (boundary >> 31) {
    Sum<CMP> aB[V][3];
#pragma unroll
    for (int l = 0; l < V; ++l)
#pragma unroll
      for (int a = 0; a < 3; ++a) aB[l][a].init(0.0);
    for (uint32_t e0 = 0; e0 < cnt; e0 += NB) {
      uint32_t u[NB];
      batch(e0, u);
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (u[q] >> 31)
          (void)T.boundary(s, enrm, bnrow, bw, bscale, xi, u[q] & 0x7fffffffu, aS[q % V], aB[q % V]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) B[a] = total(aB[0][a], aB[1][a], aB[2][a], aB[3][a]);
  }
  S = total(aS[0], aS[1], aS[2], aS[3]);
  Pi[2] = B[2] = 0.0;
}

// Appends the hits among tag[0, NB) (0xffffffff: no hit) to a particle's
// column of the LDS ring (slot k at rc[k * stride], slot = entry mod LR) and
// stores each list block they complete to *wp as two 16-byte writes, while
// the capacity of nblk blocks allows.  With a ring of two blocks or more the
// block a batch completes is still whole after the batch (NB <= LB hits
// reach at most LB - 1 entries into the next block), so the test for a
// store runs once per batch instead of once per hit.
template <int NB, int LR>
__host__ __device__ __forceinline__ void append_hits(const uint32_t (&tag)[NB], uint32_t *rc,
                                                     int stride, uint32_t &count, uint4 *&wp,
                                                     uint32_t wstep, uint32_t nblk) {
  static_assert(NB <= LB && LR % LB == 0, "a batch completes at most one block");
  if constexpr (LR >= 2 * LB) {
    const uint32_t c0 = count;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (tag[q] != 0xffffffffu) {
        rc[(count % LR) * stride] = tag[q];
        ++count;
      }
    }
    if (count / LB != c0 / LB && count / LB <= nblk) {
      const uint32_t k0 = (c0 / LB * LB) % LR;
      wp[0] = make_uint4(rc[k0 * stride], rc[(k0 + 1) * stride], rc[(k0 + 2) * stride],
                         rc[(k0 + 3) * stride]);
      wp[1] = make_uint4(rc[(k0 + 4) * stride], rc[(k0 + 5) * stride], rc[(k0 + 6) * stride],
                         rc[(k0 + 7) * stride]);
      wp += wstep;
    }
  } else {
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (tag[q] != 0xffffffffu) {
        const uint32_t k = count % LR;
        rc[k * stride] = tag[q];
        ++count;
        if (k % LB == LB - 1 && count / LB <= nblk) {
          const uint32_t k0 = k - (LB - 1);
          wp[0] = make_uint4(rc[k0 * stride], rc[(k0 + 1) * stride], rc[(k0 + 2) * stride],
                             rc[(k0 + 3) * stride]);
          wp[1] = make_uint4(rc[(k0 + 4) * stride], rc[(k0 + 5) * stride], rc[(k0 + 6) * stride],
                             rc[(k0 + 7) * stride]);
          wp += wstep;
        }
      }
    }
  }
}

// the classification's band (JobDev) of a particle that lies outside its job's
// box, where the caller may have put it
template <int D, int MODE>
__device__ __forceinline__ void band_beyond(const JobDev &J, const double4 &xi, float &cin, float &cout) {
  double xb = __builtin_fabs(xi.x);
  xb = __builtin_fabs(xi.y) > xb ? __builtin_fabs(xi.y) : xb;
  if (D == 3) xb = __builtin_fabs(xi.z) > xb ? __builtin_fabs(xi.z) : xb;
  xb += 2.0 * J.rmax_s + 2.0 * J.G.cmax;
  const double w = (D == 2 ? 2e-6 : 2e-5) +
                   (D == 3 ? 1.7320508075688772 : 1.4142135623730951) * 0x1p-23 * xb * 1.01 * J.iband;
  const double k = MODE == 1 ? 0.5 * J.ksup_s : J.klen;
  cin = w < 1.0 ? (float)((1.0 - w) * (1.0 - w) * k * k) : -1.0f;
  cout = (float)((1.0 + w) * (1.0 + w) * k * k);
}

// a word of a record that no kernel of the launch writes, at an address all
// lanes of the wave share: one scalar load, and no vector register
template <typename T>
__device__ __forceinline__ T sload(const T &v) {
  return *(const T __attribute__((address_space(4))) *)(uintptr_t)&v;
}

// Jobs that a launch covers: a block works on particles of one job,
// so that the job's record is uniform.  One job is passed by value; several
// are looked up by their first block.
static_assert(MAXJ <= 64, "a lane per span");
struct Span {
  int block, job, first, end;   // first block; the job's slot; its particles' slots
};
struct Spans {
  int count;
  Span one;
  const Span *tab;
};
__device__ __forceinline__ void span_of(const Spans &sp, int b, int pb, int &job, int &first, int &end) {
  Span s = sp.one;
  if (sp.count > 1) {   // the last span that starts at b or before: a lane per span
    const int l = __lane_id();
    const bool at = l < sp.count && sp.tab[l].block <= b;
    const int k = __popcll(__builtin_amdgcn_ballot_w64(at)) - 1;
    const Span *t = sp.tab + k;
    s.block = sload(t->block);
    s.job = sload(t->job);
    s.first = sload(t->first);
    s.end = sload(t->end);
  }
  job = s.job;
  first = s.first + (b - s.block) * pb;
  end = s.end;
}

// ---------------------------------------------------------------------------
// neighbour list (Algorithm 1 "construct Verlet neighbor list") and, in the
// same launch, sweep A over it; FORCES = false builds lists only.  Two kernels
// make the same lists: k_nbr_forces, one lane per particle, and k_nbr_group, G
// lanes per particle.  The candidate scan covers, for every cell row within
// R_i of x_i, only the cells under the chord of the disc (sphere) of radius
// R_i, so no neighbour is skipped and fewer non-neighbours are tested.  The pair
// sums then run over the list just written, so the force math executes once
// per neighbour instead of once per candidate.  Every particle reads its own
// job's geometry and grid; cells of different jobs never meet.
//
// k_nbr_forces: one lane per particle, a block on particles of one job.  It is the
// faster for large 2D batches (small_job, launch_build), whose short lists do not
// fill several lanes: of 1,000,000 particles, FP32, cell scan, 117 us against 135
// with 2 lanes and 148 with 4; the list build 170 against 225 us.
// MODE 0: candidates from the cell scan, as above.  MODE 1 (FORCES = false,
// only when a rebuild is due): the Verlet candidate list of every
// non-singular particle, the cell scan at the reach (c + delta) h with the
// FP32 test alone, widened by its error bound so that it keeps every pair
// within that reach.
// ---------------------------------------------------------------------------
template <typename R, bool FORCES, int NB, bool CMP, int MODE, int SUMS>
__global__ __launch_bounds__(BLOCK, SUMS != AS_ONE && sizeof(R) == 8 ? 4 : 1) void k_nbr_forces(
    Batch B, Parts s, const uint32_t *__restrict__ cstart, int all, uint32_t *__restrict__ nbr,
    uint32_t *__restrict__ nnb, typename Vec4<R>::T *__restrict__ ap,
    double *__restrict__ dbg_gam, double *__restrict__ dbg_vt, Parts home, Spans sp) {
  constexpr int D = 2;
  static_assert(MODE == 0 || (MODE == 1 && !FORCES), "candidate list modes");
  if (MODE == 1) {
    if (B.vstate[VS_REBUILD] == 0ull) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) B.vstate[VS_BUILDS] += 1ull;
  }
  // the block's job and its particles [first, end)
  int job, first, end;
  span_of(sp, xcd_block(), BLOCK, job, first, end);
  if (MODE == 1) {
    // s holds the particles just sorted; they go back to the buffer the
    // steps use between rebuilds (no kernel of this launch reads it)
    const int c = first + (int)threadIdx.x;
    if (c < end) {
      home.xh[c] = s.xh[c];
      home.v[c] = s.v[c];
      home.f[c] = s.f[c];
      home.oid[c] = s.oid[c];
      home.xf[c] = s.xf[c];
    }
  }
  using R4 = typename Vec4<R>::T;
  // hits collect in the thread's own column of an LDS ring of LR entries (a
  // multiple of LB; see the append below); it keeps the last LR entries, so
  // that in the FP32 modes a list no longer than LR stays whole in LDS,
  // where the pair sums read it (the FP64 sums read the list from memory:
  // the ring's addressing would cost them a wave per SIMD); the Verlet build
  // keeps two blocks, so that its block stores are tested once per batch
  constexpr bool LDS_SUMS = FORCES && sizeof(R) == 4;
  constexpr int LR = LDS_SUMS ? SPH_LDS_LIST : (MODE == 1 ? 2 * LB : LB);
  static_assert(LR % LB == 0, "the ring holds whole blocks");
  __shared__ uint32_t ring[LR][BLOCK];
  const int col = (int)threadIdx.x;
  const int n = B.n;
  const int i = first + (int)threadIdx.x;
  bool act = false;
  int fi = 0;
  unsigned long long dtb = ~0ull, vfix = 0ull, mine = 0ull;
  const JobDev &J = B.jobs[job];
  if (i < end) {
    fi = s.f[i];
    const Feat F = B.feat[fi];
    const bool moving = F.type != T_SI && B.grp[fi].active;
    const bool want = F.type != T_SI && (all || MODE == 1 || B.grp[fi].active);
    act = FORCES && moving;
    uint32_t count = 0;
    const double4 xi = s.xh[i];
    if (want) {
      const Grid &G = J.G;
      // scan reach: the cut-off radius, or the Verlet list's in MODE 1
      const double ksup = MODE == 1 ? J.ksup_s : J.ksup;
      double Rs = (MODE == 1 ? J.rfac_s : G.rfac) * xi.w;
      const double rmax = MODE == 1 ? J.rmax_s : G.rmax;
      Rs = Rs < rmax ? Rs : rmax;
      const double pc[2] = {xi.x, xi.y};
      // cell levels that can hold a neighbour: h is L-Lipschitz, so a
      // neighbour (r < R_i) has |h_j - h_i| <= L R_i (widened for rounding)
      int lv0 = 0, lv1 = G.nlev - 1;
      if (G.nlev > 1) {
        const double dh = G.lip * Rs * (1.0 + 1e-9);
        lv0 = h_level(G, (xi.w - dh) * (1.0 - 1e-12));
        lv1 = h_level(G, (xi.w + dh) * (1.0 + 1e-12));
      }
      // features that bound fi (bit = local feature id); a candidate of fi's
      // own feature interacts as "same", one of a bounding feature of the same
      // job as "boundary".  The scan only visits cells of i's own job, so a
      // candidate's feature slot is in i's job range and its local id is its
      // low 6 bits.
      const unsigned long long accept = B.bmask[fi] | (1ull << (fi & (MAXF - 1)));
      const double kc2 = J.ksup2;   // c^2, c = support radius / h
      const double A4 = kc2 * (xi.w * xi.w);
      // Candidates are classified in FP32 from the scan records (which hold
      // 2h) by the job's band (JobDev): a certain neighbour below H^2 band_in, a
      // certain non-neighbour above H^2 band_out, H = 2 max(h_i, h_j); in
      // between the exact FP64 predicate decides, so the classification always
      // equals it
      const float4 xif = scan_record<D>(xi, (uint32_t)fi);
      const float Hif = xif.z;
      float cin = J.band_in, cout = MODE == 1 ? J.band_reach : J.band_out;
      if (__builtin_fabs(xi.x) > J.band_x || __builtin_fabs(xi.y) > J.band_x)
        band_beyond<D, MODE>(J, xi, cin, cout);
      static_assert(NB >= 1 && NB <= 8, "records are padded by 8");
      // hits collect in the thread's own column of the LDS ring (entry-major,
      // so the lanes of a wave hit distinct banks whatever their fill); each
      // block of LB entries is stored as one 32-byte sector when full (and
      // the last once more, partly filled, at the end).  One LDS write per
      // hit replaces a select over LB registers, which every lane would
      // execute whenever any lane of the wave hits.
      static_assert(LB == 8, "the ring is flushed as two 16-byte stores");
      uint4 *wp = reinterpret_cast<uint4 *>(MODE == 1 ? B.skin : nbr) + (size_t)i * (LB / 4);
      const uint32_t wstep = (uint32_t)n * (LB / 4);
      const uint32_t nblk = (uint32_t)(MODE == 1 ? B.skin_cap : B.cap) / LB;   // blocks of capacity
      for (int lv = lv0; lv <= lv1; ++lv) {
        // a level-lv candidate has h_j < hcap[lv], so none beyond
        // c max(h_i, hcap[lv]) is a neighbour
        double Rl = ksup * (xi.w > G.hcap[lv] ? xi.w : G.hcap[lv]) * (1.0 + 1e-9);
        Rl = Rl < Rs ? Rl : Rs;
        const double R2 = Rl * Rl;
        const int ylo = cell_coord(G, lv, 1, pc[1] - Rl), yhi = cell_coord(G, lv, 1, pc[1] + Rl);
        // grid values the row loop needs, kept in registers
        const double c0 = G.c[lv][0], inv0 = G.inv_c[lv][0], lo1 = G.lo[1], c1 = G.c[lv][1];
        const uint32_t nc0 = (uint32_t)G.nc[lv][0];
        const uint32_t cbase = G.cbase + G.lbase[lv];
        const double u0 = (pc[0] - G.lo[0]) * inv0;     // x of i in cell units
        const double top0 = (double)(G.nc[lv][0] - 1);
        for (int cy = ylo; cy <= yhi; ++cy) {
          const double y0 = lo1 + cy * c1;
          double dy = y0 - pc[1] > pc[1] - (y0 + c1) ? y0 - pc[1] : pc[1] - (y0 + c1);
          dy = dy - 1e-7 * c1;
          dy = dy > 0.0 ? dy : 0.0;
          const double w2 = R2 - dy * dy;
          if (w2 < 0.0) continue;
          // half chord of the row; the FP32 square root (error < 2e-7
          // relative) is covered by the 1e-6 relative widening
          const double wx = (double)sqrt_((float)w2) * (1.0 + 1e-6) + 1e-7 * c0;
          const double wu = wx * inv0;
          double t0 = __builtin_floor(u0 - wu), t1 = __builtin_floor(u0 + wu);
          t0 = t0 >= 0.0 ? t0 : 0.0;   // also maps NaN to cell 0
          t1 = t1 >= 0.0 ? t1 : 0.0;
          t0 = t0 < top0 ? t0 : top0;
          t1 = t1 < top0 ? t1 : top0;
          const uint32_t row = cbase + cell_row<D>(G, lv, (uint32_t)cy, 0u) * nc0;
          const uint32_t jb = cstart[row + (uint32_t)t0], je = cstart[row + (uint32_t)t1 + 1];
          // NB candidates per pass: records loaded together (the arrays are
          // padded by 8 past the capacity), the predicate evaluated for all of
          // them without early exits, then the hits appended in order
          for (uint32_t j0 = jb; j0 < je; j0 += NB) {
            const float4 *rp = s.xf + j0;
            float4 xr[NB];
            uint32_t fr[NB];   // job-local feature id of the candidate
#pragma unroll
            for (int q = 0; q < NB; ++q) {
              xr[q] = rp[q];
              fr[q] = __float_as_uint(xr[q].w) & (MAXF - 1);
            }
            uint32_t tag[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) {
              const uint32_t j = j0 + q;
              const bool rel = (accept >> (fr[q] & (MAXF - 1))) & 1ull;
              const bool cand = rel & (j < je) & (j != (uint32_t)i);
              const float ex = xif.x - xr[q].x, ey = xif.y - xr[q].y;
              const float d2 = ex * ex + ey * ey;
              const float H = __builtin_fmaxf(Hif, xr[q].z);
              const float H2 = H * H;
              const float tin = H2 * cin, tout = H2 * cout;
              bool hit;
              if constexpr (MODE == 1) {   // Verlet list: all that may lie within reach
                hit = cand & !(d2 > tout);
              } else {
                hit = cand & (d2 < tin);
                if (cand & !(d2 < tin) & !(d2 > tout))   // near the support radius: exact test
                  hit = within_a4<D>(xi, A4, kc2, s.xh[j]);
              }
              tag[q] = hit ? (j | (fr[q] == (uint32_t)(fi & (MAXF - 1)) ? 0u : 0x80000000u))
                           : 0xffffffffu;
            }
            append_hits<NB, LR>(tag, &ring[0][col], BLOCK, count, wp, wstep, nblk);
          }
        }
      }
      if (count % LB != 0 && count / LB < nblk) {   // the last, partly filled block
        const uint32_t k0 = (count / LB * LB) % LR;
        wp[0] = make_uint4(ring[k0][col], ring[k0 + 1][col], ring[k0 + 2][col], ring[k0 + 3][col]);
        wp[1] = make_uint4(ring[k0 + 4][col], ring[k0 + 5][col], ring[k0 + 6][col], ring[k0 + 7][col]);
      }
      if (MODE == 1 && (int)count > B.skin_cap) {
        atomicMax(&B.st[job].skin_max, count);
        atomicExch(&B.st[job].skin_overflow, 1u);
        count = B.skin_cap;
      } else if (MODE != 1 && (int)count > B.cap) {
        atomicMax(&B.st[job].overflow_max, count);
        atomicExch(&B.st[job].overflow, 1u);
        count = B.cap;
      }
    }
    if (FORCES && act) {
      const int k = F.k;
      double4 v4 = s.v[i];
      if (B.grp[fi].reset_now) {
        v4 = make_double4(0.0, 0.0, 0.0, 0.0);
        s.v[i] = v4;
      }
      const BNorm *bnrow = B.bn + (size_t)fi * MAXF;
      double S, gam, Pi[3], B3[3];
      const uint32_t *rg = LDS_SUMS ? &ring[0][col] : nullptr;
      if (SUMS == AS_FOUR || (SUMS == AS_JOB && J.four)) {
        if (k == D)
          four_sums<D, R, CMP>(s, B.enrm, bnrow, J.bw, J.p0, J.klen, J.bscale, nbr, n, i, count, xi, S, gam, Pi, B3,
                               rg, LR, BLOCK);
        else
          four_sums<1, R, CMP>(s, B.enrm, bnrow, J.bw, J.p0, J.klen, J.bscale, nbr, n, i, count, xi, S, gam, Pi, B3,
                               rg, LR, BLOCK);
      } else {
        if (k == D)
          sweep_a_sums<D, D, R, CMP>(J.g, s, B.enrm, bnrow, J.bw, J.p0, J.klen, J.bscale, nbr, n, i, count, xi, fi,
                                     false, S, gam, Pi, B3, rg, LR, BLOCK);
        else
          sweep_a_sums<D, 1, R, CMP>(J.g, s, B.enrm, bnrow, J.bw, J.p0, J.klen, J.bscale, nbr, n, i, count, xi, fi,
                                     false, S, gam, Pi, B3, rg, LR, BLOCK);
      }
      // the FP32 modes store a^p in FP32 and hold V~ and the time steps to
      // 1e-5: FP32 reciprocals and roots suffice there (relative error 2^-23)
      constexpr bool F32 = sizeof(R) == 4;
      double a3[3] = {0.0, 0.0, 0.0};
      const double ig = F32 ? (double)rcp_((float)gam) : 0.0;
#pragma unroll
      for (int a = 0; a < D; ++a) a3[a] = F32 ? -((Pi[a] + B3[a]) * ig) : -((Pi[a] + B3[a]) / gam);
      double xa[3] = {xi.x, xi.y, xi.z};
      tangent_at<D>(J.g, F, xa, B.enrm, i, a3);
      // in 2D the record's free slots carry v^n (after any reset) in the
      // sweep precision, so sweep B gathers one record per neighbour less
      R4 o;
      o.x = (R)a3[0];
      o.y = (R)a3[1];
      o.z = (R)v4.x;
      o.w = (R)v4.y;
      const double vt = F32 ? (double)rcp_((float)S) : 1.0 / S;
      ap[i] = o;
      if (dbg_gam) dbg_gam[i] = gam;
      if (dbg_vt) dbg_vt[i] = vt;
      // Eq. (fa_time_step_size) terms from a^p and v^n
      const double rc = J.ksup * xi.w;
      const double dt = step_terms<F32>(rc, sum2<3>(a3[0], a3[1], a3[2]), sum2<3>(v4.x, v4.y, v4.z));
      dtb = dbits(dt);
      vfix = (unsigned long long)__builtin_llrint(vt * B.grp[fi].vscale);
    } else if (FORCES) {
      R4 z;
      z.x = z.y = z.z = z.w = R(0);
      ap[i] = z;
      if (dbg_gam) dbg_gam[i] = 0.0;
      if (dbg_vt) dbg_vt[i] = 0.0;
    }
    if (MODE == 1) {
      B.nsk[i] = count;
    } else {
      nnb[i] = count;
      mine = count;
    }
  }
  if (FORCES) {
    wave_commit(act, fi, dtb, vfix, B.smin, DT1, B.ssum);
    wave_count(i < end && mine != 0ull, job, mine, B.scnt, SC_PAIRS);
  }
}

// A position of u cells along an axis as whole cells and a fraction.  A
// particle the caller put 2^30 cells or farther off the grid (of at most 2^29
// cells) is taken to be that far off: its ranges end in the same border cells,
// and a whole part plus a half chord stays an int.  On the device the conversion
// saturates (and gives 0 for a NaN, which has no neighbours), so that the limits
// are integers: of 1,000,000 particles in 3D, FP32, 505.6 us, clamped as doubles
// 510.7 (without limits 506.1).
__host__ __device__ __forceinline__ void cell_split(double u, int &whole, float &frac) {
  constexpr int FAR = 1 << 30;
  const double f = __builtin_floor(u);
#ifdef __HIP_DEVICE_COMPILE__
  asm("v_cvt_i32_f64 %0, %1" : "=v"(whole) : "v"(f));
  whole = whole < FAR ? whole : FAR;
  whole = whole > -FAR ? whole : -FAR;
#else
  whole = f < FAR ? (f > -FAR ? (int)f : -FAR) : FAR;
#endif
  frac = (float)(u - f);
}
// the cells [t0, t1] of a row of nc that a half chord of w cells about that position touches
__host__ __device__ __forceinline__ void row_range(int whole, float frac, float w, int nc, int &t0, int &t1) {
  w = __builtin_fminf(w, 1e9f);
  t0 = whole + (int)__builtin_floorf(frac - w);
  t1 = whole + (int)__builtin_floorf(frac + w);
  t0 = t0 > 0 ? (t0 < nc - 1 ? t0 : nc - 1) : 0;
  t1 = t1 > 0 ? (t1 < nc - 1 ? t1 : nc - 1) : 0;
}

// ---------------------------------------------------------------------------
// lanes of one group of G (aligned) exchange values by DPP
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = dbits(v);
  const uint32_t lo = dpp_u32<CTRL>((uint32_t)b), hi = dpp_u32<CTRL>((uint32_t)(b >> 32));
  return bitsd(((unsigned long long)hi << 32) | lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_SHR1 = 0x111,
              DPP_SHR2 = 0x112, DPP_SHR4 = 0x114;
// sum over the group, the same bits in every lane (each step adds the same
// two partial sums in either order)
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_f64<DPP_XOR1>(v);
  if (G >= 4) v += dpp_f64<DPP_XOR2>(v);
  if (G == 8) v += dpp_f64<DPP_HALF_MIRROR>(v);
  return v;
}
template <int G>
__device__ __forceinline__ uint32_t group_or(uint32_t v) {
  v |= dpp_u32<DPP_XOR1>(v);
  if (G >= 4) v |= dpp_u32<DPP_XOR2>(v);
  if (G == 8) v |= dpp_u32<DPP_HALF_MIRROR>(v);
  return v;
}
// inclusive prefix sum over the group's lanes (gl the lane in the group)
template <int G>
__device__ __forceinline__ uint32_t group_scan(uint32_t v, int gl) {
  uint32_t t = dpp_u32<DPP_SHR1>(v);
  v += gl >= 1 ? t : 0u;
  if (G >= 4) {
    t = dpp_u32<DPP_SHR2>(v);
    v += gl >= 2 ? t : 0u;
  }
  if (G == 8) {
    t = dpp_u32<DPP_SHR4>(v);
    v += gl >= 4 ? t : 0u;
  }
  return v;
}


// ---------------------------------------------------------------------------
// neighbour list (Algorithm 1 "construct Verlet neighbor list") and, in the
// same launch, sweep A over it, G lanes per particle; FORCES = false builds
// the lists only.
// MODE 0: candidates from the cell scan: for every cell row within R_i of x_i
// the cells under the chord of the disc (sphere) of radius R_i.  MODE 1
// (FORCES = false, only when a rebuild is due): the Verlet candidate list of
// every non-singular particle, the cell scan at the reach (c + delta) h with
// the FP32 test alone, widened by its error bound so that it keeps every pair
// within that reach.  MODE 2: candidates from the particle's Verlet list.
//
// A particle's candidates are one stream of places.  The cell scan's ranges are
// laid end to end: each lane of the group works out one row, a prefix sum places
// the ranges, the rows that start within the next WIN places are a bit mask,
// and a lane counts in it to find its row.  The group takes WIN places at a time
// (G consecutive ones per load, so a row's records come in few cache lines);
// hits collect in the particle's LDS ring in the order of their places, in
// whole blocks to memory, and the pair sums read them there.  Loops end with
// the longest list of the wave and run without divergence.  PN: geometries
// whose patches need pair normals (group_sums).
//
// With one lane per particle a launch of few particles leaves most of the chip
// idle behind one long serial chain per lane, and a launch of many waits for
// gathers that 4 waves of 120+ registers hide badly.  G lanes make the chain
// shorter and the waves more; one job per block makes its record scalar.  Verlet
// lists take 64 to 80 registers in FP32 and 80 to 96 in FP64.  us per launch before
// and now: 4,352 particles in 2D, FP64, 25.7 / 14; 2,503, FP32, 29.4 / 14; cube
// minus ball with the cell scan and a reach of 2.5h, 66,000, FP32, 238 / 78; Verlet
// lists of 30,000, FP64, 57 / 26 (their builds, a step's share, 46 / 11); 300,000
// between ellipsoids 241 / 190 (351 / 152); 2,000,000, FP32, 684 / 528 (211 / 201).
// The arithmetic of the sums and the gathers bound it from 100,000 particles up, the
// chain of dependent loads below.  The cell scan is bound to 96 registers, 5 waves a
// SIMD instead of 4, for 4 spilled in 2D and 17 to 19 (72 to 80 bytes a lane) in 3D:
// 66,000 particles 85 / 78, the ellipsoids' build 172 / 152; with 6 waves (3D, 80
// registers, 200 bytes spilled) 127 and 160.
// ---------------------------------------------------------------------------
template <int D, typename R, bool FORCES, bool CMP, int MODE, int G, bool PN>
__global__ __launch_bounds__(BLOCK, MODE == 2 && sizeof(R) == 4 ? 6 : 5) void k_nbr_group(
    Batch B, Parts s, const uint32_t *__restrict__ cstart, int all, uint32_t *__restrict__ nbr,
    uint32_t *__restrict__ nnb, typename Vec4<R>::T *__restrict__ ap,
    double *__restrict__ dbg_gam, double *__restrict__ dbg_vt, Parts home, Spans sp) {
  static_assert(MODE == 0 || (MODE == 1 && !FORCES) || MODE == 2, "candidate list modes");
  static_assert(G == 4 || G == 8 || (G == 2 && MODE == 2), "two lanes filter Verlet lists only");
  static_assert(!PN || (D == 3 && FORCES), "pair normals: patches in 3D");
  using R4 = typename Vec4<R>::T;
  constexpr int PB = BLOCK / G;        // particles per block
  constexpr int Q = 4;                 // places per lane and pass
  constexpr int WIN = Q * G;           // places per pass
  // list entries kept in LDS per particle: the lists of most waves whole
  constexpr int RL = D == 2 ? (G == 8 ? 64 : 32) : (G == 8 ? 128 : 64);
  static_assert(RL >= 2 * WIN, "room for a pass beside what waits to be stored");
  constexpr bool RUNS = G == 2;        // a lane takes Q consecutive places (else G lanes take G)
  constexpr int NS = 2 + 2 * D;        // sums per particle
  constexpr int NB = 4;                // entries per lane and pass of the sums
  constexpr uint32_t GM = (1u << G) - 1u;
  __shared__ uint32_t ring[PB][RL + G];
  __shared__ uint32_t rowb[MODE == 2 ? 1 : PB][G + 1];
  __shared__ double red[FORCES ? NS : 1][FORCES ? PB : 1];
  __shared__ uint32_t scount[FORCES ? PB : 1];
  const int n = B.n;
  if (MODE == 1) {
    if (B.vstate[VS_REBUILD] == 0ull) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) B.vstate[VS_BUILDS] += 1ull;
  }
  const int col = (int)threadIdx.x / G, gl = (int)threadIdx.x % G;
  // the block's job and its particles [first, end)
  int job, first, end;
  span_of(sp, xcd_block(), PB, job, first, end);
  const int i = first + col;
  // the group's bits of a wave's ballot: word half and shift; lanes below
  const bool upper = (threadIdx.x & 32) != 0;
  const uint32_t gshift = threadIdx.x & 31u & ~(uint32_t)(G - 1);
  const uint32_t lt = (1u << gl) - 1u, le = 2u * lt + 1u;   // lanes below (and this one) in the group
  auto group_bits = [&](bool v) -> uint32_t {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(v);
    return (upper ? (uint32_t)(m >> 32) : (uint32_t)m) >> gshift & GM;
  };
  uint32_t count = 0;
  // loads that need nothing but the slot come first, in flight together
  const int il = i < end ? i : 0;
  const int fi = s.f[il];
  const double4 xi = s.xh[il];
  const uint32_t ns = MODE == 2 ? B.nsk[il] : 0u;
  // MODE 2: the entries of a pass from place b0 (uniform); blocks past the
  // capacity are not there, entries past the list are not used
  const size_t sstep = (size_t)n * LB;
  const uint32_t lastb = MODE == 2 ? (uint32_t)B.skin_cap / LB - 1u : 0u;
  const uint32_t *sk = (MODE == 2 ? B.skin : nullptr) + (size_t)il * LB;
  auto entries = [&](uint32_t b0, uint32_t (&u)[Q]) {
    if constexpr (RUNS) {   // a lane's four entries: half a block
      const uint32_t b = b0 / LB < lastb ? b0 / LB : lastb;
      const uint4 w = *reinterpret_cast<const uint4 *>(sk + (size_t)b * sstep + b0 % LB + Q * gl);
      u[0] = w.x;
      u[1] = w.y;
      u[2] = w.z;
      u[3] = w.w;
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t e = b0 + q * G, b = e / LB < lastb ? e / LB : lastb;
        u[q] = sk[(size_t)b * sstep + e % LB + gl];
      }
    }
  };
  uint32_t nx[Q];
  if constexpr (MODE == 2) entries(0u, nx);
  uint32_t fw;   // the feature's type, k and kind (its record's first bytes)
  __builtin_memcpy(&fw, &B.feat[fi], 4);
  const int ftype = fw & 0xff, fk = (fw >> 8) & 0xff, fkind = (fw >> 16) & 0xff;
  const bool active = B.grp[fi].active != 0;
  const JobDev &J = B.jobs[job];   // uniform: read by scalar loads
  if (i < end) {
    if (MODE == 1) {   // the sorted particle goes back to the buffer the steps use
      if (gl == 0) home.xh[i] = xi;
      if (gl == 1) home.v[i] = s.v[i];
      if (gl == 2) home.xf[i] = s.xf[i];
      if (gl == 3) {
        home.f[i] = (uint16_t)fi;
        home.oid[i] = s.oid[i];
      }
    }
    const bool moving = ftype != T_SI && active;
    const bool want = ftype != T_SI && (all || MODE == 1 || active);
    if (want) {
      const double kc2 = sload(J.ksup2);   // c^2, c = support radius / h
      const double A4 = kc2 * (xi.w * xi.w);
      const float4 xif = scan_record<D>(xi, (uint32_t)fi);
      const float Hif = D == 2 ? xif.z : xif.w;
      float cin = sload(J.band_in), cout = MODE == 1 ? sload(J.band_reach) : sload(J.band_out);
      const double bx = sload(J.band_x);
      if (__builtin_fabs(xi.x) > bx || __builtin_fabs(xi.y) > bx || (D == 3 && __builtin_fabs(xi.z) > bx))
        band_beyond<D, MODE>(J, xi, cin, cout);
      uint32_t *list = (MODE == 1 ? B.skin : nbr) + (size_t)i * LB;
      const uint32_t nblk = (uint32_t)(MODE == 1 ? B.skin_cap : B.cap) / LB;   // blocks of capacity
      uint32_t stored = 0;   // whole blocks stored
      // features that interact with fi: its own ("same") and the bounding
      // ones of its job (bit = local feature id)
      const unsigned long long accept = MODE == 2 ? 0ull : B.bmask[fi] | (1ull << (fi & (MAXF - 1)));
      auto store_blocks = [&](uint32_t upto) {
        lane_sync();
        for (; any_lane(stored < upto); ++stored) {
          if (stored < upto && stored < nblk) {
            uint32_t *w = list + (size_t)stored * sstep;
            const uint32_t k = (stored * LB + LB / G * gl) % RL;
            const uint32_t *rg = &ring[col][k];
            if (G == 8) w[gl] = rg[0];
            if (G == 4) reinterpret_cast<uint2 *>(w)[gl] = make_uint2(rg[0], rg[1]);
            if (G == 2) reinterpret_cast<uint4 *>(w)[gl] = make_uint4(rg[0], rg[1], rg[2], rg[3]);
          }
        }
        if (stored > upto) stored = upto;
      };
      // candidates jr with list entries tg: the hits enter the ring in the
      // order of their places; a pass adds at most WIN, so whole blocks are
      // stored as soon as less than a pass' room is left
      auto classify = [&](const float4 (&xr)[Q], const uint32_t (&jr)[Q], const uint32_t (&tg)[Q],
                          const bool (&cand)[Q]) {
        bool hits[Q];
        uint32_t tags[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          if (!RUNS && q > 0 && !any_lane(cand[q])) break;   // no group of the wave has places left
          const float ex = xif.x - xr[q].x, ey = xif.y - xr[q].y;
          const float ez = D == 3 ? xif.z - xr[q].z : 0.0f;
          const float d2 = ex * ex + ey * ey + ez * ez;
          const float Hj = D == 2 ? xr[q].z : xr[q].w;
          const float H = __builtin_fmaxf(Hif, Hj);
          const float H2 = H * H;
          const float tout = H2 * cout;
          bool c = cand[q];
          tags[q] = tg[q];
          if constexpr (MODE != 2) {   // the scan's candidates: relation of the features
            const uint32_t fr = __float_as_uint(xr[q].w) & (MAXF - 1);
            c = c & (bool)((accept >> fr) & 1ull);
            tags[q] = jr[q] | (fr == (uint32_t)(fi & (MAXF - 1)) ? 0u : 0x80000000u);
          }
          if constexpr (MODE == 1) {   // Verlet list: all that may lie within reach
            hits[q] = c & !(d2 > tout);
          } else {
            const float tin = H2 * cin;
            hits[q] = c & (d2 < tin);
            const bool band = c & !(d2 < tin) & !(d2 > tout);   // near the support radius: exact test
            if (any_lane(band)) {
              if (band) hits[q] = within_a4<D>(xi, A4, kc2, s.xh[jr[q]]);
            }
          }
          if constexpr (!RUNS) {
            const uint32_t bits = group_bits(hits[q]);
            if (hits[q]) ring[col][(count + __popc(bits & lt)) % RL] = tags[q];
            count += __popc(bits);
          }
        }
        if constexpr (RUNS) {
          uint32_t nh = 0;
#pragma unroll
          for (int q = 0; q < Q; ++q) nh += hits[q] ? 1u : 0u;
          const uint32_t other = dpp_u32<DPP_XOR1>(nh);
          uint32_t k = count + (gl ? other : 0u);
#pragma unroll
          for (int q = 0; q < Q; ++q)
            if (hits[q]) ring[col][k++ % RL] = tags[q];
          count += nh + other;
        }
        const bool full = count - stored * LB > (uint32_t)(RL - WIN);
        if (any_lane(full)) store_blocks(full ? count / LB : stored);
      };
      if constexpr (MODE == 2) {
        for (uint32_t b0 = 0; any_lane(b0 < ns); b0 += WIN) {
          uint32_t tg[Q], jr[Q];
          bool cand[Q];
          float4 xr[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            tg[q] = nx[q];
            cand[q] = b0 + (RUNS ? gl * Q + q : q * G + gl) < ns;
            jr[q] = cand[q] ? nx[q] & 0x7fffffffu : (uint32_t)i;
            xr[q] = s.xf[jr[q]];
          }
          entries(b0 + WIN, nx);   // the next pass', in flight behind the records
          classify(xr, jr, tg, cand);
        }
      } else {
        const Grid &Gr = J.G;
        const double ksup = MODE == 1 ? sload(J.ksup_s) : sload(J.ksup);
        double Rs = (MODE == 1 ? sload(J.rfac_s) : sload(Gr.rfac)) * xi.w;
        const double rmax = MODE == 1 ? sload(J.rmax_s) : sload(Gr.rmax);
        Rs = Rs < rmax ? Rs : rmax;
        // cell levels that can hold a neighbour: h is L-Lipschitz, so a
        // neighbour (r < R_i) has |h_j - h_i| <= L R_i (widened for rounding)
        const int nlev = sload(Gr.nlev);
        const double dh = sload(Gr.lip) * Rs * (1.0 + 1e-9);
        const double hlo = (xi.w - dh) * (1.0 - 1e-12), hup = (xi.w + dh) * (1.0 + 1e-12);
        auto coord = [&](double p, double lo, double inv, int top) -> int {   // as cell_coord
          double c = __builtin_floor((p - lo) * inv);
          c = c >= 0.0 ? c : 0.0;   // also maps NaN to cell 0
          const double tp = (double)top;
          return (int)(c > tp ? tp : c);
        };
        for (int lv = 0; lv < nlev; ++lv) {
          if (nlev > 1) {   // the particle's levels: h_level(hlo) .. h_level(hup)
            const bool below = lv + 1 < nlev && hlo >= sload(Gr.hthr[lv + 1]);
            const bool above = lv > 0 && !(hup >= sload(Gr.hthr[lv]));
            if (below || above) continue;
          }
          const double hcap = sload(Gr.hcap[lv]);
          // a level-lv candidate has h_j < hcap[lv], so none beyond
          // c max(h_i, hcap[lv]) is a neighbour
          double Rl = ksup * (xi.w > hcap ? xi.w : hcap) * (1.0 + 1e-9);
          Rl = Rl < Rs ? Rl : Rs;
          const int nc[3] = {sload(Gr.nc[lv][0]), sload(Gr.nc[lv][1]), D == 3 ? sload(Gr.nc[lv][2]) : 1};
          const uint32_t nc0 = (uint32_t)nc[0];
          const uint32_t cbase = sload(Gr.cbase) + sload(Gr.lbase[lv]);
          // x_i in cells of the level: whole part and fraction.  The rows'
          // distances and chords are FP32 and widened past their rounding (a
          // few 1e-6 of a cell or of the reach): a cell too many costs its
          // candidates' tests, the lists are decided by those
          float fr[3] = {0.0f, 0.0f, 0.0f};
          int ic[3] = {0, 0, 0}, rlo[3] = {0, 0, 0}, rhi[3] = {0, 0, 0};
          const double xd[3] = {xi.x, xi.y, xi.z};
#pragma unroll
          for (int a = 0; a < D; ++a) {
            const double lo = sload(Gr.lo[a]), inv = sload(Gr.inv_c[lv][a]);
            cell_split((xd[a] - lo) * inv, ic[a], fr[a]);
            if (a > 0) {
              rlo[a] = coord(xd[a] - Rl, lo, inv, nc[a] - 1);
              rhi[a] = coord(xd[a] + Rl, lo, inv, nc[a] - 1);
            }
          }
          const float R2 = (float)(Rl * Rl) * (1.0f + 4e-6f);
          const float c1 = (float)sload(Gr.c[lv][1]) * (1.0f - 1e-6f);
          const float c2 = D == 3 ? (float)sload(Gr.c[lv][2]) * (1.0f - 1e-6f) : 0.0f;
          const float inv0 = (float)sload(Gr.inv_c[lv][0]) * (1.0f + 2e-6f);
          const bool tiled = rows_tiled(D, nc);
          const uint32_t nyt = ((uint32_t)nc[1] + 7u) >> 3;
          const int ylo = rlo[1], yhi = rhi[1], zlo = rlo[2], zhi = rhi[2];
          const int ny = yhi - ylo + 1;
          const int nrows = ny * (zhi - zlo + 1);
          int cy = ylo + gl, cz = zlo;
          for (int r0 = 0; any_lane(r0 < nrows); r0 += G, cy += G) {
            if (D == 3)
              while (cy > yhi) {
                cy -= ny;
                ++cz;
              }
            uint32_t jb = 0, len = 0;
            if (r0 + gl < nrows) {   // this lane's row
              // distance to the row in cells, from x's own cell
              auto gap = [](int d, float f) {
                const float g = d > 0 ? (float)d - f : f - (float)(d + 1);
                const float h = g * (1.0f - 1e-6f) - 2e-5f;
                return h > 0.0f ? h : 0.0f;
              };
              const float dy = gap(cy - ic[1], fr[1]) * c1;
              const float dz = D == 3 ? gap(cz - ic[2], fr[2]) * c2 : 0.0f;
              const float w2 = R2 - dy * dy - dz * dz;
              if (!(w2 < 0.0f)) {
                int t0, t1;
                row_range(ic[0], fr[0], sqrt_(w2) * inv0 + 2e-5f, nc[0], t0, t1);
                // as cell_row
                const uint32_t ry = (uint32_t)cy, rz = (uint32_t)cz;
                const uint32_t rw = tiled ? (((rz >> 3) * nyt + (ry >> 3)) << 6) + ((rz & 7u) << 3) + (ry & 7u)
                                          : rz * (uint32_t)nc[1] + ry;
                const uint32_t row = cbase + rw * nc0;
                jb = cstart[row + (uint32_t)t0];
                const uint32_t je = cstart[row + (uint32_t)t1 + 1];
                len = je > jb ? je - jb : 0u;
              }
            }
            const uint32_t incl = group_scan<G>(len, gl), excl = incl - len;
            const uint32_t total = (uint32_t)__shfl((int)incl, (int)((threadIdx.x & 63u) | (G - 1)));
            // row r of the non-empty ones holds the places from its start on:
            // its place t is slot rowb[r + 1] + t
            const uint32_t ne = group_bits(len != 0u);
            lane_sync();
            if (len != 0u) rowb[col][__popc(ne & le)] = jb - excl;
            lane_sync();
            uint32_t before = 0;   // rows that start before the pass
            for (uint32_t w0 = 0; any_lane(w0 < total); w0 += WIN) {
              const uint32_t sb = excl - w0;
              const uint32_t mine = len != 0u && sb < (uint32_t)WIN ? 1u << (sb & 31u) : 0u;
              const uint32_t starts = group_or<G>(mine);
              uint32_t jr[Q], tg[Q];
              bool cand[Q];
              float4 xr[Q];
#pragma unroll
              for (int q = 0; q < Q; ++q) {
                const uint32_t f = starts >> (q * G) & GM;
                const uint32_t k = before + __popc(f & le);   // rows started up to this place
                before += __popc(f);
                const uint32_t t = w0 + (uint32_t)(q * G + gl);
                const uint32_t j = rowb[col][k] + t;
                cand[q] = t < total;
                jr[q] = cand[q] ? j : (uint32_t)i;
                cand[q] = jr[q] != (uint32_t)i;
                tg[q] = 0u;
                xr[q] = s.xf[jr[q]];
              }
              classify(xr, jr, tg, cand);
            }
          }
        }
      }
      // the blocks left in the ring, the last one partly filled
      store_blocks((count + LB - 1) / LB);
      if (MODE == 1 && (int)count > B.skin_cap) {
        if (gl == 0) {
          atomicMax(&B.st[job].skin_max, count);
          atomicExch(&B.st[job].skin_overflow, 1u);
        }
        count = B.skin_cap;
      } else if (MODE != 1 && (int)count > B.cap) {
        if (gl == 0) {
          atomicMax(&B.st[job].overflow_max, count);
          atomicExch(&B.st[job].overflow, 1u);
        }
        count = B.cap;
      }
    }
    if (gl == 0) {
      if (MODE == 1) B.nsk[i] = count; else nnb[i] = count;
    }
    if (FORCES) {
      if (gl == 0) scount[col] = count;
      if (moving) {
        lane_sync();   // the group's blocks and ring entries are read by all its lanes
        const BNorm *bnrow = B.bn + (size_t)fi * MAXF;
        // a 3D patch of a level set with imported curves: pair-dependent normals
        const bool pairn = PN && fkind == K_LEVEL && sload(J.g.cpts) != nullptr;
        const int bw = sload(J.bw);
        const double p0 = sload(J.p0), klen = sload(J.klen), bscale = sload(J.bscale);
        double S, gam, Pi[3], B3[3];
        const LdsList lring = (LdsList)&ring[col][0];
        if (fk == D)
          group_sums<D, D, R, CMP, PN, NB, G>(J.g, s, B.enrm, bnrow, bw, p0, klen, bscale, nbr, n, i, count, xi,
                                         pairn, S, gam, Pi, B3, lring, RL, gl);
        else if (fk == D - 1)
          group_sums<D, D - 1, R, CMP, PN, NB, G>(J.g, s, B.enrm, bnrow, bw, p0, klen, bscale, nbr, n, i, count,
                                             xi, pairn, S, gam, Pi, B3, lring, RL, gl);
        else
          group_sums<D, 1, R, CMP, PN, NB, G>(J.g, s, B.enrm, bnrow, bw, p0, klen, bscale, nbr, n, i, count, xi,
                                         pairn, S, gam, Pi, B3, lring, RL, gl);
        S = group_sum<G>(S);
        gam = group_sum<G>(gam);
#pragma unroll
        for (int a = 0; a < D; ++a) Pi[a] = group_sum<G>(Pi[a]);
        // boundary terms come up only beside the boundary
        if (any_lane(B3[0] != 0.0 || B3[1] != 0.0 || (D == 3 && B3[2] != 0.0))) {
#pragma unroll
          for (int a = 0; a < D; ++a) B3[a] = group_sum<G>(B3[a]);
        }
        if (gl == 0) {
          red[0][col] = S;
          red[1][col] = gam;
#pragma unroll
          for (int a = 0; a < D; ++a) {
            red[2 + a][col] = Pi[a];
            red[2 + D + a][col] = B3[a];
          }
        }
      }
    }
  }
  if (!FORCES) return;
  // the particles' own part, one lane each
  const int c = (int)threadIdx.x;
  const int p = first + c;
  const bool have = c < PB && p < end;
  int fp = 0;
  double4 xp = make_double4(0.0, 0.0, 0.0, 0.0), v4 = xp;
  if (have) {
    fp = s.f[p];
    xp = s.xh[p];
    v4 = s.v[p];
  }
  __syncthreads();
  if ((int)threadIdx.x >= (PB < 64 ? 64 : PB)) return;
  bool act = false;
  unsigned long long dtb = ~0ull, vfix = 0ull, mine = 0ull;
  if (have) {
    const Feat Fp = B.feat[fp];
    mine = scount[c];
    act = Fp.type != T_SI && B.grp[fp].active;
    R4 o;
    o.x = o.y = o.z = o.w = R(0);
    double gam = 0.0, vt = 0.0;
    if (act) {
      if (B.grp[fp].reset_now) {
        v4 = make_double4(0.0, 0.0, 0.0, 0.0);
        s.v[p] = v4;
      }
      const double S = red[0][c];
      gam = red[1][c];
      // the FP32 modes store a^p in FP32 and hold V~ and the time steps to
      // 1e-5: FP32 reciprocals and roots suffice there (relative error 2^-23)
      constexpr bool F32 = sizeof(R) == 4;
      double a3[3] = {0.0, 0.0, 0.0};
      const double ig = F32 ? (double)rcp_((float)gam) : 0.0;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const double t = red[2 + a][c] + red[2 + D + a][c];
        a3[a] = F32 ? -(t * ig) : -(t / gam);
      }
      double xa[3] = {xp.x, xp.y, xp.z};
      tangent_at<D>(J.g, Fp, xa, B.enrm, p, a3);
      // in 2D the record's free slots carry v^n (after any reset) in the
      // sweep precision, so sweep B gathers one record per neighbour less
      o.x = (R)a3[0];
      o.y = (R)a3[1];
      o.z = D == 2 ? (R)v4.x : (R)a3[2];
      o.w = D == 2 ? (R)v4.y : R(0);
      vt = F32 ? (double)rcp_((float)S) : 1.0 / S;
      // Eq. (fa_time_step_size) terms from a^p and v^n
      const double rc = J.ksup * xp.w;
      dtb = dbits(step_terms<F32>(rc, sum2<3>(a3[0], a3[1], a3[2]), sum2<3>(v4.x, v4.y, v4.z)));
      vfix = (unsigned long long)__builtin_llrint(vt * B.grp[fp].vscale);
    }
    ap[p] = o;
    if (dbg_gam) dbg_gam[p] = gam;
    if (dbg_vt) dbg_vt[p] = vt;
  }
  wave_commit(act, fp, dtb, vfix, B.smin, DT1, B.ssum, PB > 64 ? PB / 64 : 1);
  wave_count(have && mine != 0ull, job, mine, B.scnt, SC_PAIRS, PB > 64 ? PB / 64 : 1);
}

// ---------------------------------------------------------------------------
// mid-point velocity of every moving particle, once: v~ = v + dt_1/2 a^p
// (Eq. momentum_equation_discretized's v~) and eta = 0.2 h |v~| / h^k
// (Eq. viscosity_coefficient), in the sweep precision, so that sweep B
// gathers one 16-byte (FP32) record per neighbour instead of v and a^p.  Bound
// by memory; the fold of dt_1 (fold_rows) costs it 3 to 5 us where its launch
// took 4: of 2,000,000 particles, FP32, 33.1 us with the loads ahead of the fold,
// 34.9 behind it.
// ---------------------------------------------------------------------------
template <int D, typename R>
__global__ __launch_bounds__(BLOCK) void k_midpoint(Batch B, Parts s,
                                                    const typename Vec4<R>::T *__restrict__ ap,
                                                    typename Vec4<R>::T *__restrict__ mid, Spans sp) {
  using R4 = typename Vec4<R>::T;
  __shared__ FoldParts part;
  int job, first, end;
  span_of(sp, (int)blockIdx.x, BLOCK, job, first, end);
  const int i = first + (int)threadIdx.x;
  const bool have = i < end;
  // the particle's loads are in flight while the copies are folded (slot 0 for a
  // place past the job: blocks are rounded up, so `first` may lie past the end)
  const int il = have ? i : 0;
  const int fi = s.f[il];
  const double4 v = s.v[il];
  const R4 a = ap[il];
  const R h = (R)s.xh[il].w;
  fold_rows(B, DT1, job, part);
  const Feat F = B.feat[fi];
  const bool act = have && F.type != T_SI && B.grp[fi].active;
  __syncthreads();
  if (!have) return;
  const unsigned long long dt1 = step_bits(B, part, fi);
  R4 o;
  o.x = o.y = o.z = o.w = R(0);
  if (act) {
    // sweep B reads it there; every writer stores the same value
    if (B.grp[fi].dt1_bits != dt1) B.grp[fi].dt1_bits = dt1;
    const R halfR = (R)(0.5 * bitsd(dt1));
    o.x = (R)v.x + halfR * a.x;
    o.y = (R)v.y + halfR * a.y;
    o.z = D == 3 ? (R)v.z + halfR * a.z : R(0);
    const R vm = sqrt_(o.x * o.x + o.y * o.y + o.z * o.z);
    const R hk = F.k == 1 ? powK<1>(h) : (F.k == 2 ? powK<2>(h) : powK<3>(h));
    o.w = (R)(0.1 * B.jobs[fi / MAXF].ksup) * h * vm * rcp_(hk);   // eta = rho_t 0.1 r_c |v~|
  }
  mid[i] = o;
}

// ---------------------------------------------------------------------------
// sweep B pair sums: viscous force of Eq. (momentum_equation_discretized)
// with eta = rho_t nu, nu = 0.1 r_c |v~| (Eq. (viscosity_coefficient)), the
// mid-point velocities v~_j = v_j + dt_1/2 a^p_j formed on the fly
// ---------------------------------------------------------------------------
// MID: neighbours' v~ and eta come from their mid-point records (3D);
// otherwise they are formed here from the a^p record, which in 2D also holds
// v (an extra pass for mid-point records costs more than it saves in 2D).
// XF (FP32 sums): a neighbour's position and h come from its 16-byte FP32
// scan record instead of the 32-byte FP64 one, so the pair differences are
// those of FP32-rounded coordinates; in 3D that record's h carries the
// feature id in its 6 low mantissa bits (relative change below 2^-17).  The
// FP64 mode gathers the FP64 record.
// Lane l of the particle's G takes the entries l, l + G, ..., NB of them at a
// time; boundary entries and places past the list take the particle itself,
// with no weight.  The caller adds the lanes' sums.
// A lane alone reads half a block of its list at a time, and in FP32 leaves the
// loop and skips boundary entries by itself, which gathers less (1,000,000
// particles in 2D: 53.5 us, all lanes together 56); the FP64 sums lose by that
// (96.8 against 94).  FOUR: entry e in sum e % 4, as four lanes add them, with the
// multiply-adds written out as in TermsA.
template <int D, int K, typename R, bool MID, bool CMP, int G, bool FOUR>
__device__ __forceinline__ void sweep_b_sums(const Parts &s, const typename Vec4<R>::T *__restrict__ ap,
                                             const typename Vec4<R>::T *__restrict__ mid,
                                             const uint32_t *__restrict__ nbr, int n, int i,
                                             uint32_t cnt, const double4 &xi, const double vti[3],
                                             double vmi, double half, double klen, double Fv[3],
                                             uint32_t lane) {
  using R4 = typename Vec4<R>::T;
  const R hi = (R)xi.w;
  constexpr R alpha = kalphaK<K, R>();
  const R hik = powK<K>(hi), hi2k = hik * hik;
  const R kl = (R)klen;
  const R nuf = (R)(0.2 * klen);   // nu = 0.1 r_c |v~| = 0.2 klen h |v~|
  const R etai = (R)(0.2 * klen * xi.w * vmi) * rcp_(hik);
  const R vtiR[3] = {(R)vti[0], (R)vti[1], (R)vti[2]};
  const R halfR = (R)half;
  constexpr bool XF = sizeof(R) == 4;
  const float3 xfi = make_float3((float)xi.x, (float)xi.y, (float)xi.z);
  static_assert(!FOUR || G == 1, "one lane for four");
  constexpr int V = FOUR ? 4 : 1;   // entry e in sum e % 4, as four lanes add them
  Sum<CMP> aF[V][3];
#pragma unroll
  for (int l = 0; l < V; ++l)
#pragma unroll
    for (int a = 0; a < 3; ++a) aF[l][a].init(0.0);
  constexpr int NB = 4;
  static_assert(LB % NB == 0 && NB % V == 0, "half a block at a time");
  constexpr bool ALONE = G == 1 && sizeof(R) == 4;
  for (uint32_t e0 = 0; ALONE ? e0 < cnt : any_lane(e0 < cnt); e0 += NB * G) {
    uint32_t u[NB];
    if constexpr (G == 1) {
      uint4 w = make_uint4(0u, 0u, 0u, 0u);
      if (e0 < cnt)
        w = reinterpret_cast<const uint4 *>(nbr)[((size_t)(e0 / LB) * n + i) * (LB / 4) + e0 % LB / 4];
      u[0] = w.x;
      u[1] = w.y;
      u[2] = w.z;
      u[3] = w.w;
#pragma unroll
      for (int q = 0; q < NB; ++q) u[q] = e0 + q < cnt ? u[q] : 0x80000000u;
    } else {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const uint32_t e = e0 + q * G + lane;
        u[q] = e < cnt ? nbr[((size_t)(e / LB) * n + i) * LB + e % LB] : 0x80000000u;
      }
    }
    double4 xr[NB];
    float4 fr[NB];
    R4 mr[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const uint32_t j = u[q] >> 31 ? (uint32_t)i : u[q];
      if constexpr (XF) fr[q] = s.xf[j]; else xr[q] = s.xh[j];
      mr[q] = MID ? mid[j] : ap[j];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      // No list of the wave goes on.  The FP64 sums, bound by their arithmetic,
      // look each time; the FP32 ones, bound by the gathers, gain more from
      // entries that overlap (2,000,000 particles in 3D, at 5 waves a SIMD, 290
      // us, looking 333).
      if (sizeof(R) == 8 && q > 0 && !any_lane(e0 + q * G + lane < cnt)) break;
      if (ALONE && u[q] >> 31) continue;
      R dx0, dx1, dx2, hj;
      if constexpr (XF) {
        dx0 = (R)(xfi.x - fr[q].x);
        dx1 = (R)(xfi.y - fr[q].y);
        dx2 = D == 3 ? (R)(xfi.z - fr[q].z) : R(0);
        hj = (R)(0.5f * (D == 3 ? fr[q].w : fr[q].z));
      } else {
        const double4 xj = xr[q];
        dx0 = (R)(xi.x - xj.x);
        dx1 = (R)(xi.y - xj.y);
        dx2 = D == 3 ? (R)(xi.z - xj.z) : R(0);
        hj = (R)xj.w;
      }
      const R rr = sqrt_(sum2<D>(dx0, dx1, dx2));
      const R hjk = powK<K>(hj);
      R vtj[3], etaj;
      if (MID) {
        vtj[0] = mr[q].x;
        vtj[1] = mr[q].y;
        vtj[2] = D == 3 ? mr[q].z : R(0);
        etaj = mr[q].w;
      } else {   // 2D: {a^p_x, a^p_y, v_x, v_y} in the sweep precision
        static_assert(MID || D == 2, "the a^p record carries v only in 2D");
        const R4 apj = mr[q];
        vtj[0] = fma_(halfR, apj.x, apj.z);
        vtj[1] = fma_(halfR, apj.y, apj.w);
        vtj[2] = R(0);
        const R vmj = sqrt_(sum2<2>(vtj[0], vtj[1], R(0)));
        etaj = nuf * hj * vmj * rcp_(hjk);
      }
      const R es = etai + etaj;
      const R H = es > R(0) && !(u[q] >> 31) ? R(2) * etai * etaj * rcp_(es) : R(0);
      const R ihij = rcp_(kl * (R(0.5) * (hi + hj)));
      const R ih2 = ihij * ihij;
      const R ihk2 = K == 1 ? ih2 * ihij : (K == 2 ? ih2 * ih2 : ih2 * ih2 * ihij);
      const R c = H * fma_(hjk, hjk, hi2k) * alpha * dwqK<K>(rr * ihij) * ihk2;
#pragma unroll
      for (int a = 0; a < D; ++a) aF[q % V][a].add_term(c, vtiR[a] - vtj[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
    Fv[a] = V == 1 ? aF[0][a].get()
                   : (aF[0][a].get() + aF[1 % V][a].get()) + (aF[2 % V][a].get() + aF[3 % V][a].get());
}

// ---------------------------------------------------------------------------
// sweep B: mid-point velocity, viscous force, damping.  G lanes per particle,
// a block on particles of one job, as in k_nbr_group; neighbouring lanes gather
// neighbouring entries, which share cache lines.  Bound by the two gathers per
// neighbour in FP32, by the arithmetic in FP64 and, for a few thousand
// particles, by the chain of loads.  us before (one lane in 2D, two in 3D) and
// now: 4,352 particles in 2D, FP64, 13.6 / 7.8; 2,503, FP32, 11.3 / 7.7; 3D
// 30,000, FP64, 20.6 / 16; 66,000, FP32, calibrated, 25 / 20; 300,000 between
// ellipsoids 65 / 52; 2,000,000 295 / 268.  Large 2D batches take one lane
// (small_job).  The gathers want waves: of 2,000,000 particles in 3D 296 us with
// 86 registers (5 waves a SIMD), 268 with 80 (6), 420 with 72, which spill.
// ---------------------------------------------------------------------------
template <int D, typename R, bool CMP, int G, int SUMS>
__global__ __launch_bounds__(BLOCK, sizeof(R) == 4 ? (SUMS == AS_ONE ? 6 : 5) : 4) void k_sweep_b(Batch B, Parts s,
                                                   const uint32_t *__restrict__ nbr,
                                                   const uint32_t *__restrict__ nnb,
                                                   const typename Vec4<R>::T *__restrict__ ap,
                                                   const typename Vec4<R>::T *__restrict__ mid,
                                                   typename Vec4<R>::T *__restrict__ acc,
                                                   double4 *__restrict__ dbg_vm, Spans sp) {
  using R4 = typename Vec4<R>::T;
  constexpr int PB = BLOCK / G;
  __shared__ double red[D][PB], halves[PB];
  __shared__ FoldParts part;
  // the Verlet lists of this step are built: the next rebuild is asked for by
  // k_integrate_hash
  if (B.skin_on && blockIdx.x == 0 && threadIdx.x == 0) B.vstate[VS_REBUILD] = 0ull;
  const int col = (int)threadIdx.x / G, gl = (int)threadIdx.x % G;
  int job, first, end;
  span_of(sp, xcd_block(), PB, job, first, end);
  const JobDev &J = B.jobs[job];
  // v~ = v + dt_1/2 a^p of particle p
  auto midpoint = [&](int p, double half, const double4 &v4, double api[3], double vt[3]) {
    const R4 a4 = ap[p];
    api[0] = (double)a4.x;
    api[1] = (double)a4.y;
    api[2] = D == 3 ? (double)a4.z : 0.0;
    vt[0] = fma_(half, api[0], v4.x);
    vt[1] = fma_(half, api[1], v4.y);
    vt[2] = fma_(half, api[2], v4.z);
  };
  const int i = first + col;
  const int fi = i < end ? (int)s.f[i] : job * MAXF;
  const bool moving = i < end && B.feat[fi].type != T_SI && B.grp[fi].active;
  if (D == 2) {   // 3D: k_midpoint has folded the copies
    fold_rows(B, DT1, job, part);
    __syncthreads();
  }
  {
    if (moving) {
      const int k = B.feat[fi].k;
      const double4 xi = s.xh[i];
      const double half = 0.5 * bitsd(D == 3 ? B.grp[fi].dt1_bits : step_bits(B, part, fi));
      double api[3], vti[3];
      midpoint(i, half, s.v[i], api, vti);
      if (gl == 0) halves[col] = half;
      const double vmi = __builtin_sqrt(sum2<3>(vti[0], vti[1], vti[2]));
      const uint32_t cnt = nnb[i];
      const double klen = sload(J.klen);
      double fv[3];
      bool four = false;
      if constexpr (SUMS != AS_ONE) {
        static_assert(D == 2 && G == 1, "one lane for four");
        four = SUMS == AS_FOUR || J.four;
        if (four && k == D)
          sweep_b_sums<D, D, R, false, CMP, 1, true>(s, ap, mid, nbr, B.n, i, cnt, xi, vti, vmi, half, klen, fv, gl);
        else if (four)
          sweep_b_sums<D, 1, R, false, CMP, 1, true>(s, ap, mid, nbr, B.n, i, cnt, xi, vti, vmi, half, klen, fv, gl);
      }
      if (!four) {
        if (k == D)
          sweep_b_sums<D, D, R, D == 3, CMP, G, false>(s, ap, mid, nbr, B.n, i, cnt, xi, vti, vmi, half, klen, fv, gl);
        else if (k == D - 1)
          sweep_b_sums<D, D - 1, R, D == 3, CMP, G, false>(s, ap, mid, nbr, B.n, i, cnt, xi, vti, vmi, half, klen, fv, gl);
        else
          sweep_b_sums<D, 1, R, D == 3, CMP, G, false>(s, ap, mid, nbr, B.n, i, cnt, xi, vti, vmi, half, klen, fv, gl);
      }
#pragma unroll
      for (int a = 0; a < D; ++a) {
        if constexpr (G > 1) fv[a] = group_sum<G>(fv[a]);
        if (gl == 0) red[a][col] = fv[a];
      }
    }
  }
  // the particles' own part, one lane each
  const int c = (int)threadIdx.x;
  const int p = first + c;
  const bool have = c < PB && p < end;
  int fp = 0;
  double4 xp = make_double4(0.0, 0.0, 0.0, 0.0), vp = xp;
  if (have) {
    fp = s.f[p];
    xp = s.xh[p];
    vp = s.v[p];
  }
  if (G > 1) __syncthreads();   // a lane alone reads what it wrote
  if ((int)threadIdx.x >= (PB < 64 ? 64 : PB)) return;
  bool act = false;
  unsigned long long dtb = ~0ull;
  if (have) {
    const Feat F = B.feat[fp];
    act = F.type != T_SI && B.grp[fp].active;
    R4 o;
    o.x = o.y = o.z = o.w = R(0);
    double vt[3] = {0.0, 0.0, 0.0};
    if (act) {
      double api[3], fv[3] = {0.0, 0.0, 0.0};
      midpoint(p, halves[c], vp, api, vt);
#pragma unroll
      for (int a = 0; a < D; ++a) fv[a] = red[a][c];
      double xa[3] = {xp.x, xp.y, xp.z};
      tangent_at<D>(J.g, F, xa, B.enrm, p, fv);
      const double eps = B.grp[fp].eps;
      const double vi[3] = {vp.x, vp.y, vp.z};
      double a3[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) a3[a] = fma_(-eps, vi[a], api[a] + fv[a]);
      o.x = (R)a3[0];
      o.y = (R)a3[1];
      o.z = (R)a3[2];
      const double rc = J.ksup * xp.w;
      const double dt = step_terms<sizeof(R) == 4>(rc, sum2<3>(a3[0], a3[1], a3[2]), sum2<3>(vt[0], vt[1], vt[2]));
      dtb = dbits(dt);
    }
    acc[p] = o;
    if (dbg_vm) dbg_vm[p] = make_double4(vt[0], vt[1], vt[2], 0.0);
  }
  wave_commit(act, fp, dtb, 0ull, B.smin, DT, nullptr, PB > 64 ? PB / 64 : 1);
}

// ---------------------------------------------------------------------------
// integration with feature projection (FP64 in every precision mode), then
// h, cell and rank of every particle for the next step's sort.  Bound by memory
// (214 bytes a particle with Verlet lists: 2,000,000 in 103 us, 4.1 TB/s), between
// ellipsoids by the distance solves for h.  Bound to 80 registers, 6 waves a SIMD
// (3D, 12 bytes spilled): 2,000,000 particles 103 us, with 87 registers (5 waves)
// 109, unbound with 105 (4) 114; 300,000 between ellipsoids 78, 78 and 88.
// ---------------------------------------------------------------------------
template <int D, typename R>
__global__ __launch_bounds__(BLOCK, 6) void k_integrate_hash(
    Batch B, Parts s, const typename Vec4<R>::T *__restrict__ acc,
    uint32_t *__restrict__ cell, uint32_t *__restrict__ rank, uint32_t *__restrict__ cnt, Spans sp) {
  __shared__ FoldParts part;
  int job, first, end;
  span_of(sp, (int)blockIdx.x, BLOCK, job, first, end);
  const JobDev &J = B.jobs[job];
  const int i = first + (int)threadIdx.x;
  const bool have = i < end;
  bool escaped = false;
  uint32_t cc = 0;
  double moved = 0.0;
  int fi = job * MAXF;
  double4 xh = make_double4(0.0, 0.0, 0.0, 0.0), v4 = xh;
  typename Vec4<R>::T a4;
  a4.x = a4.y = a4.z = a4.w = R(0);
  if (have) {
    fi = s.f[i];
    xh = s.xh[i];
    v4 = s.v[i];
    a4 = acc[i];
  }
  fold_rows(B, DT, job, part);
  __syncthreads();
  if (have) {
    const Feat F = B.feat[fi];
    if (F.type != T_SI && B.grp[fi].active) {
      const double dt = bitsd(step_bits(B, part, fi));
      const double a3[3] = {(double)a4.x, (double)a4.y, (double)a4.z};
      const double x[3] = {xh.x, xh.y, xh.z};
      const double v[3] = {v4.x, v4.y, v4.z};
      double vh[3] = {0.0, 0.0, 0.0}, xs[3] = {0.0, 0.0, 0.0};
      bool finite = true;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        vh[a] = v[a] + 0.5 * dt * a3[a];
        xs[a] = x[a] + dt * vh[a];
        finite = finite && __builtin_isfinite(xs[a]);
      }
      if (!finite) {
        if (atomicExch(&B.st[job].nan_flag, 1u) == 0u) B.st[job].nan_oid = s.oid[i];
      } else if (F.kind == K_VOL && !inside<D>(J.g, xs)) {
        escaped = true;                                   // rejected move: stay, stop
        v4 = make_double4(0.0, 0.0, 0.0, 0.0);
      } else {
        if (F.kind != K_VOL) project<D>(J.g, F, xs);
        // the velocity carried into the next step is v^{n+1/2}, tangent to
        // the feature at x^{n+1}: Algorithm 1 updates the predicted velocity
        // and the position, and no velocity after them
        double vn[3] = {vh[0], vh[1], vh[2]};
        if (F.kind != K_VOL) tangent<D>(J.g, F, xs, vn);
        xh.x = xs[0];
        xh.y = xs[1];
        if (D == 3) xh.z = xs[2];
        v4 = make_double4(vn[0], vn[1], D == 3 ? vn[2] : 0.0, 0.0);
      }
    }
    hash_one<D>(J.g, J.G, xh, cc);
    const float4 rec = scan_record<D>(xh, (uint32_t)fi);
    s.xh[i] = xh;
    s.v[i] = v4;
    s.xf[i] = rec;
    cell[i] = cc;
    if (B.skin_on) {   // displacement since the Verlet list's build, in units of its limit
      const double4 r = B.xref[i];
      const double d0 = xh.x - r.x, d1 = xh.y - r.y, d2 = D == 3 ? xh.z - r.z : 0.0;
      const double d = __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      moved = d > 0.0 ? d / (J.move_eps * r.w) : 0.0;
    }
  }
  const uint32_t r = rank_in_cell(cc, have, cnt);
  if (have) rank[i] = r;
  wave_count(escaped, job, 1ull, B.scnt, SC_ESCAPED);
  // a wave with a particle past its limit (or non-finite) asks for a rebuild of
  // the lists before the next step; every writer stores the same value
  if (B.skin_on && __ballot(!(moved <= 1.0)) && __lane_id() == 0) B.vstate[VS_REBUILD] = 1ull;
}

// ---------------------------------------------------------------------------
// the control law alone over a synthetic series (test entry point); state is
// the control state of the one feature replayed, set to a fresh feature's
// (Phase One, no window yet) before the series
__global__ void k_control_replay(Ctl P, int n, const double *__restrict__ vbar,
                                 const double *__restrict__ dt, int32_t *__restrict__ phase,
                                 int32_t *__restrict__ reset, double *__restrict__ esys,
                                 Group *state) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  Group &G = *state;
  {
    Group g0;
    unsigned char *z = reinterpret_cast<unsigned char *>(&g0);
    for (size_t b = 0; b < sizeof g0; ++b) z[b] = 0;
    g0.phase = PH_ONE;
    g0.esys = __builtin_inf();
    g0.tracked = 1;
    G = g0;
  }
  for (int k = 0; k < n; ++k) {
    if (G.phase != PH_FROZEN) control_law(P, G, vbar[k], dt[k]);
    phase[k] = G.phase;
    reset[k] = G.reset_next;
    esys[k] = G.esys;
  }
}

// ---------------------------------------------------------------------------
// read-back: what the host asks for, laid out as it wants it
// ---------------------------------------------------------------------------
// a job's error flags and per-feature control state, written to host memory
struct Report {
  JobStat st;
  uint32_t gflags, pad;
  struct {
    double esys;
    int32_t phase, tracked;
  } f[MAXF];
};
__global__ __launch_bounds__(MAXF) void k_report(Batch B, int job, Report *__restrict__ out) {
  const int f = (int)threadIdx.x;
  const Group &g = B.grp[job * MAXF + f];
  out->f[f].esys = g.esys;
  out->f[f].phase = g.phase;
  out->f[f].tracked = g.tracked;
  if (f == 0) {
    out->st = B.st[job];
    out->gflags = B.gflags[0];
  }
}

// Vectors (and features) of the particles [first, first + n) in the caller's
// order, 24 (and 4) bytes each, behind the job's error flags: one contiguous
// piece for the copy to the host, which reads 24 bytes a particle instead of 36
// and has nothing left to sort.  The rows go out in 24-byte pieces scattered
// over L2: 0.52 ms for 20,000,000 particles beside 9 ms of copying.
struct OutHead {
  JobStat st;
  uint32_t gflags;
};
constexpr size_t OUT_HEAD = 128;   // bytes; the rows start behind it
static_assert(sizeof(OutHead) <= OUT_HEAD, "room for the flags");
// The row of the particle with caller id o among n.  After a lost scan tile the
// ids may be anything: the caller of the read-back learns of it from the flags
// that come with the rows, so a row out of range is left out.
template <int D>
__host__ __device__ __forceinline__ void put_row(char *p, int n, uint32_t o, const double4 &x, int f, int rows,
                                                 int features) {
  if (o >= (uint32_t)n) return;
  if (rows) {
    double *r = reinterpret_cast<double *>(p) + 3 * (size_t)o;
    r[0] = x.x;
    r[1] = x.y;
    r[2] = D == 3 ? x.z : 0.0;
    p += 24 * (size_t)n;
  }
  if (features) reinterpret_cast<int32_t *>(p)[o] = f % MAXF;
}
template <int D>
__global__ __launch_bounds__(BLOCK) void k_unsort(Batch B, int job, Parts s, const double4 *__restrict__ v,
                                                  int first, int n, char *__restrict__ out, int rows,
                                                  int features) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    OutHead *h = reinterpret_cast<OutHead *>(out);
    h->st = B.st[job];
    h->gflags = B.gflags[0];
  }
  const int k = (int)(blockIdx.x * BLOCK + threadIdx.x);
  if (k >= n) return;
  const double4 x = rows ? v[first + k] : make_double4(0.0, 0.0, 0.0, 0.0);
  put_row<D>(out + OUT_HEAD, n, s.oid[first + k], x, features ? (int)s.f[first + k] : 0, rows, features);
}

}  // namespace sph
