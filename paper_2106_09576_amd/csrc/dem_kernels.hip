// HIP kernels (gfx950, wave64) of the soft-sphere DEM hot path.
//
// Method: Golshan et al., "Lethe-DEM" (arXiv 2106.09576).
//   contact search   Sec. 3.2: particles sorted into cells, broad search over
//                    a cell and its neighbour cells, fine search keeping pairs
//                    closer than the threshold; rerun every K steps (Sec. 3.1)
//   contact law      Sec. 2.1: Eqs. (deltan), (vecn), (delta_t), (vrt),
//                    (normal_force), (tangential_force), (nonlinearkn)-
//                    (nonlinearetat), effective-parameter table, (torque_t),
//                    constant rolling model, (coulomb_overlap)-(coulomb_overlap3)
//   walls            Sec. 2.1 last paragraph: same law against a wall
//   integration      Sec. 2.2: Eqs. (integ_EE), (halfstep), (newvv)
//
// Design (MI355X): a thread per particle, or several where a launch of one each
// leaves the chip idle (the force kernel of small contexts, the mesh kernels).
// The force kernel is a gather over each particle's full neighbour row, so every
// particle sums its own forces in a fixed order (deterministic, no atomics).  Both directions of
// a pair keep their own copy of the tangential overlap; the contact law is
// written so that evaluating it from j's side gives exactly -F and -delta_t
// (IEEE negation symmetry; this file is compiled without FP contraction), so
// the two copies never drift apart.  Rows are stored column-major inside each
// wavefront's slab, so every load of a neighbour index or history component is
// one coalesced 64-lane access.  The force kernel also integrates its own
// particle (ping-pong state buffers), so a time step is one launch, and for a
// context that one workgroup holds all steps between two searches are.
#include "dem_device.hpp"

#include <algorithm>

namespace demgpu {

// ------------------------------------------------------------------ helpers

// Blocks of a 1-D launch are spread over the 8 XCDs round-robin; remap so each
// XCD works on a contiguous range of particles (neighbours then share its L2).
__device__ inline int xcd_block() {
  const unsigned nb = gridDim.x;
  const unsigned b = blockIdx.x;
  if ((nb & 7u) != 0u) return (int)b;
  return (int)((b & 7u) * (nb >> 3) + (b >> 3));
}

static inline unsigned grid_for(int64_t n, int block = kBlock) {
  int64_t b = (n + block - 1) / block;
  if (b < 1) b = 1;
  b = (b + 7) & ~int64_t(7);
  return (unsigned)b;
}

__device__ inline bool finite3(double a, double b, double c) {
  return isfinite(a) && isfinite(b) && isfinite(c);
}

__device__ inline int cell_coord(double x, double lo, double h, int nc) {
  int c = (int)floor((x - lo) / h);
  return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__device__ inline uint32_t cell_key(const GridDev& g, int cx, int cy, int cz) {
  return g.ckey[(cz * g.nc[1] + cy) * g.nc[0] + cx];  // fewer than 2^30 cells
}

// Slot of the displacement-bound ring (StepParams) for absolute step s + d
// (s >= 0; 2^32 = 1 mod 3, so s mod 3 follows from its two 32-bit halves).
__device__ __forceinline__ int bound_slot(int64_t s, int d) {
  const uint64_t u = (uint64_t)s;
  const uint32_t r = ((uint32_t)(u >> 32) % 3u + (uint32_t)u % 3u) % 3u;
  return (int)((r + 3u + (uint32_t)d) % 3u);
}

// ------------------------------------------------------------------ fill

__global__ void k_fill_i32(int* p, int v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

hipError_t launch_fill_i32(int* p, int v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t b = (n + kBlock - 1) / kBlock;
  unsigned nb = (unsigned)(b > 65536 ? 65536 : b);
  hipLaunchKernelGGL(k_fill_i32, dim3(nb), dim3(kBlock), 0, s, p, v, n);
  return hipGetLastError();
}

// ------------------------------------------------------------- sort: keys

// Cell key of particle i; deactivates it outside the domain box, checks the
// displacement guard and the state.
__device__ __forceinline__ uint32_t particle_key(const InstDev* __restrict__ inst,
                                                 const StepParams& sp, int i,
                                                 const double4* __restrict__ pos,
                                                 const double4* __restrict__ vel,
                                                 int* __restrict__ info,
                                                 const double4* __restrict__ xref,
                                                 int check_guard, int* __restrict__ flags) {
  const int inf = info[i];
  if (inf & kInactive) return sp.n_keys;
  const InstDev& I = inst[inf >> kInstShift];
  const GridDev& g = I.grid;
  const double4 p = pos[i];
  const double4 v = vel[i];
  if (!finite3(p.x, p.y, p.z) || !finite3(v.x, v.y, v.z)) atomicOr(flags, kFlagNonFinite);
  if (check_guard) {
    const double4 r = xref[i];
    const double dx = p.x - r.x, dy = p.y - r.y, dz = p.z - r.z;
    const double d2 = (dx * dx + dy * dy) + dz * dz;
    if (d2 > I.guard2) atomicOr(flags, kFlagGuard);
  }
  const bool inside = p.x >= g.lo[0] && p.x < g.hi[0] && p.y >= g.lo[1] && p.y < g.hi[1] &&
                      p.z >= g.lo[2] && p.z < g.hi[2];
  if (!inside) {
    info[i] = inf | kInactive;
    return sp.n_keys;
  }
  const int cx = cell_coord(p.x, g.lo[0], g.h, g.nc[0]);
  const int cy = cell_coord(p.y, g.lo[1], g.h, g.nc[1]);
  const int cz = cell_coord(p.z, g.lo[2], g.h, g.nc[2]);
  return I.key_base + cell_key(g, cx, cy, cz);
}

// Cell key of every particle, counted per cell (the returned atomic slot is
// the particle's provisional rank in its cell).
__global__ void k_keys(const InstDev* __restrict__ inst, StepParams sp,
                       const double4* __restrict__ pos,
                       const double4* __restrict__ vel, int* __restrict__ info,
                       const double4* __restrict__ xref, int check_guard,
                       uint32_t* __restrict__ keys, int* __restrict__ rank,
                       int* __restrict__ count, int* __restrict__ flags) {
  int i = xcd_block() * kBlock + threadIdx.x;
  // every lane stays to the end: the ranks are handed out per run of equal
  // keys in the wavefront (below)
  const bool valid = i < sp.n;
  const uint32_t key = valid ? particle_key(inst, sp, i, pos, vel, info, xref, check_guard, flags)
                             : 0xffffffffu;
  // Particles come in the previous search's spatial order, so lanes with the
  // same cell mostly sit side by side: the first lane of each run of equal
  // keys reserves the whole run with one atomic and hands consecutive ranks
  // to the run (the order within a cell is fixed later by k_cell_rank).
  const int lane = threadIdx.x & 63;
  const uint32_t prev = __shfl_up(key, 1, 64);
  const bool first = lane == 0 || prev != key;
  const unsigned long long starts = __builtin_amdgcn_ballot_w64(first);
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  const int lead = 63 - __builtin_clzll(starts & upto);
  const unsigned long long after = lane == 63 ? 0ull : (starts & ~upto);
  const int next = after ? __builtin_ctzll(after) : 64;
  int base = 0;
  if (first && valid) base = atomicAdd(&count[key], next - lane);
  base = __shfl(base, lead, 64);
  if (valid) {
    keys[i] = key;
    rank[i] = base + (lane - lead);
  }
}

hipError_t launch_keys(const InstDev* inst, const StepParams& sp, const double4* pos,
                       const double4* vel, int* info, const double4* xref, int check_guard,
                       uint32_t* keys, int* rank, int* count, int* flags, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_keys, dim3(grid_for(sp.n)), dim3(kBlock), 0, s, inst, sp, pos, vel, info,
                     xref, check_guard, keys, rank, count, flags);
  return hipGetLastError();
}

// ------------------------------------------------------------- sort: scan
// Three-phase exclusive scan: tile sums, one-block scan of the tile sums,
// tile-local scan plus offset.  Tiles of 1024 elements (256 threads x 4).

constexpr int kScanTile = 1024;

__device__ inline int block_exclusive_scan(int v, int* sh, int* total) {
  // 256 threads, 4 waves: wave-level inclusive scan via shuffles, then waves.
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[w] = x;
  __syncthreads();
  int wsum = 0;
  for (int k = 0; k < w; ++k) wsum += sh[k];
  int tot = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  *total = tot;
  return x - v + wsum;
}

__global__ void k_scan_tiles(const int* __restrict__ in, int64_t m, int* __restrict__ tsum) {
  __shared__ int sh[4];
  int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
  int s = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (base + k < m) s += in[base + k];
  int tot;
  block_exclusive_scan(s, sh, &tot);
  if (threadIdx.x == 0) tsum[blockIdx.x] = tot;
}

// One workgroup: thread t takes the contiguous chunk [t c, (t + 1) c) of the
// nt tile sums (c = ceil(nt / kBlock)), adds it up (independent loads, not
// one dependent round per kBlock sums), the chunk totals are scanned across
// the workgroup, and each thread writes its chunk's exclusive prefixes.
__global__ void k_scan_sums(int* __restrict__ tsum, int64_t nt) {
  __shared__ int sh[4];
  const int64_t c = (nt + kBlock - 1) / kBlock;
  const int64_t a = (int64_t)threadIdx.x * c;
  const int64_t b = a + c < nt ? a + c : nt;
  int s = 0;
#pragma unroll 8
  for (int64_t i = a; i < b; ++i) s += tsum[i];
  int tot;
  int ex = block_exclusive_scan(s, sh, &tot);
  for (int64_t i = a; i < b; ++i) {
    const int v = tsum[i];
    tsum[i] = ex;
    ex += v;
  }
}

// With cse: also the (start, end) pair of each of the first n_cells keys,
// stored at that key's cell (key_cell), for lookups by cell position.
__global__ void k_scan_apply(const int* __restrict__ in, int64_t m, const int* __restrict__ tsum,
                             int* __restrict__ out, const uint32_t* __restrict__ key_cell,
                             int2* __restrict__ cse, int64_t n_cells) {
  __shared__ int sh[4];
  int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
  int v[4];
  int s = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = (base + k < m) ? in[base + k] : 0;
    s += v[k];
  }
  int tot;
  int ex = block_exclusive_scan(s, sh, &tot) + tsum[blockIdx.x];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (base + k < m) out[base + k] = ex;
    if (cse && base + k < n_cells) cse[key_cell[base + k]] = make_int2(ex, ex + v[k]);
    ex += v[k];
  }
  // the element after the last one holds the total
  if (base <= m - 1 && m - 1 < base + 4) out[m] = ex;
}

hipError_t launch_scan(const int* count, int* start, int64_t m, int* tile_sums, hipStream_t s,
                       const uint32_t* key_cell, int2* cse, int64_t n_cells) {
  if (m <= 0) return hipSuccess;
  int64_t nt = (m + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nt), dim3(kBlock), 0, s, count, m, tile_sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kBlock), 0, s, tile_sums, nt);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nt), dim3(kBlock), 0, s, count, m, tile_sums,
                     start, key_cell, cse, n_cells);
  return hipGetLastError();
}

// ---------------------------------------------------------- sort: scatter

__global__ void k_scatter(int n, const uint32_t* __restrict__ keys, const int* __restrict__ rank,
                          const int* __restrict__ start, int* __restrict__ perm0) {
  int i = xcd_block() * kBlock + threadIdx.x;
  if (i >= n) return;
  perm0[start[keys[i]] + rank[i]] = i;
}

hipError_t launch_scatter(int n, const uint32_t* keys, const int* rank, const int* start,
                          int* perm0, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3(grid_for(n)), dim3(kBlock), 0, s, n, keys, rank, start,
                     perm0);
  return hipGetLastError();
}

// Within a cell, order particles by gid so the sorted order (and with it every
// summation order) is independent of atomic arrival order.  Inactive particles
// (last key) keep their arrival order: they take part in no computation.
__global__ void k_cell_rank(int n, uint32_t n_keys, const int* __restrict__ perm0,
                            const uint32_t* __restrict__ keys, const int* __restrict__ start,
                            const int* __restrict__ gid, int* __restrict__ perm) {
  int p = xcd_block() * kBlock + threadIdx.x;
  if (p >= n) return;
  int o = perm0[p];
  uint32_t k = keys[o];
  if (k == n_keys) {
    perm[p] = o;
    return;
  }
  int s = start[k], e = start[k + 1];
  int g = gid[o];
  int r = 0;
  for (int q = s; q < e; ++q) r += gid[perm0[q]] < g ? 1 : 0;
  perm[s + r] = o;
}

hipError_t launch_cell_rank(int n, int64_t n_keys, const int* perm0, const uint32_t* keys,
                            const int* start, const int* gid, int* perm, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cell_rank, dim3(grid_for(n)), dim3(kBlock), 0, s, n, (uint32_t)n_keys,
                     perm0, keys, start, gid, perm);
  return hipGetLastError();
}

// ------------------------------------------------------- sort: small contexts
//
// Keys, counts, their scan, the cells' ranges and the order of the particles by
// one workgroup, the counts in LDS.  The seven launches it stands for take 20
// us and the gaps between them for 1,000 particles, all of it latency
// (search chain 64 -> 52 us).

constexpr int kSortThreads = 1024;
constexpr int kSortPer = 4;  // particles per thread
constexpr size_t kSortLds = 64 * 1024 - 256;

// counts (and a total), three words per particle; a scan goes through an odd
// number of counts per thread, so that the chunks lie on different banks
static int sort_chunk(int64_t n_keys) {
  return (int)((n_keys + 1 + kSortThreads - 1) / kSortThreads) | 1;
}
static size_t sort_lds(int n, int64_t n_keys) {
  return sizeof(int) * ((size_t)n_keys + 2 + 3 * (size_t)n);
}
bool small_sort_fits(int n, int64_t n_keys) {
  return n <= kSortThreads * kSortPer && n_keys < 16384 && sort_lds(n, n_keys) <= kSortLds;
}

__global__ void __launch_bounds__(kSortThreads)
k_sort_small(const InstDev* __restrict__ inst, StepParams sp, int chunk,
             const double4* __restrict__ pos, const double4* __restrict__ vel,
             int* __restrict__ info, const double4* __restrict__ xref, int check_guard,
             const int* __restrict__ gid, const uint32_t* __restrict__ key_cell,
             int2* __restrict__ cse, int* __restrict__ start, int* __restrict__ perm,
             int* __restrict__ flags) {
  extern __shared__ int sort_lds_words[];
  __shared__ int sums[kSortThreads / 64];
  int* at = sort_lds_words;  // counts, then first places; at[m] for the end of key m - 1
  const int m = (int)sp.n_keys + 1;
  int* slot_of = at + m + 1;    // particle at each place of its cell, as it arrived
  int* slot_gid = slot_of + sp.n;
  int* slot_key = slot_gid + sp.n;
  const int tid = threadIdx.x;
  for (int k = tid; k <= m; k += kSortThreads) at[k] = 0;
  __syncthreads();
  int key[kSortPer], rank[kSortPer], g[kSortPer];
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const int i = tid + u * kSortThreads;
    if (i >= sp.n) continue;
    g[u] = gid[i];
    key[u] = (int)particle_key(inst, sp, i, pos, vel, info, xref, check_guard, flags);
    rank[u] = atomicAdd(&at[key[u]], 1);
  }
  __syncthreads();
  // exclusive scan: a chunk per thread, the chunks' sums over the wavefronts
  int sum = 0;
  const int k0 = tid * chunk, k1 = k0 + chunk < m ? k0 + chunk : m;
  for (int k = k0; k < k1; ++k) sum += at[k];
  int x = sum;
  const int lane = tid & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sums[tid >> 6] = x;
  __syncthreads();
  int ex = x - sum;
  for (int w = 0; w < (tid >> 6); ++w) ex += sums[w];
  for (int k = k0; k < k1; ++k) {
    const int v = at[k];
    at[k] = ex;
    ex += v;
  }
  if (tid == kSortThreads - 1) at[m] = ex;
  __syncthreads();
  const int n_keys = (int)sp.n_keys;
  for (int k = tid; k <= m; k += kSortThreads) {
    start[k] = at[k];
    if (k < n_keys) cse[key_cell[k]] = make_int2(at[k], at[k + 1]);
  }
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const int i = tid + u * kSortThreads;
    if (i >= sp.n) continue;
    const int s = at[key[u]] + rank[u];
    slot_of[s] = i;
    slot_gid[s] = g[u];
    slot_key[s] = key[u];
  }
  __syncthreads();
  // within a cell by gid; inactive particles as they arrived (k_cell_rank)
  for (int s = tid; s < sp.n; s += kSortThreads) {
    const int c = slot_key[s];
    int to = s;
    if (c != n_keys) {
      const int own = slot_gid[s];
      to = at[c];
      for (int q = at[c]; q < at[c + 1]; ++q) to += slot_gid[q] < own ? 1 : 0;
    }
    perm[to] = slot_of[s];
  }
}

hipError_t launch_sort_small(const InstDev* inst, const StepParams& sp, const double4* pos,
                             const double4* vel, int* info, const double4* xref, int check_guard,
                             const int* gid, const uint32_t* key_cell, int2* cse, int* start,
                             int* perm, int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(kSortThreads), sort_lds(sp.n, sp.n_keys), s, inst,
                     sp, sort_chunk(sp.n_keys), pos, vel, info, xref, check_guard, gid, key_cell,
                     cse, start, perm, flags);
  return hipGetLastError();
}

// ------------------------------------------------------------------ walls

// Candidate / touching predicates of particle centre x (radius R) against a
// wall at time t, evaluated without square roots; when touching also the unit
// normal from the particle to the wall, the overlap and the lever arm of the
// contact point about the wall's rotation axis (x_c - ax(t)).
struct WallGeo {
  bool candidate, touching;
  // scalars: as arrays filled in branches they ended up in scratch memory
  double n0 = 0.0, n1 = 0.0, n2 = 0.0, dn = 0.0, a0 = 0.0, a1 = 0.0, a2 = 0.0;
  __device__ __forceinline__ void set(double nx, double ny, double nz, double overlap, double ax,
                                      double ay, double az) {
    n0 = nx;
    n1 = ny;
    n2 = nz;
    dn = overlap;
    a0 = ax;
    a1 = ay;
    a2 = az;
  }
};

__device__ inline double dot3(const double* a, const double* b) {
  return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}

__device__ inline void wall_geo(const WallDev& W, const double x[3], double R, double skin,
                                bool need_contact, double t, WallGeo& g) {
  g.candidate = false;
  g.touching = false;
  const double P[3] = {W.p[0] + W.vel[0] * t, W.p[1] + W.vel[1] * t, W.p[2] + W.vel[2] * t};
  double rel[3] = {x[0] - P[0], x[1] - P[1], x[2] - P[2]};
  if (W.kind == 0) {
    double dist = dot3(rel, W.nrm);
    if (W.bounded) {
      double a = dot3(rel, W.u), b = dot3(rel, W.vax);
      if (!(fabs(a) <= W.hu && fabs(b) <= W.hv)) return;
    }
    g.candidate = (dist < R + skin) && (dist > -R);
    g.touching = dist < R;
    if (g.touching && need_contact)
      g.set(-W.nrm[0], -W.nrm[1], -W.nrm[2], R - dist, (rel[0] - dist * W.nrm[0]) - W.axo[0],
            (rel[1] - dist * W.nrm[1]) - W.axo[1], (rel[2] - dist * W.nrm[2]) - W.axo[2]);
    return;
  }
  double sax = dot3(rel, W.nrm);
  if (!(sax >= W.smin && sax <= W.smax)) return;
  double r[3] = {rel[0] - sax * W.nrm[0], rel[1] - sax * W.nrm[1], rel[2] - sax * W.nrm[2]};
  double rho2 = dot3(r, r);
  if (!(rho2 > 0.0)) return;
  if (W.kind == 2) {
    // cone: distance (r(s) - rho) / q inside, (rho - r(s)) / q outside, tested
    // as rho^2 against squared bounds; outward normal (e_rho - slope nrm) / q
    const double q = W.q;
    const double rs = W.radius + W.slope * sax;
    if (W.inside) {
      double lo = rs - (R + skin) * q;
      double hi = rs + R * q;
      bool above = (lo <= 0.0) || (rho2 > lo * lo);
      g.candidate = above && (hi > 0.0) && (rho2 < hi * hi);
      double lt = rs - R * q;
      g.touching = (lt <= 0.0) || (rho2 > lt * lt);
    } else {
      double hi = rs + (R + skin) * q;
      double lo = rs - R * q;
      bool above = (lo <= 0.0) || (rho2 > lo * lo);
      g.candidate = above && (hi > 0.0) && (rho2 < hi * hi);
      double lt = rs + R * q;
      g.touching = (lt > 0.0) && (rho2 < lt * lt);
    }
    if (g.touching && need_contact) {
      const double rho = sqrt(rho2);
      const double dist = W.inside ? (rs - rho) / q : (rho - rs) / q;
      const double m0 = (r[0] / rho - W.slope * W.nrm[0]) / q;
      const double m1 = (r[1] / rho - W.slope * W.nrm[1]) / q;
      const double m2 = (r[2] / rho - W.slope * W.nrm[2]) / q;
      const double n0 = W.inside ? m0 : -m0, n1 = W.inside ? m1 : -m1, n2 = W.inside ? m2 : -m2;
      g.set(n0, n1, n2, R - dist, (rel[0] + dist * n0) - W.axo[0], (rel[1] + dist * n1) - W.axo[1],
            (rel[2] + dist * n2) - W.axo[2]);
    }
    return;
  }
  const double Rc = W.radius;
  if (W.inside) {
    double lo = Rc - (R + skin);
    double hi = Rc + R;
    bool above = (lo <= 0.0) || (rho2 > lo * lo);
    g.candidate = above && (rho2 < hi * hi);
    double lt = Rc - R;
    g.touching = (lt <= 0.0) || (rho2 > lt * lt);
  } else {
    double hi = Rc + R + skin;
    double lo = Rc - R;
    bool above = (lo <= 0.0) || (rho2 > lo * lo);
    g.candidate = above && (rho2 < hi * hi);
    double lt = Rc + R;
    g.touching = rho2 < lt * lt;
  }
  if (g.touching && need_contact) {
    const double rho = sqrt(rho2);
    const double e0 = r[0] / rho, e1 = r[1] / rho, e2 = r[2] / rho;
    const double dist = W.inside ? (Rc - rho) : (rho - Rc);
    g.set(W.inside ? e0 : -e0, W.inside ? e1 : -e1, W.inside ? e2 : -e2, R - dist,
          (sax * W.nrm[0] + Rc * e0) - W.axo[0], (sax * W.nrm[1] + Rc * e1) - W.axo[1],
          (sax * W.nrm[2] + Rc * e2) - W.axo[2]);
  }
}

// ------------------------------------------------------------ mesh walls

// Closest point of the closed triangle T, moved by vel t, to the point x: the
// projection onto the triangle's plane when it lies strictly inside all
// three edges (a face), else the closest of the three edges' own closest
// points (the projection onto the edge line clamped to the edge), on an edge
// when strictly inside it and on a corner otherwise.  s is the signed
// distance from the plane along the unit normal, d2 the squared distance.
struct TriGeo {
  int feature;  // 0 face, 1 edge (corners a, b = a + 1 mod 3), 2 vertex (corner a)
  int a, b;
  double s, d2;
  double q[3];
};

__device__ inline void cross3(const double* a, const double* b, double* r) {
  r[0] = a[1] * b[2] - a[2] * b[1];
  r[1] = a[2] * b[0] - a[0] * b[2];
  r[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ inline void tri_closest(const TriDev& T, const double vel[3], double t,
                                   const double x[3], TriGeo& g) {
  double P[3][3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int k = 0; k < 3; ++k) P[c][k] = T.p[c][k] + vel[k] * t;
  const double rel[3] = {x[0] - P[0][0], x[1] - P[0][1], x[2] - P[0][2]};
  g.s = dot3(rel, T.n);
  bool inside = true;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double r[3] = {x[0] - P[c][0], x[1] - P[c][1], x[2] - P[c][2]};
    double cr[3];
    cross3(T.e[c], r, cr);
    if (!(dot3(cr, T.n) > 0.0)) inside = false;
  }
  if (inside) {
    g.feature = 0;
    g.a = g.b = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) g.q[k] = x[k] - g.s * T.n[k];
    g.d2 = g.s * g.s;
    return;
  }
  g.d2 = INFINITY;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double* E = T.e[c];
    const double r[3] = {x[0] - P[c][0], x[1] - P[c][1], x[2] - P[c][2]};
    const double u = dot3(r, E) / dot3(E, E);
    const double uc = u <= 0.0 ? 0.0 : (u >= 1.0 ? 1.0 : u);
    const double q[3] = {P[c][0] + uc * E[0], P[c][1] + uc * E[1], P[c][2] + uc * E[2]};
    const double dq[3] = {x[0] - q[0], x[1] - q[1], x[2] - q[2]};
    const double d2 = dot3(dq, dq);
    if (d2 < g.d2) {
      g.d2 = d2;
      g.q[0] = q[0];
      g.q[1] = q[1];
      g.q[2] = q[2];
      const int c1 = c == 2 ? 0 : c + 1;
      if (u <= 0.0) {
        g.feature = 2;
        g.a = g.b = c;
      } else if (u >= 1.0) {
        g.feature = 2;
        g.a = g.b = c1;
      } else {
        g.feature = 1;
        g.a = c;
        g.b = c1;
      }
    }
  }
}

// the cell of mesh W's grid that x lies in at time t (-1: outside the grid)
__device__ inline int mesh_cell(const WallDev& W, const double x[3], double t) {
  int c3[3];
  bool in = true;
  for (int k = 0; k < 3; ++k) {
    const double u = (x[k] - W.vel[k] * t - W.mlo[k]) / W.mh;
    if (!(u >= 0.0 && u < (double)W.mnc[k])) in = false;
    c3[k] = in ? (int)u : 0;
  }
  return in ? W.cell_base + c3[0] + W.mnc[0] * (c3[1] + W.mnc[1] * c3[2]) : -1;
}

// ----------------------------------------------------------------- reorder

// Gather every particle array into sorted order, record the reference
// position of the displacement guard, and redo the particle-wall search at
// the new position carrying the tangential overlap of walls already listed.
__global__ void k_reorder(StepParams sp, const InstDev* __restrict__ inst,
                          const int* __restrict__ perm, int* __restrict__ inv, ParticleBufs src,
                          ParticleBufs dst, const int* __restrict__ gid_src,
                          int* __restrict__ gid_dst, const int* __restrict__ info_src,
                          int* __restrict__ info_dst, double4* __restrict__ xref,
                          WallSlots ws_src, WallSlots ws_dst, const WallDev* __restrict__ walls,
                          MeshTables mt, MeshSlots ms_dst, int* __restrict__ near_list,
                          const double4* __restrict__ F_src, const double4* __restrict__ T_src,
                          double4* __restrict__ F_dst, double4* __restrict__ T_dst,
                          const int64_t* __restrict__ clock, int64_t step_rel,
                          int64_t bound_step_rel, int* __restrict__ n_occupied,
                          int* __restrict__ flags) {
  int p = xcd_block() * kBlock + threadIdx.x;
  const int n = sp.n;
  if (blockIdx.x == 0 && threadIdx.x < kDriftSpread) {
    // the positions of the next force evaluation are where this search sees them
    const int r = bound_slot(*clock + bound_step_rel, 0);
    sp.brec[r * kDriftRec + threadIdx.x * kDriftStride] = 0ull;
    if (threadIdx.x == 0) {
      sp.bacc[bound_slot(*clock + bound_step_rel, -1)] = 0.0;
      *n_occupied = 0;  // (k_occupied counts)
    }
  }
  if (p >= n) return;
  const double t = (double)(*clock + step_rel) * sp.dt;  // walls where they are now
  int o = perm[p];
  inv[o] = p;
  double4 ps = src.pos[o];
  dst.pos[p] = ps;
  dst.vel[p] = src.vel[o];
  dst.omg[p] = src.omg[o];
  gid_dst[p] = gid_src[o];
  int inf = info_src[o];
  info_dst[p] = inf;
  xref[p] = ps;
  if (F_src) {
    F_dst[p] = F_src[o];
    T_dst[p] = T_src[o];
  }
  int c = 0;
  if (!(inf & kInactive)) {
    const InstDev& I = inst[inf >> kInstShift];
    double x[3] = {ps.x, ps.y, ps.z};
    for (int w = I.wall_begin; w < I.wall_end; ++w) {
      if (walls[w].kind == 3) continue;
      WallGeo g;
      wall_geo(walls[w], x, ps.w, I.skin, false, t, g);
      if (!g.candidate) continue;
      if (c == kWallSlots) {
        atomicOr(flags, kFlagWallOverflow);
        break;
      }
      double h0 = 0.0, h1 = 0.0, h2 = 0.0;
      for (int s = 0; s < kWallSlots; ++s) {
        int ow = ws_src.wid[(int64_t)s * n + o];
        if (ow < 0) break;
        if (ow == w) {
          h0 = ws_src.hist[(int64_t)(3 * s + 0) * n + o];
          h1 = ws_src.hist[(int64_t)(3 * s + 1) * n + o];
          h2 = ws_src.hist[(int64_t)(3 * s + 2) * n + o];
          break;
        }
      }
      ws_dst.wid[(int64_t)c * n + p] = w;
      ws_dst.hist[(int64_t)(3 * c + 0) * n + p] = h0;
      ws_dst.hist[(int64_t)(3 * c + 1) * n + p] = h1;
      ws_dst.hist[(int64_t)(3 * c + 2) * n + p] = h2;
      ++c;
    }
  }
  for (; c < kWallSlots; ++c) ws_dst.wid[(int64_t)c * n + p] = -1;
  if (!mt.tri) return;
  // the particles whose cell lists a triangle, for k_mesh_find
  for (int s = 0; s < kMeshSlots; ++s) ms_dst.tri[(int64_t)s * n + p] = -1;
  if (!(inf & kInactive)) {
    const InstDev& I = inst[inf >> kInstShift];
    const double x[3] = {ps.x, ps.y, ps.z};
    bool near = false;
    for (int w = I.wall_begin; w < I.wall_end && !near; ++w) {
      if (walls[w].kind != 3) continue;
      const int cb = mesh_cell(walls[w], x, t);
      near = cb >= 0 && mt.cell[cb] < mt.cell[cb + 1];
    }
    if (near) near_list[atomicAdd(ms_dst.list + n + 1, 1)] = p;
  }
}

// Particle-triangle candidates of the sorted particles: the triangles listed
// in the centre's cell of each mesh grid that lie less than R + skin away from
// it, with the centre less than R behind their plane, in that order; overlaps
// carried by triangle.
//
// Over the list of the particles whose cell lists a triangle (k_reorder), with
// eight lanes each: they take the triangles of the cell eight at a time, and a
// candidate's slot follows from the ballot of the lanes before it.  What
// bounds it is a chain of dependent reads per particle (cell, triangle number,
// triangle, old slots).  In a drum of 200,000 one thread per particle, in
// k_reorder, took that to 143 us; eight lanes for every particle of the
// context took 82 here and 14 there, the list 59 and 28, and with the tighter
// lists of cells (build_meshes) 29 and 23.
__global__ void __launch_bounds__(kBlock)
k_mesh_find(StepParams sp, const InstDev* __restrict__ inst, const int* __restrict__ perm,
            const int* __restrict__ near_list, const double4* __restrict__ pos,
            const int* __restrict__ info,
            const WallDev* __restrict__ walls, MeshTables mt, MeshSlots src, MeshSlots dst,
            const int64_t* __restrict__ clock, int64_t step_rel, int* __restrict__ flags) {
  static_assert(kMeshSlots == 8, "a lane per slot");
  const int n = sp.n, count = dst.list[n + 1];
  const int lane = threadIdx.x & 7, shift = threadIdx.x & 56;
  for (int at = (int)(blockIdx.x * kBlock + threadIdx.x) >> 3; at < count;
       at += (int)(gridDim.x * kBlock) >> 3) {
    const int p = near_list[at];
    const int o = perm[p];
    const int inf = info[p];
    const int old = src.tri[(int64_t)lane * n + o];
    int cm = 0;
    const InstDev& I = inst[inf >> kInstShift];
    const double t = (double)(*clock + step_rel) * sp.dt;  // meshes where they are now
    const double4 ps = pos[p];
    const double x[3] = {ps.x, ps.y, ps.z};
    const double R = ps.w;
    const double m = R + I.skin;
    for (int w = I.wall_begin; w < I.wall_end && cm <= kMeshSlots; ++w) {
      const WallDev& W = walls[w];
      if (W.kind != 3) continue;
      const int cb = mesh_cell(W, x, t);
      if (cb < 0) continue;
      const int q1 = mt.cell[cb + 1];
      for (int q = mt.cell[cb]; q < q1; q += 8) {
        const int tr = q + lane < q1 ? mt.cell_tri[q + lane] : -1;
        bool near = false;
        if (tr >= 0) {
          TriGeo g;
          tri_closest(mt.tri[tr], W.vel, t, x, g);
          near = g.s > -R && g.d2 < m * m;
        }
        const unsigned found = (unsigned)(__ballot(near) >> shift) & 0xffu;
        if (found == 0u) continue;
        int from = -1;  // the slot that had this triangle (a triangle is in one only)
#pragma unroll
        for (int s = 0; s < kMeshSlots; ++s)
          if (__shfl(old, shift + s, 64) == tr) from = s;
        const int slot = cm + __popc(found & ((1u << lane) - 1u));
        if (near && slot < kMeshSlots) {
          double h0 = 0.0, h1 = 0.0, h2 = 0.0;
          if (from >= 0) {
            h0 = src.hist[(int64_t)(3 * from + 0) * n + o];
            h1 = src.hist[(int64_t)(3 * from + 1) * n + o];
            h2 = src.hist[(int64_t)(3 * from + 2) * n + o];
          }
          dst.tri[(int64_t)slot * n + p] = tr;
          dst.hist[(int64_t)(3 * slot + 0) * n + p] = h0;
          dst.hist[(int64_t)(3 * slot + 1) * n + p] = h1;
          dst.hist[(int64_t)(3 * slot + 2) * n + p] = h2;
        }
        cm += __popc(found);
        if (cm > kMeshSlots) {
          if (lane == 0) atomicOr(flags, kFlagMeshOverflow);
          break;
        }
      }
    }
    if (lane >= cm) dst.tri[(int64_t)lane * n + p] = -1;
    if (lane == 0 && cm > 0) dst.list[atomicAdd(dst.list + n, 1)] = p;
  }
}

// Workgroups of 32 particles each: enough to keep the chip busy, and no more
// than a context can need (one for a context without particles: a launch has
// to have one).
static unsigned mesh_grid(int n) {
  const int64_t b = std::max<int64_t>(((int64_t)n + 31) / 32, 1);
  return (unsigned)(b < 2048 ? b : 2048);
}

hipError_t launch_reorder(const StepParams& sp, const InstDev* inst, const int* perm, int* inv,
                          ParticleBufs src, ParticleBufs dst, const int* gid_src, int* gid_dst,
                          const int* info_src, int* info_dst, double4* xref,
                          WallSlots ws_src, WallSlots ws_dst, const WallDev* walls,
                          MeshTables mt, MeshSlots ms_src, MeshSlots ms_dst, int* near_list,
                          const double4* F_src, const double4* T_src, double4* F_dst,
                          double4* T_dst, const int64_t* clock, int64_t step_rel,
                          int64_t bound_step_rel, int* n_occupied, int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_reorder, dim3(grid_for(sp.n)), dim3(kBlock), 0, s, sp, inst, perm, inv,
                     src, dst,
                     gid_src, gid_dst, info_src, info_dst, xref, ws_src, ws_dst, walls, mt, ms_dst,
                     near_list, F_src, T_src, F_dst, T_dst, clock, step_rel, bound_step_rel,
                     n_occupied, flags);
  if (mt.tri)
    hipLaunchKernelGGL(k_mesh_find, dim3(mesh_grid(sp.n)), dim3(kBlock), 0, s, sp, inst, perm,
                       near_list, dst.pos, info_dst, walls, mt, ms_src, ms_dst, clock, step_rel,
                       flags);
  return hipGetLastError();
}

// ------------------------------------------------------------------ search

// Gap class of a candidate pair at distance^2 d2 (radius sum rsum, skin sk):
// 0 touching, 1..3 gap d - rsum below kCutFrac[0..2] skins, 4 farther
// (compared as squares, so no square root; the force evaluation keeps a
// relative margin far above the rounding of these comparisons).
__device__ __forceinline__ int gap_class(double d2, double rsum, double sk) {
  const double a = rsum + kCutFrac[0] * sk, b = rsum + kCutFrac[1] * sk,
               c = rsum + kCutFrac[2] * sk;
  return d2 < rsum * rsum ? 0 : (d2 < a * a ? 1 : (d2 < b * b ? 2 : (d2 < c * c ? 3 : 4)));
}

constexpr unsigned kRowIndexMask = (1u << kClassShift) - 1u;

// A row being sorted: its first `cap` entries in the workgroup's LDS (column
// threadIdx.x, so the lanes of a wavefront always hit distinct banks), the
// rest in place in the neighbour list.
constexpr int kCarryBatch = 8;
struct BuildRow {
  unsigned* lds;  // &buf[0][threadIdx.x], stride kBlock
  int* nbr;
  int p, max_nb, cap;
  __device__ __forceinline__ unsigned load(int t) const {
    return t < cap ? lds[t * kBlock] : (unsigned)nbr[nbr_entry(p, t, max_nb)];
  }
  __device__ __forceinline__ void store(int t, unsigned v) const {
    if (t < cap)
      lds[t * kBlock] = v;
    else
      nbr[nbr_entry(p, t, max_nb)] = (int)v;
  }
};

// Broad + fine search: the pairs of particles of a cell and its 26 neighbours
// with |x_q - x_p|^2 < r_s^2 (evaluated in FP64 in a fixed order without fused
// operations).
//
// A workgroup takes a block of cells (4 x 4 x 4 for equal spheres).  The
// particles of the block's cells and of the layer of cells around it are
// staged in LDS, in the order of the cells (x fastest), as FP32 coordinates in
// cell edges from the region's corner with the sorted index beside them: 16
// bytes each, and the three cells x - 1, x, x + 1 of a scan lie side by side,
// so a particle goes through 9 stretches of LDS instead of 27 cells of the
// position array.  What the scan lets through is a little more than r_s
// (near2 covers the rounding of the coordinates); those, about 9 of the 67
// candidates, are then tested on their FP64 positions, in the order found.
// Bound by the latency of LDS and of those positions; a workgroup per occupied
// block spreads the work best (workgroups that go through several blocks took
// twice as long, the occupied blocks being unevenly spread).  Where blocks hold
// too few particles for a workgroup, each particle's 27 cells are read by a
// thread of its own (search_way).
//
// The rows come out in the order of a scan of the 27 cells (z, y, x).  A
// second kernel puts the pairs that touch now at the front (during the next
// steps the history accesses of a wavefront then stay in few cache lines) and
// the others behind them in the order of their gap class (the row cuts of
// NbrList), and carries the tangential overlaps over: it needs other
// resources (many wavefronts for its chain of loads, no region in LDS), and
// together the two take 249 us for a bed of 1M equal spheres and 1.88 ms for
// 4.3M log-normal ones, where one kernel over the sorted particles, testing
// every candidate's FP64 position, took 337 us and 2.96 ms.

constexpr int kRegionCells = 6 * 6 * 6;
constexpr int kNearBatch = 4;
constexpr int kScanBatch = 4;

struct RegionTile {
  float4 p[kSearchRegion + kScanBatch];  // x, y, z in cell edges; sorted index as bits
  int first[kRegionCells + 1];   // local start of each region cell
  int sums[kBlock / 64];
};

// Row of particle p from the positions alone, in the same order as the scan of
// the staged region (used where the region does not fit in LDS, or where the
// FP32 pretest let more through than its list holds).  Returns the number of
// pairs, of which the first max_nb are stored.
// held: positions of the particles [h0, h0 + n_held).
__device__ __forceinline__ int scan_cells(const InstDev& I, const double4* held, int h0,
                                          int n_held, const double4* __restrict__ pos,
                                          const int2* __restrict__ cse, int* __restrict__ nbr,
                                          int p, int max_nb, const double4 pp, int cx, int cy,
                                          int cz) {
  const GridDev& g = I.grid;
  int len = 0;
  for (int z = cz > 0 ? cz - 1 : 0; z <= cz + 1 && z < g.nc[2]; ++z)
    for (int y = cy > 0 ? cy - 1 : 0; y <= cy + 1 && y < g.nc[1]; ++y) {
      // the cells of row (y, z), each with its (start, end) in sorted order
      // (fewer than 2^30 cells: the index fits an int)
      const int2* crow = cse + I.key_base + (z * g.nc[1] + y) * g.nc[0];
      for (int x = cx > 0 ? cx - 1 : 0; x <= cx + 1 && x < g.nc[0]; ++x) {
        const int2 se = crow[x];
        for (int q = se.x; q < se.y; ++q) {
          if (q == p) continue;
          const double4 pq = (unsigned)(q - h0) < (unsigned)n_held ? held[q - h0] : pos[q];
          const double dx = pq.x - pp.x, dy = pq.y - pp.y, dz = pq.z - pp.z;
          const double d2 = (dx * dx + dy * dy) + dz * dz;
          if (!(d2 < I.rs2)) continue;
          const int c = gap_class(d2, pp.w + pq.w, I.skin);
          if (len < max_nb)
            nbr[nbr_entry(p, len, max_nb)] = (int)((unsigned)q | ((unsigned)c << kClassShift));
          ++len;
        }
      }
    }
  return len;
}

// The length of the row found for particle p; with more than max_nb pairs the
// row is incomplete and the step fails (marked by the sign for k_finish_rows).
__device__ __forceinline__ void store_len(const StepParams& sp, const NbrList& l, int p, int len,
                                          int* __restrict__ flags) {
  if (len > sp.max_nb) {
    atomicOr(flags, kFlagNbrOverflow);
    len = -sp.max_nb;
  }
  l.rowlen[p] = len;
}

// Row of particle p through the staged region: the candidates within near2
// first (their local indices to `list`, stride kBlock), then the exact test of
// those, kNearBatch positions in flight at a time.  Nearly all of them pass,
// so the entries of a wavefront's rows are stored in step, whole lines at a
// time.  Returns -1 when more passed the pretest than the list holds.
__device__ __forceinline__ int scan_region(const InstDev& I, const RegionTile& tile,
                                           uint16_t* list, int cap, int r0, int r01,
                                           const double4* __restrict__ pos,
                                           int* __restrict__ nbr, int p, int max_nb,
                                           const double4 pp, const float3 pf, int lc) {
  const float near2 = I.near2;
  int near = 0;
  for (int dz = -r01; dz <= r01; dz += r01)
    for (int dy = -r0; dy <= r0; dy += r0) {
      const int c = lc + dz + dy;
      const int e = tile.first[c + 2];
      for (int j0 = tile.first[c - 1]; j0 < e; j0 += kScanBatch) {
        float4 f[kScanBatch];  // (past the end: the particles that follow, not counted)
#pragma unroll
        for (int u = 0; u < kScanBatch; ++u) f[u] = tile.p[j0 + u];
#pragma unroll
        for (int u = 0; u < kScanBatch; ++u) {
          const float dx = f[u].x - pf.x, dy1 = f[u].y - pf.y, dz1 = f[u].z - pf.z;
          const float d2 = __builtin_fmaf(dz1, dz1, __builtin_fmaf(dy1, dy1, dx * dx));
          if (!(d2 < near2) || j0 + u >= e || __float_as_int(f[u].w) == p) continue;
          if (near < cap) list[near * kBlock] = (uint16_t)(j0 + u);
          ++near;
        }
      }
    }
  if (near > cap) return -1;
  const double rs2 = I.rs2, sk = I.skin;
  int len = 0;
  for (int t0 = 0; t0 < near; t0 += kNearBatch) {
    int q[kNearBatch];
    double4 pq[kNearBatch];
#pragma unroll
    for (int j = 0; j < kNearBatch; ++j)
      if (t0 + j < near) q[j] = __float_as_int(tile.p[list[(t0 + j) * kBlock]].w);
#pragma unroll
    for (int j = 0; j < kNearBatch; ++j)
      if (t0 + j < near) pq[j] = pos[q[j]];
#pragma unroll
    for (int j = 0; j < kNearBatch; ++j) {
      if (t0 + j >= near) continue;
      const double dx = pq[j].x - pp.x, dy = pq[j].y - pp.y, dz = pq[j].z - pp.z;
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      if (!(d2 < rs2)) continue;
      const int c = gap_class(d2, pp.w + pq[j].w, sk);
      if (len < max_nb)
        nbr[nbr_entry(p, len, max_nb)] = (int)((unsigned)q[j] | ((unsigned)c << kClassShift));
      ++len;
    }
  }
  return len;
}

// Occupied search blocks (in any order: no result depends on it) and their
// number, with one atomic to a workgroup.
__global__ void k_occupied(const SearchBlock* __restrict__ blocks, int n_blocks,
                           const int* __restrict__ start, int* __restrict__ list,
                           int* __restrict__ count) {
  __shared__ int sh[4], first;
  const int b = (int)blockIdx.x * kBlock + (int)threadIdx.x;
  bool full = false;
  if (b < n_blocks) full = start[blocks[b].key] < start[blocks[b].key + blocks[b].ncell];
  int total;
  const int at = block_exclusive_scan(full ? 1 : 0, sh, &total);
  if (threadIdx.x == 0 && total > 0) first = atomicAdd(count, total);
  __syncthreads();
  if (full) list[first + at] = b;
}

// Whether a search with a list of the occupied blocks goes by blocks: where
// these hold fewer than kBlockMin particles on average the rows are taken one
// thread per sorted particle instead, since the time of a workgroup is that of
// its region (up to 216 cell ranges), whatever the block holds.
__device__ __forceinline__ bool by_blocks(const int* __restrict__ count, int n_active) {
  return (int64_t)*count * kBlockMin <= n_active;
}

// Every row, one thread per sorted particle (with count: unless by_blocks).  The
// workgroup's positions are staged in LDS: most candidates of particles in
// spatial order lie among them.  Bound by the latency of the candidates' loads,
// hence eight wavefronts per SIMD.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8)))
k_scan_each(const InstDev* __restrict__ inst, StepParams sp, const int* __restrict__ count,
            const double4* __restrict__ pos, const int* __restrict__ info,
            const int2* __restrict__ cse, const int* __restrict__ start, NbrList l,
            int* __restrict__ flags) {
  __shared__ double4 held[kBlock];
  const int n_active = start[sp.n_keys];  // particles in cells: they come first
  if (count && by_blocks(count, n_active)) return;
  const int p0 = xcd_block() * kBlock, p = p0 + (int)threadIdx.x;
  double4 pp = make_double4(0.0, 0.0, 0.0, 0.0);
  if (p < n_active) held[threadIdx.x] = pp = pos[p];
  __syncthreads();
  if (p >= n_active) return;
  const int n_held = n_active - p0 < kBlock ? n_active - p0 : kBlock;
  // once for every instance among the wavefront's lanes (nearly always one,
  // whose table entry then sits in scalar registers)
  const int b = info[p] >> kInstShift;
  for (;;) {
    const int u = __builtin_amdgcn_readfirstlane(b);
    if (b != u) continue;
    const InstDev& I = inst[u];
    const GridDev& g = I.grid;
    store_len(sp, l, p,
              scan_cells(I, held, p0, n_held, pos, cse, l.nbr, p, sp.max_nb, pp,
                         cell_coord(pp.x, g.lo[0], g.h, g.nc[0]),
                         cell_coord(pp.y, g.lo[1], g.h, g.nc[1]),
                         cell_coord(pp.z, g.lo[2], g.h, g.nc[2])),
              flags);
    return;
  }
}

// One workgroup per block, or with a list per occupied block (blocks list[0 ..
// *count)) if by_blocks.
// The rows are left in the order found, the gap class in the top bits of each
// entry, for k_finish_rows.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6)))
k_scan_rows(const InstDev* __restrict__ inst, StepParams sp,
            const SearchBlock* __restrict__ blocks, const int* __restrict__ list,
            const int* __restrict__ count, const double4* __restrict__ pos,
            const int2* __restrict__ cse, const int* __restrict__ start, NbrList l,
            int* __restrict__ flags) {
  __shared__ RegionTile tile;
  extern __shared__ uint16_t near_lists[];  // sp.list_cap x kBlock
  const int tid = threadIdx.x;
  int b = blockIdx.x;
  if (list) {
    if (b >= *count || !by_blocks(count, start[sp.n_keys])) return;
    b = list[b];
  }
  const SearchBlock B = blocks[b];
  const int p0 = start[B.key], p1 = start[B.key + B.ncell];
  if (p0 == p1) return;
  const InstDev& I = inst[B.inst];
  const GridDev& g = I.grid;
  // region: the block's cells and one layer around them (cells outside
  // the grid are empty)
  const int r0 = (1 << sp.sb_bits[0]) + 2, r1 = (1 << sp.sb_bits[1]) + 2;
  const int ncr = r0 * r1 * ((1 << sp.sb_bits[2]) + 2);
  int2 se = make_int2(0, 0);
  if (tid < ncr) {
    const int ryz = tid / r0;
    const int x = B.x - 1 + (tid - ryz * r0), y = B.y - 1 + ryz % r1, z = B.z - 1 + ryz / r1;
    if (x >= 0 && x < g.nc[0] && y >= 0 && y < g.nc[1] && z >= 0 && z < g.nc[2])
      se = cse[I.key_base + (z * g.nc[1] + y) * g.nc[0] + x];
  }
  int total;
  const int at = block_exclusive_scan(se.y - se.x, tile.sums, &total);
  if (tid <= ncr) tile.first[tid] = at;
  const bool staged = total <= kSearchRegion;
  // coordinates in cell edges from the corner of cell (B.x - 1, ...)
  const double o0 = g.lo[0] + (B.x - 1) * g.h, o1 = g.lo[1] + (B.y - 1) * g.h,
               o2 = g.lo[2] + (B.z - 1) * g.h;
  if (staged)
    for (int q0 = se.x; q0 < se.y; q0 += kNearBatch) {
      double4 x[kNearBatch];
#pragma unroll
      for (int u = 0; u < kNearBatch; ++u)
        if (q0 + u < se.y) x[u] = pos[q0 + u];
#pragma unroll
      for (int u = 0; u < kNearBatch; ++u)
        if (q0 + u < se.y)
          tile.p[at + (q0 + u - se.x)] = make_float4(
              (float)((x[u].x - o0) * I.ih), (float)((x[u].y - o1) * I.ih),
              (float)((x[u].z - o2) * I.ih), __int_as_float(q0 + u));
    }
  __syncthreads();
  for (int p = p0 + tid; p < p1; p += kBlock) {
    const double4 pp = pos[p];
    const int cx = cell_coord(pp.x, g.lo[0], g.h, g.nc[0]);
    const int cy = cell_coord(pp.y, g.lo[1], g.h, g.nc[1]);
    const int cz = cell_coord(pp.z, g.lo[2], g.h, g.nc[2]);
    int len = -1;
    if (staged)
      len = scan_region(I, tile, near_lists + tid, sp.list_cap, r0, r0 * r1, pos, l.nbr, p,
                        sp.max_nb, pp,
                        make_float3((float)((pp.x - o0) * I.ih), (float)((pp.y - o1) * I.ih),
                                    (float)((pp.z - o2) * I.ih)),
                        ((cz - B.z + 1) * r1 + (cy - B.y + 1)) * r0 + (cx - B.x + 1));
    if (len < 0)
      len = scan_cells(I, nullptr, 0, 0, pos, cse, l.nbr, p, sp.max_nb, pp, cx, cy, cz);
    store_len(sp, l, p, len, flags);
  }
}

// The rows of k_scan_rows sorted by class in place, clearing the class bits,
// and the tangential overlaps carried over: those of the pairs that touched at
// the last force evaluation and touch now (a pair that does not touch now has
// its overlap restarted at zero by the first evaluation, at these positions,
// anyway).  One thread per particle at eight wavefronts per SIMD: it is bound
// by the chain of loads of the carry-over.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8)))
k_finish_rows(int n, int max_nb, const int* __restrict__ info, const int* __restrict__ perm,
              const int* __restrict__ inv, NbrList old_l, NbrList new_l, int row_cap) {
  extern __shared__ unsigned row_lds[];  // row_cap x kBlock
  const int p = xcd_block() * kBlock + threadIdx.x;
  if (p >= n) return;
  if (info[p] & kInactive) {
    new_l.rowlen[p] = 0;
    new_l.rowcut[p] = 0;
    return;
  }
  const BuildRow row{row_lds + threadIdx.x, new_l.nbr, p, max_nb, row_cap};
  int len = new_l.rowlen[p];
  const bool overflow = len < 0;
  if (overflow) len = -len;
  const int held = len < row_cap ? len : row_cap;
  for (int k0 = 0; k0 < held; k0 += kCarryBatch) {
    int e[kCarryBatch];
#pragma unroll
    for (int j = 0; j < kCarryBatch; ++j)
      if (k0 + j < held) e[j] = new_l.nbr[nbr_entry(p, k0 + j, max_nb)];
#pragma unroll
    for (int j = 0; j < kCarryBatch; ++j)
      if (k0 + j < held) row.lds[(k0 + j) * kBlock] = (unsigned)e[j];
  }
  int front = 0;
  int cut = (kCutMask << (2 * kCutBits)) | (kCutMask << kCutBits) | kCutMask;
  if (!overflow) {
    // class sizes (classes 0..3; 16 bits each) and the ends of classes 0..3
    uint64_t at = 0;
    for (int t = 0; t < len; ++t) {
      const unsigned c = row.load(t) >> kClassShift;
      at += c < 4u ? 1ull << (16u * c) : 0ull;
    }
    const int e0 = (int)(at & 0xffff), e1 = e0 + (int)((at >> 16) & 0xffff),
              e2 = e1 + (int)((at >> 32) & 0xffff), e3 = e2 + (int)(at >> 48);
    // In-place sort by class: the slots of class 0, 1, 2, 3 are filled in
    // order; an entry found in one of them that belongs to a later class goes
    // to the next free slot of its class, whose occupant moves on in turn,
    // until an entry of the slot's own class comes back (the rest is class 4).
    // One move per turn of a single loop, so that the lanes of a wavefront, at
    // different slots and classes, stay together (a loop per class with a loop
    // per chain inside: 1.03 instead of 0.56 ms for 4.3M rows of 24 entries
    // without histories, 66 instead of 50 us for 1M of 9).
    uint64_t nx = (uint64_t)e0 | ((uint64_t)e1 << 16) | ((uint64_t)e2 << 32) | ((uint64_t)e3 << 48);
    int c = 0, t = 0, end = e0;
    bool held_one = false;
    unsigned v = 0;
    while (c < 4) {
      if (t == end) {
        // next class: its slots from the first that no chain has filled
        t = (int)((nx >> (16 * c)) & 0xffff);
        ++c;
        end = c == 1 ? e1 : (c == 2 ? e2 : e3);
        continue;
      }
      if (!held_one) v = row.load(t);
      const int k = (int)(v >> kClassShift);
      if (k == c) {
        if (held_one) row.store(t, v);
        held_one = false;
        ++t;
      } else {
        const int u = (int)((nx >> (16 * (k - 1))) & 0xffff);
        nx += 1ull << (16 * (k - 1));
        const unsigned f = row.load(u);
        row.store(u, v);
        v = f;
        held_one = true;
      }
    }
    front = e0;
    const int c1 = e1 < kCutMask ? e1 : kCutMask;
    const int c2 = e2 < kCutMask ? e2 : kCutMask;
    const int c3 = e3 < kCutMask ? e3 : kCutMask;
    cut = c1 | (c2 << kCutBits) | (c3 << (2 * kCutBits));
  }
  new_l.rowlen[p] = len;
  new_l.rowcut[p] = cut;
  // every entry of p's old row with bit 31 names its partner by old index; inv
  // maps it to the new index, which is looked up among the touching entries of
  // the new row.  Entries without bit 31 have zero history, which is never
  // stored.  The old entries, their inverse-permutation lookups and the
  // histories of the matched pairs are fetched kCarryBatch entries at a time,
  // so that their loads are in flight together.
  const int op = perm[p];
  const int olen = old_l.rowlen[op];
  for (int k0 = 0; k0 < olen; k0 += kCarryBatch) {
    int oj[kCarryBatch], qn[kCarryBatch];
#pragma unroll
    for (int j = 0; j < kCarryBatch; ++j)
      oj[j] = k0 + j < olen ? old_l.nbr[nbr_entry(op, k0 + j, max_nb)] : 0;
#pragma unroll
    for (int j = 0; j < kCarryBatch; ++j)
      qn[j] = (oj[j] & (int)0x80000000u) ? inv[oj[j] & 0x7fffffff] : -1;
    int mj[kCarryBatch];
#pragma unroll
    for (int j = 0; j < kCarryBatch; ++j) {
      mj[j] = -1;
      if (qn[j] < 0) continue;
      const unsigned q = (unsigned)qn[j];
      for (int m = 0; m < front; ++m) {
        if (row.load(m) == q) {
          row.store(m, q | 0x80000000u);
          mj[j] = m;
          break;
        }
      }
    }
    // (four histories at a time: registers)
#pragma unroll
    for (int j0 = 0; j0 < kCarryBatch; j0 += 4) {
      double h0[4], h1[4], h2[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (mj[j0 + j] < 0) continue;
        const int64_t oe = nbr_entry(op, k0 + j0 + j, max_nb);
        h0[j] = old_l.hist[oe];
        h1[j] = old_l.hist[old_l.cap + oe];
        h2[j] = old_l.hist[2 * old_l.cap + oe];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (mj[j0 + j] < 0) continue;
        const int64_t ne = nbr_entry(p, mj[j0 + j], max_nb);
        new_l.hist[ne] = h0[j];
        new_l.hist[new_l.cap + ne] = h1[j];
        new_l.hist[2 * new_l.cap + ne] = h2[j];
      }
    }
  }
  // the part of the row held in LDS goes out entry by entry for the whole
  // wavefront at once (whole cache lines; the part beyond is in place), without
  // the class bits (those of touching pairs are zero; their top bit is set
  // where a history was carried)
  for (int k = 0; k < len; ++k) {
    const unsigned v = row.load(k);
    if (k < held || k >= front)
      new_l.nbr[nbr_entry(p, k, max_nb)] = (int)(k < front ? v : v & kRowIndexMask);
  }
}

hipError_t launch_search(const InstDev* inst, const StepParams& sp, const SearchBlock* blocks,
                         int n_blocks, int* occupied, const double4* pos, const int* info,
                         const int2* cse, const int* start, const int* perm, const int* inv,
                         NbrList old_l, NbrList new_l, int* flags, hipStream_t s) {
  if (sp.n <= 0 || n_blocks <= 0) return hipSuccess;
  const int way = search_way(sp.n, n_blocks, sp.sb_fits);
  int* list = way == kSearchListed ? occupied : nullptr;
  int* count = list ? list + n_blocks : nullptr;
  if (list)
    hipLaunchKernelGGL(k_occupied, dim3((unsigned)((n_blocks + kBlock - 1) / kBlock)), dim3(kBlock),
                       0, s, blocks, n_blocks, start, list, count);
  if (way != kSearchBlocks)
    hipLaunchKernelGGL(k_scan_each, dim3(grid_for(sp.n)), dim3(kBlock), 0, s, inst, sp, count, pos,
                       info, cse, start, new_l, flags);
  if (way != kSearchEach)
    hipLaunchKernelGGL(k_scan_rows, dim3(search_workgroups(sp.n, n_blocks, way)), dim3(kBlock),
                       (size_t)sp.list_cap * kBlock * sizeof(uint16_t), s, inst, sp, blocks, list,
                       count, pos, cse, start, new_l, flags);
  hipLaunchKernelGGL(k_finish_rows, dim3(grid_for(sp.n)), dim3(kBlock),
                     (size_t)sp.row_cap * kBlock * sizeof(unsigned), s, sp.n, sp.max_nb, info,
                     perm, inv, old_l, new_l, sp.row_cap);
  return hipGetLastError();
}

// ------------------------------------------------------------- contact law

// Square roots and reciprocals.  Double: the hardware estimates refined by two
// Newton-Raphson steps each (rsqrt: y <- y (3 - x y^2) / 2; reciprocal:
// y <- y (2 - x y)), a few ulp from the correctly rounded value, far cheaper
// than the correctly rounded library sequences.  Float: the single hardware
// instructions (about 1 ulp).  Every function of a symmetric argument returns
// the same value whichever side of the pair evaluates it.
template <typename R>
struct Fast;

template <>
struct Fast<double> {
  static __device__ __forceinline__ double rsqrt(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double h = 0.5 * x;
    y = y * fma(-h * y, y, 1.5);
    y = y * fma(-h * y, y, 1.5);
    return y;
  }
  static __device__ __forceinline__ double rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    y = fma(y, fma(-x, y, 1.0), y);
    return y;
  }
  static __device__ __forceinline__ double sqrt(double x) {
    return x > 0.0 ? x * rsqrt(x) : 0.0;
  }
  // fifth root: a single-precision estimate 2^(log2(x) / 5) refined by two
  // steps of Newton's iteration for y^5 = x, y <- (4 y + x / y^4) / 5 (the
  // error squares at each step: about 1e-7, 1e-14, then FP64 rounding)
  static __device__ __forceinline__ double root5(double x) {
    if (!(x > 0.0)) return 0.0;
    double y = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)x) * 0.2f);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const double y2 = y * y;
      y = 0.8 * y + (0.2 * x) * rcp(y2 * y2);
    }
    return y;
  }
};

template <>
struct Fast<float> {
  static __device__ __forceinline__ float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
  static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
  static __device__ __forceinline__ float sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
  static __device__ __forceinline__ float root5(float x) { return ::powf(x, 0.2f); }
};

// The spring-dashpot law (Sec. 2.1) in arithmetic type R for one contact,
// given the overlap dn >= 0, the unit normal n from body i to body j, the
// contact relative velocity vij, wrel = omega_i - omega_j, the rolling speed
// vr = |V_omega| (table of rolling models; used by the viscous model), the effective mass
// and radius and the lever arm Ri.  The tangential overlap dtl stays in FP64
// and is updated in place (Eq. delta_t before the force, Coulomb truncation
// of Eqs. coulomb_overlap..3 after it).  Output: force and torque on body i.
// model 0, Hertz-Mindlin: k_n = (4/3) Y_e q, k_t = 8 G_e q, eta = -2 sqrt(5/6)
// beta sqrt(S m_e), q = sqrt(R_e dn); the per-pair constants are c.kn = 4/3
// Y_e, c.kt = 8 G_e, c.en = -2 sqrt(5/6) beta sqrt(2 Y_e), c.et = -2 sqrt(5/6)
// beta sqrt(8 G_e).  model 1, linear (Eqs. linearkn, linearetan, the same
// constants tangentially): k = c.kn (R_e^2 m_e)^(1/5) with c.kn = (16/15) Y_e
// (15 V^2 / (16 Y_e))^(1/5), eta = c.en sqrt(m_e k) with c.en = 2 / sqrt(1 +
// (pi / ln e)^2).
template <typename R>
__device__ __forceinline__ void hm_law(const PairCoef& c, int rolling, int model, double dt,
                                       R dn, const R n[3], const R vij[3], const R wrel[3],
                                       R vr, R me, R Re, R Ri, double dtl[3],
                                       double Fi[3], double Mi[3]) {
  using M = Fast<R>;
  const R vn = (vij[0] * n[0] + vij[1] * n[1]) + vij[2] * n[2];
  const R vrn[3] = {vn * n[0], vn * n[1], vn * n[2]};
  const R vrt[3] = {vij[0] - vrn[0], vij[1] - vrn[1], vij[2] - vrn[2]};
  dtl[0] = dtl[0] + (double)vrt[0] * dt;
  dtl[1] = dtl[1] + (double)vrt[1] * dt;
  dtl[2] = dtl[2] + (double)vrt[2] * dt;
  R kn, kt, etan, etat;
  if (model == 0) {
    const R q = M::sqrt(Re * dn);
    kn = (R)c.kn * q;
    kt = (R)c.kt * q;
    const R sq = M::sqrt(me * q);
    etan = (R)c.en * sq;
    etat = (R)c.et * sq;
  } else {
    kn = (R)c.kn * M::root5((Re * Re) * me);
    kt = kn;
    etan = (R)c.en * M::sqrt(me * kn);
    etat = etan;
  }
  const R knd = kn * dn;
  R Fn[3], Ft[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Fn[k] = -(knd * n[k]) - etan * vrn[k];
    Ft[k] = -(kt * (R)dtl[k]) - etat * vrt[k];
  }
  const R fn2 = (Fn[0] * Fn[0] + Fn[1] * Fn[1]) + Fn[2] * Fn[2];
  const R ft2 = (Ft[0] * Ft[0] + Ft[1] * Ft[1]) + Ft[2] * Ft[2];
  const R fn = M::sqrt(fn2);
  const R mufn = (R)c.mu * fn;
  if (ft2 >= mufn * mufn && ft2 > (R)0) {
    const R ratio = mufn * M::rsqrt(ft2);
    const R mikt = -M::rcp(kt);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const R fhat = ratio * Ft[k];
      dtl[k] = (double)((fhat + etat * vrt[k]) * mikt);
      Ft[k] = fhat;
    }
  }
  R Mr[3] = {(R)0, (R)0, (R)0};
  if (rolling != 0) {
    const R wn2 = (wrel[0] * wrel[0] + wrel[1] * wrel[1]) + wrel[2] * wrel[2];
    if (wn2 > (R)0) {
      R mag = (R)c.mur * Re * fn;  // constant torque; viscous: times |V_omega|
      if (rolling == 2) mag = mag * vr;
      const R sc = -mag * M::rsqrt(wn2);
      Mr[0] = sc * wrel[0];
      Mr[1] = sc * wrel[1];
      Mr[2] = sc * wrel[2];
    }
  }
  const R nx[3] = {n[1] * Ft[2] - n[2] * Ft[1], n[2] * Ft[0] - n[0] * Ft[2],
                   n[0] * Ft[1] - n[1] * Ft[0]};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Fi[k] = (double)(Fn[k] + Ft[k]);
    Mi[k] = (double)(Ri * nx[k] + Mr[k]);
  }
}

// Particle i against a touching neighbour j, evaluated from i's side
// (pos = (x, R), vel = (v, 1/m), omg = (omega, 1/I)).  Written so that the
// evaluation from j's side gives exactly -F and -delta_t: every symmetric
// quantity is formed from commutative operations of the two particles' data.
template <typename R>
__device__ __forceinline__ void pp_contact(const PairCoef& c, int rolling, int model, double dt,
                                           double4 xi, double4 vi, double4 wi, double4 xj,
                                           double4 vj, double4 wj, double dtl[3], double Fi[3],
                                           double Mi[3]);

template <>
__device__ __forceinline__ void pp_contact<double>(const PairCoef& c, int rolling, int model,
                                                   double dt,
                                                   double4 xi, double4 vi, double4 wi,
                                                   double4 xj, double4 vj, double4 wj,
                                                   double dtl[3], double Fi[3], double Mi[3]) {
  using M = Fast<double>;
  const double dx[3] = {xj.x - xi.x, xj.y - xi.y, xj.z - xi.z};
  const double d2 = (dx[0] * dx[0] + dx[1] * dx[1]) + dx[2] * dx[2];
  const double Ri = xi.w, Rj = xj.w;
  const double rsum = Ri + Rj;
  const double inv_d = M::rsqrt(d2);
  double dn = rsum - d2 * inv_d;
  if (dn < 0.0) dn = 0.0;
  const double n[3] = {dx[0] * inv_d, dx[1] * inv_d, dx[2] * inv_d};
  const double rw[3] = {Ri * wi.x + Rj * wj.x, Ri * wi.y + Rj * wj.y, Ri * wi.z + Rj * wj.z};
  // rolling velocity V_omega = (R_i w_i + R_j w_j) x n, part of the contact velocity
  const double vroll[3] = {rw[1] * n[2] - rw[2] * n[1], rw[2] * n[0] - rw[0] * n[2],
                           rw[0] * n[1] - rw[1] * n[0]};
  const double vij[3] = {(vi.x - vj.x) + vroll[0], (vi.y - vj.y) + vroll[1],
                         (vi.z - vj.z) + vroll[2]};
  const double wrel[3] = {wi.x - wj.x, wi.y - wj.y, wi.z - wj.z};
  const double me = M::rcp(vi.w + vj.w);
  const double Re = (Ri * Rj) * M::rcp(rsum);
  const double vr = rolling == 2 ? M::sqrt(dot3(vroll, vroll)) : 0.0;
  hm_law<double>(c, rolling, model, dt, dn, n, vij, wrel, vr, me, Re, Ri, dtl, Fi, Mi);
}

// FP32 contact law.  The overlap is formed without cancellation:
// dn = (rsum^2 - d^2) / (rsum + d) with the numerator from FP64 positions.
template <>
__device__ __forceinline__ void pp_contact<float>(const PairCoef& c, int rolling, int model,
                                                  double dt,
                                                  double4 xi, double4 vi, double4 wi,
                                                  double4 xj, double4 vj, double4 wj,
                                                  double dtl[3], double Fi[3], double Mi[3]) {
  using M = Fast<float>;
  const double dx[3] = {xj.x - xi.x, xj.y - xi.y, xj.z - xi.z};
  const double d2 = (dx[0] * dx[0] + dx[1] * dx[1]) + dx[2] * dx[2];
  const double rsum = xi.w + xj.w;
  const float d2f = (float)d2;
  const float inv_d = M::rsqrt(d2f);
  const float num = (float)(rsum * rsum - d2);
  float dn = num * M::rcp((float)rsum + d2f * inv_d);
  if (dn < 0.0f) dn = 0.0f;
  const float n[3] = {(float)dx[0] * inv_d, (float)dx[1] * inv_d, (float)dx[2] * inv_d};
  const float Ri = (float)xi.w, Rj = (float)xj.w;
  const float rw[3] = {Ri * (float)wi.x + Rj * (float)wj.x, Ri * (float)wi.y + Rj * (float)wj.y,
                       Ri * (float)wi.z + Rj * (float)wj.z};
  const float vroll[3] = {rw[1] * n[2] - rw[2] * n[1], rw[2] * n[0] - rw[0] * n[2],
                          rw[0] * n[1] - rw[1] * n[0]};
  const float vij[3] = {(float)(vi.x - vj.x) + vroll[0], (float)(vi.y - vj.y) + vroll[1],
                        (float)(vi.z - vj.z) + vroll[2]};
  const float wrel[3] = {(float)(wi.x - wj.x), (float)(wi.y - wj.y), (float)(wi.z - wj.z)};
  const float me = M::rcp((float)(vi.w + vj.w));
  const float Re = (Ri * Rj) * M::rcp(Ri + Rj);
  const float vr =
      rolling == 2 ? M::sqrt((vroll[0] * vroll[0] + vroll[1] * vroll[1]) + vroll[2] * vroll[2])
                   : 0.0f;
  hm_law<float>(c, rolling, model, dt, dn, n, vij, wrel, vr, me, Re, Ri, dtl, Fi, Mi);
}

// The law against wall W, a body of infinite mass and radius whose contact
// point moves with the wall's surface velocity: unit normal gn from the
// particle to the wall, overlap gdn, lever arm of the contact point about the
// wall's rotation axis.
template <typename R>
__device__ __forceinline__ void wall_law(const PairCoef& c, int rolling, int model, double dt,
                                         const WallDev& W, const double gn[3], double gdn,
                                         const double arm[3], double4 xi, double4 vi,
                                         double4 wi, double dtl[3], double Fi[3],
                                         double Mi[3]) {
  const double dn = gdn < 0.0 ? 0.0 : gdn;
  const double vw[3] = {W.vel[0] + (W.omega[1] * arm[2] - W.omega[2] * arm[1]),
                        W.vel[1] + (W.omega[2] * arm[0] - W.omega[0] * arm[2]),
                        W.vel[2] + (W.omega[0] * arm[1] - W.omega[1] * arm[0])};
  const double Ri = xi.w;
  const double rw[3] = {Ri * wi.x, Ri * wi.y, Ri * wi.z};
  const double vd[3] = {(vi.x - vw[0]) + (rw[1] * gn[2] - rw[2] * gn[1]),
                        (vi.y - vw[1]) + (rw[2] * gn[0] - rw[0] * gn[2]),
                        (vi.z - vw[2]) + (rw[0] * gn[1] - rw[1] * gn[0])};
  const double wd[3] = {wi.x - W.omega[0], wi.y - W.omega[1], wi.z - W.omega[2]};
  const R n[3] = {(R)gn[0], (R)gn[1], (R)gn[2]};
  const R vij[3] = {(R)vd[0], (R)vd[1], (R)vd[2]};
  const R wrel[3] = {(R)wd[0], (R)wd[1], (R)wd[2]};
  // rolling speed against a wall: |R_i (omega_i - Omega_wall) x n|
  R vr = (R)0;
  if (rolling == 2) {
    const R rr[3] = {(R)Ri * wrel[0], (R)Ri * wrel[1], (R)Ri * wrel[2]};
    const R vroll[3] = {rr[1] * n[2] - rr[2] * n[1], rr[2] * n[0] - rr[0] * n[2],
                        rr[0] * n[1] - rr[1] * n[0]};
    vr = Fast<R>::sqrt((vroll[0] * vroll[0] + vroll[1] * vroll[1]) + vroll[2] * vroll[2]);
  }
  const R me = Fast<R>::rcp((R)vi.w);
  hm_law<R>(c, rolling, model, dt, (R)dn, n, vij, wrel, vr, me, (R)Ri, (R)Ri, dtl, Fi, Mi);
}

// Particle against wall W at time t.
template <typename R>
__device__ __forceinline__ void pw_contact(const PairCoef& c, int rolling, int model, double dt,
                                           const WallDev& W, double skin, double t, double4 xi,
                                           double4 vi, double4 wi, double dtl[3],
                                           double Fi[3], double Mi[3]) {
  const double x[3] = {xi.x, xi.y, xi.z};
  WallGeo g;
  wall_geo(W, x, xi.w, skin, true, t, g);
  if (!g.touching) {
    dtl[0] = dtl[1] = dtl[2] = 0.0;
    Fi[0] = Fi[1] = Fi[2] = 0.0;
    Mi[0] = Mi[1] = Mi[2] = 0.0;
    return;
  }
  const double gn[3] = {g.n0, g.n1, g.n2}, arm[3] = {g.a0, g.a1, g.a2};
  wall_law<R>(c, rolling, model, dt, W, gn, g.dn, arm, xi, vi, wi, dtl, Fi, Mi);
}

// ------------------------------------------------------------------- force
//
// A particle's lane (or its two or four lanes, see below) walks its row in
// order, every load of a row entry one coalesced access for the wavefront; the
// neighbour's velocities and
// the pair history are loaded only when the pair touches.  Bit 31 of a row
// entry marks "touching at the last evaluation" (history may be non-zero);
// histories of other entries are zero and are neither read nor written.

constexpr int kTouchedBit = (int)0x80000000u;
constexpr int kIndexMask = 0x7fffffff;

// Value of v in the lane that a DPP pattern picks (0 where it picks none): two
// 32-bit moves, at the rate of the vector unit (a shuffle goes through LDS).
template <int CTRL>
__device__ __forceinline__ double dpp0(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Largest of a wavefront's non-negative values, in lane 63: row shifts by 1,
// 2, 4 and 8, then the last lane of each row to the next rows.
__device__ __forceinline__ double wave_max63(double v) {
  v = fmax(v, dpp0<0x111>(v));
  v = fmax(v, dpp0<0x112>(v));
  v = fmax(v, dpp0<0x114>(v));
  v = fmax(v, dpp0<0x118>(v));
  v = fmax(v, dpp0<0x142>(v));
  v = fmax(v, dpp0<0x143>(v));
  return v;
}

// Raises a drift record to the largest value of a wavefront, with one atomic
// per wavefront: non-negative doubles order like their bit patterns.  Every
// lane of the wavefront calls it.  Blocks go round the 8 XCDs, so a word's
// line is mostly raised from one XCD.
__device__ __forceinline__ void raise_drift(const StepParams& sp, unsigned long long* rec,
                                            double v) {
  v = wave_max63(v);
  const int w = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) & (sp.drift_words - 1);
  if ((threadIdx.x & 63) == 63 && v > 0.0)
    atomicMax(rec + w * kDriftStride, (unsigned long long)__double_as_longlong(v));
}

// Largest value of a drift record, the same in every lane: lane w reads word w
// (a single load; one scalar load per word took 2 us longer in a launch of
// few wavefronts, which nothing hides).
__device__ __forceinline__ double drift_of(const StepParams& sp, const unsigned long long* rec) {
  const int w = (threadIdx.x & 63) & (sp.drift_words - 1);
  const double v = wave_max63(__longlong_as_double((long long)rec[w * kDriftStride]));
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// How a force launch shares its work among the lanes and which of its accesses
// stream past the caches (non-temporal).  kLanes lanes work on one particle:
// lane g takes the row's entries g, g + kLanes, ... (several entries in flight
// where one lane would go through them one after the other), and the
// contributions are added in row order, so the sums are the same for every
// kLanes.  See force_way for where each is used.
struct WaySmall4 {
  static constexpr int kLanes = 4;
  static constexpr bool kRowNt = false, kHistLdNt = false, kHistStNt = false, kStateNt = false;
};
struct WaySmall2 {
  static constexpr int kLanes = 2;
  static constexpr bool kRowNt = false, kHistLdNt = false, kHistStNt = false, kStateNt = false;
};
struct WayCached {
  static constexpr int kLanes = 1;
  static constexpr bool kRowNt = false, kHistLdNt = false, kHistStNt = false, kStateNt = false;
};
struct WayMid {
  static constexpr int kLanes = 1;
  static constexpr bool kRowNt = false, kHistLdNt = true, kHistStNt = true, kStateNt = false;
};
struct WayLarge {
  static constexpr int kLanes = 1;
  static constexpr bool kRowNt = true, kHistLdNt = false, kHistStNt = true, kStateNt = true;
};

template <bool NT, typename T>
__device__ __forceinline__ T ld_own(const T* p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void st_own(T v, T* p) {
  if (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}
typedef double own_d4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ void st_own(const double4& v, double4* p) {
  if (NT) {
    const own_d4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<own_d4*>(p));
  } else {
    *p = v;
  }
}

// acc[c] += the values v[c] of the G lanes of a particle, lane by lane: lane g
// of the particle is lane g (64 / G) + its place in the wavefront, so whole
// rows of 16 lanes are handed round.  All lanes of the particle get the same
// sums.
template <int G>
__device__ __forceinline__ void add_in_order(double* acc, const double* v, int n);

__device__ __forceinline__ void swap32(double v, double& x, double& y) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false,
                                                  false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false,
                                                  false);
  x = __hiloint2double((int)h[0], (int)l[0]);
  y = __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ void swap16(double v, double& x, double& y) {
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false,
                                                  false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false,
                                                  false);
  x = __hiloint2double((int)h[0], (int)l[0]);
  y = __hiloint2double((int)h[1], (int)l[1]);
}
template <>
__device__ __forceinline__ void add_in_order<1>(double* acc, const double* v, int n) {
#pragma unroll
  for (int c = 0; c < n; ++c) acc[c] += v[c];
}
template <>
__device__ __forceinline__ void add_in_order<2>(double* acc, const double* v, int n) {
#pragma unroll
  for (int c = 0; c < n; ++c) {
    double a, b;
    swap32(v[c], a, b);
    acc[c] = (acc[c] + a) + b;
  }
}
template <>
__device__ __forceinline__ void add_in_order<4>(double* acc, const double* v, int n) {
#pragma unroll
  for (int c = 0; c < n; ++c) {
    double a, b, q[4];
    swap32(v[c], a, b);
    swap16(a, q[0], q[1]);
    swap16(b, q[2], q[3]);
    acc[c] = (((acc[c] + q[0]) + q[1]) + q[2]) + q[3];
  }
}
// The states of the consecutive sorted particles of a force block, staged in
// LDS: in spatial (Morton) order most neighbours of a block's particles lie
// inside the block, and they are then read from LDS instead of through the
// cache hierarchy.  One record of position, velocity and spin per particle,
// the info words behind the records.
template <int G>
struct Tile {
  double4* rec;
  int* in;
  int lo, cnt;  // staged particles [lo, lo + cnt)

  // the lanes of a particle share the loads of its record, all of them in
  // flight before the first is waited for
  __device__ __forceinline__ void stage(const ParticleBufs& src, const int* __restrict__ info,
                                        int t, int g) {
    if (t >= cnt) return;
    const int inf = info[lo + t];
    if (G == 1) {
      const double4 p = src.pos[lo + t], v = src.vel[lo + t], w = src.omg[lo + t];
      rec[3 * t] = p;
      rec[3 * t + 1] = v;
      rec[3 * t + 2] = w;
    } else {
      const int c = G == 2 ? g : (g < 2 ? g : 2);
      const double4* __restrict__ from = c == 0 ? src.pos : (c == 1 ? src.vel : src.omg);
      const double4 a = from[lo + t];
      if (G == 2 && g == 0) rec[3 * t + 2] = src.omg[lo + t];
      rec[3 * t + c] = a;
    }
    if (g == 0) in[t] = inf;
  }
  __device__ __forceinline__ bool has(int j) const { return (unsigned)(j - lo) < (unsigned)cnt; }
  __device__ __forceinline__ double4 pos(const ParticleBufs& g, int j) const {
    return has(j) ? rec[3 * (j - lo)] : g.pos[j];
  }
  __device__ __forceinline__ double4 vel(const ParticleBufs& g, int j) const {
    return has(j) ? rec[3 * (j - lo) + 1] : g.vel[j];
  }
  __device__ __forceinline__ double4 omg(const ParticleBufs& g, int j) const {
    return has(j) ? rec[3 * (j - lo) + 2] : g.omg[j];
  }
  __device__ __forceinline__ int info(const int* __restrict__ g, int j) const {
    return has(j) ? in[j - lo] : g[j];
  }
};

// The states of a context that one workgroup holds as a whole (k_force_steps).
struct TileAll {
  double4* rec;
  int* in;
  static constexpr int lo = 0;
  __device__ __forceinline__ double4 pos(const ParticleBufs&, int j) const { return rec[3 * j]; }
  __device__ __forceinline__ double4 vel(const ParticleBufs&, int j) const { return rec[3 * j + 1]; }
  __device__ __forceinline__ double4 omg(const ParticleBufs&, int j) const { return rec[3 * j + 2]; }
  __device__ __forceinline__ int info(const int* __restrict__, int j) const { return in[j]; }
};

// Where the updated state of particle i goes: the context's other buffers, or
// a workgroup's records.
template <bool NT>
struct ToBufs {
  ParticleBufs b;
  __device__ __forceinline__ void pos(int i, const double4& v) const { st_own<NT>(v, b.pos + i); }
  __device__ __forceinline__ void vel(int i, const double4& v) const { st_own<NT>(v, b.vel + i); }
  __device__ __forceinline__ void omg(int i, const double4& v) const { st_own<NT>(v, b.omg + i); }
};
struct ToRecords {
  double4* rec;
  __device__ __forceinline__ void pos(int i, const double4& v) const { rec[3 * i] = v; }
  __device__ __forceinline__ void vel(int i, const double4& v) const { rec[3 * i + 1] = v; }
  __device__ __forceinline__ void omg(int i, const double4& v) const { rec[3 * i + 2] = v; }
};

// Square of a step's drift |v| dt in units of half the skin: scale = dt * 2 /
// skin.  Maxima of squares are taken on the device, the root on the host.
__device__ __forceinline__ double drift2(const double4& v, double scale) {
  const double s2 = scale * scale;
  return ((v.x * v.x + v.y * v.y) + v.z * v.z) * s2;
}

// dt * 2 / skin of the particle's instance (uniform when all skins agree)
__device__ __forceinline__ double drift_scale(const StepParams& sp,
                                              const InstDev* __restrict__ inst, int inf) {
  return sp.drift_scale > 0.0 ? sp.drift_scale : sp.dt * inst[inf >> kInstShift].ihs;
}

// Forces on particle i and its integration; returns the squared drift of
// this step in units of half the instance's skin (for the dynamic search
// trigger) when asked for it.
template <typename R, int MODE, int MODEL, typename WAY, bool REC, int PAIRS, typename TileT,
          typename OutT>
__device__ __forceinline__ double force_particle(
    const int i, const int g, const StepParams& sp, const InstDev* __restrict__ inst,
    const PairCoef* __restrict__ ppc, const PairCoef* __restrict__ pwc,
    const WallDev* __restrict__ walls, ParticleBufs in, const OutT& out,
    const int* __restrict__ info, NbrList l, WallSlots ws, double4* __restrict__ Fo,
    double4* __restrict__ To, const int64_t* __restrict__ clock, int64_t step_rel,
    const int* __restrict__ flags, const bool want_drift, const int* __restrict__ xsel,
    const double4* __restrict__ Fx, const double4* __restrict__ Tx, const TileT& tile,
    const int len, const int jr0, double* __restrict__ pf) {
  constexpr int G = WAY::kLanes;
  const int n = sp.n;
  // the particle's own velocity and spin stay in the LDS tile during the row
  // walk and are read where they are used (registers for the neighbour's)
  const int own = 3 * (i - tile.lo);
  double4 xi = tile.rec[own];
  const int inf = tile.in[i - tile.lo];
  // frozen after an error, and for inactive particles: carry the state over
  if ((inf & kInactive) || *flags != 0) {
    if (g != 0) return 0.0;
    out.pos(i, xi);
    out.vel(i, tile.rec[own + 1]);
    out.omg(i, tile.rec[own + 2]);
    if (MODE != 0) {
      Fo[i] = make_double4(0.0, 0.0, 0.0, 0.0);
      To[i] = make_double4(0.0, 0.0, 0.0, 0.0);
    }
    return 0.0;
  }
  // material-pair row of (instance, type i): instance b's table starts at
  // b * kMaxTypes^2, so it follows from the info word without a lookup
  const int ti = inf & kTypeMask;
  const int row = ((inf >> kInstShift) * kMaxTypes + ti) * kMaxTypes;
  const PairCoef* __restrict__ ppi = ppc + row;
  const PairCoef* __restrict__ pwi = pwc + row;
  // PAIRS 1: a single instance whose particles all have type 0, so every
  // pair takes the table's first entry, read once for the wavefront;
  // PAIRS 2: every particle has type 0, so the pair's entry is the first of
  // the particle's own row (its load does not wait for the neighbour's
  // type), read once for the wavefront when all its lanes share the row
  PairCoef pc0;
  if (PAIRS == 1) pc0 = ppc[0];
  bool uni = false;  // PAIRS 2: the wavefront's lanes share one row
  if (PAIRS == 2) {
    const int rowu = __builtin_amdgcn_readfirstlane(row);
    uni = __builtin_amdgcn_ballot_w64(row != rowu) == 0ull;
    if (uni) pc0 = ppc[rowu];
  }
  const double dt = sp.dt;
  double FT[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // force and torque
  const int max_nb = sp.max_nb;
  const int64_t cap = l.cap;
  // the lane's first wall slot is loaded ahead of the row walk where there are
  // registers for it
  int w_next = -1;
  if (G > 1) w_next = ws.wid[(int64_t)g * n + i];
  // the index of the lane's next entry is loaded while its entry k is worked
  // on (the row walk is a chain of dependent loads; one index ahead costs one
  // VGPR); the row length and the lane's first entry come from the caller
  int jr_next = jr0;
  for (int k0 = 0; k0 < len; k0 += G) {
    const int k = k0 + g;
    const int64_t e = nbr_entry(i, k, max_nb);
    bool touch = false;
    double C[6];  // this lane's contact: force and torque
    if (G > 1) C[0] = C[1] = C[2] = C[3] = C[4] = C[5] = 0.0;
    if (G == 1 || k < len) {
      const int jr = jr_next;
      if (k + G < len) jr_next = ld_own<WAY::kRowNt>(l.nbr + e + 64 * G);  // entry (i, k + G)
      const int j = jr & kIndexMask;
      // a pair touching at the last evaluation most likely still touches: its
      // history is loaded together with the neighbour's position
      double dtl[3] = {0.0, 0.0, 0.0};
      if (jr & kTouchedBit) {
        dtl[0] = ld_own<WAY::kHistLdNt>(l.hist + e);
        dtl[1] = ld_own<WAY::kHistLdNt>(l.hist + cap + e);
        dtl[2] = ld_own<WAY::kHistLdNt>(l.hist + 2 * cap + e);
      }
      const double4 xj = tile.pos(in, j);
      const double dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const double rsum = xi.w + xj.w;
      touch = d2 < rsum * rsum;
      if (touch) {
        const double4 vj = tile.vel(in, j);
        const double4 wj = tile.omg(in, j);
        int oi = own;
        asm volatile("" : "+v"(oi));  // keeps the LDS reads inside the loop
        const double4 vi = tile.rec[oi + 1];
        const double4 wi = tile.rec[oi + 2];
        if (PAIRS == 1) {
          pp_contact<R>(pc0, sp.rolling, MODEL, dt, xi, vi, wi, xj, vj, wj, dtl, C, C + 3);
        } else if (PAIRS == 2) {
          if (uni)
            pp_contact<R>(pc0, sp.rolling, MODEL, dt, xi, vi, wi, xj, vj, wj, dtl, C, C + 3);
          else
            pp_contact<R>(ppi[0], sp.rolling, MODEL, dt, xi, vi, wi, xj, vj, wj, dtl, C, C + 3);
        } else {
          const int tj = tile.info(info, j) & kTypeMask;
          pp_contact<R>(ppi[tj], sp.rolling, MODEL, dt, xi, vi, wi, xj, vj, wj, dtl, C, C + 3);
        }
        st_own<WAY::kHistStNt>(dtl[0], l.hist + e);
        st_own<WAY::kHistStNt>(dtl[1], l.hist + cap + e);
        st_own<WAY::kHistStNt>(dtl[2], l.hist + 2 * cap + e);
        if (!(jr & kTouchedBit)) st_own<WAY::kHistStNt>(j | kTouchedBit, l.nbr + e);
        if (REC) {
          pf[e] = C[0];
          pf[cap + e] = C[1];
          pf[2 * cap + e] = C[2];
        }
        if (G == 1) add_in_order<1>(FT, C, 6);
      } else if (jr & kTouchedBit) {
        st_own<WAY::kHistStNt>(0.0, l.hist + e);
        st_own<WAY::kHistStNt>(0.0, l.hist + cap + e);
        st_own<WAY::kHistStNt>(0.0, l.hist + 2 * cap + e);
        st_own<WAY::kHistStNt>(j, l.nbr + e);
      }
    }
    // adding the zeros of lanes without a contact changes no sum (one that
    // starts at +0 never becomes -0)
    if (G > 1 && __builtin_amdgcn_ballot_w64(touch) != 0ull) add_in_order<G>(FT, C, 6);
  }
  double4 vi = tile.rec[own + 1];
  double4 wi = tile.rec[own + 2];
  // walls: time of this force evaluation; lane g takes the slots g, g + G, ...
  const double t = (double)(*clock + step_rel) * dt;
#pragma unroll 1
  for (int s0 = 0; s0 < kWallSlots; s0 += G) {
    const int s = s0 + g;
    const int w = G > 1 && s0 == 0 ? w_next : ws.wid[(int64_t)s * n + i];
    if (G == 1 ? w < 0 : __builtin_amdgcn_ballot_w64(w >= 0) == 0ull) break;
    double C[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (w >= 0) {
      const WallDev& W = walls[w];
      double dtl[3] = {ws.hist[(int64_t)(3 * s) * n + i], ws.hist[(int64_t)(3 * s + 1) * n + i],
                       ws.hist[(int64_t)(3 * s + 2) * n + i]};
      if (t >= W.t_on && t < W.t_off)
        pw_contact<R>(pwi[W.material], sp.rolling, MODEL, dt, W, W.skin, t, xi, vi, wi, dtl, C,
                      C + 3);
      else
        dtl[0] = dtl[1] = dtl[2] = 0.0;
      st_own<WAY::kHistStNt>(dtl[0], ws.hist + (int64_t)(3 * s) * n + i);
      st_own<WAY::kHistStNt>(dtl[1], ws.hist + (int64_t)(3 * s + 1) * n + i);
      st_own<WAY::kHistStNt>(dtl[2], ws.hist + (int64_t)(3 * s + 2) * n + i);
    }
    add_in_order<G>(FT, C, 6);
  }
  double* F = FT;
  double* T = FT + 3;
  if (xsel && xsel[i] >= 0) {
    const double4 fx = Fx[i], tx = Tx[i];
    F[0] += fx.x;
    F[1] += fx.y;
    F[2] += fx.z;
    T[0] += tx.x;
    T[1] += tx.y;
    T[2] += tx.z;
  }
  // integration of particle i (vel.w = 1/m, omg.w = 1/I)
  const double im = vi.w, iI = wi.w;
  const double a[3] = {F[0] * im + sp.g[0], F[1] * im + sp.g[1], F[2] * im + sp.g[2]};
  const double al[3] = {T[0] * iI, T[1] * iI, T[2] * iI};
  double drift = 0.0;
  if (MODE == 2) {
    // explicit Euler, Eq. (integ_EE): x with the old velocity
    if (want_drift) drift = drift2(vi, drift_scale(sp, inst, inf));
    xi.x = xi.x + vi.x * dt;
    xi.y = xi.y + vi.y * dt;
    xi.z = xi.z + vi.z * dt;
    vi.x = vi.x + a[0] * dt;
    vi.y = vi.y + a[1] * dt;
    vi.z = vi.z + a[2] * dt;
    wi.x = wi.x + al[0] * dt;
    wi.y = wi.y + al[1] * dt;
    wi.z = wi.z + al[2] * dt;
  } else {
    const double h = sp.hdt;
    // second half kick of this step, Eq. (newvv)
    vi.x = vi.x + a[0] * h;
    vi.y = vi.y + a[1] * h;
    vi.z = vi.z + a[2] * h;
    wi.x = wi.x + al[0] * h;
    wi.y = wi.y + al[1] * h;
    wi.z = wi.z + al[2] * h;
    if (MODE == 0) {
      // first half kick and drift of the next step, Eq. (halfstep)
      vi.x = vi.x + a[0] * h;
      vi.y = vi.y + a[1] * h;
      vi.z = vi.z + a[2] * h;
      wi.x = wi.x + al[0] * h;
      wi.y = wi.y + al[1] * h;
      wi.z = wi.z + al[2] * h;
      xi.x = xi.x + vi.x * dt;
      xi.y = xi.y + vi.y * dt;
      xi.z = xi.z + vi.z * dt;
      if (want_drift) drift = drift2(vi, drift_scale(sp, inst, inf));
    }
  }
  if (g == 0) out.pos(i, xi);
  if (g == 1 % G) out.vel(i, vi);
  if (g == 2 % G) out.omg(i, wi);
  if (MODE != 0 && g == 3 % G) {
    Fo[i] = make_double4(F[0], F[1], F[2], 0.0);
    To[i] = make_double4(T[0], T[1], T[2], 0.0);
  }
  return drift;
}

// The row cut that a displacement bound of acc half skins allows, the same in
// every lane (a relative margin of 1e-6 covers every rounding of the bound and
// of the gaps), and the row length that it leaves.
__device__ __forceinline__ int row_cut(double acc) {
  const double accm = acc * (1.0 + 1e-6);
  const int u = accm < kCutFrac[0] ? 0 : (accm < kCutFrac[1] ? 1 : (accm < kCutFrac[2] ? 2 : 3));
  return __builtin_amdgcn_readfirstlane(u);
}
__device__ __forceinline__ int cut_row(int len, int cut, int u_cut) {
  if (u_cut < 3) {
    const int c = (cut >> (kCutBits * u_cut)) & kCutMask;
    if (c != kCutMask && c < len) return c;
  }
  return len;
}

// Occupancy floor: four wavefronts per SIMD (128 VGPRs, no spills), except
// for the linear law with explicit Euler, which would spill there and keeps
// three.
// REC: also write every touching pair's force to pf (the per-contact record;
// a separate instantiation, so the record costs the plain kernel nothing).
// PAIRS: how a pair finds its material-pair constants (see force_particle).
template <typename R, int MODE, int MODEL, typename WAY, bool REC, int PAIRS>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(MODE == 2 && MODEL == 1 ? 3 : 4)))
k_force(StepParams sp, const InstDev* __restrict__ inst, const PairCoef* __restrict__ ppc,
        const PairCoef* __restrict__ pwc, const WallDev* __restrict__ walls, ParticleBufs in,
        ParticleBufs out, const int* __restrict__ info, NbrList l, WallSlots ws,
        double4* __restrict__ Fo, double4* __restrict__ To, const int64_t* __restrict__ clock,
        int64_t step_rel, const int* __restrict__ flags, const int* __restrict__ xsel,
        const double4* __restrict__ Fx, const double4* __restrict__ Tx, double* __restrict__ pf) {
  // lanes g of a particle: 64 / G lanes apart in the wavefront (see add_in_order)
  constexpr int G = WAY::kLanes, kPerWave = 64 / G;
  const int nb = blockDim.x / G;  // particles of the block
  const int b0 = xcd_block() * nb;
  const int g = G == 1 ? 0 : (threadIdx.x & 63) / kPerWave;
  const int il = G == 1 ? threadIdx.x
                        : (threadIdx.x >> 6) * kPerWave + (threadIdx.x & (kPerWave - 1));
  const int i = b0 + il;
  const int64_t step = *clock + step_rel;  // these positions are x^step
  // the row length, its cuts and the first row entries do not depend on the
  // tile: their loads are issued before it is staged (the first max_nb entries
  // exist for every row)
  int len = 0, cut = 0, jr0 = 0;
  if (i < sp.n) {
    len = ld_own<WAY::kRowNt>(l.rowlen + i);
    cut = ld_own<WAY::kRowNt>(l.rowcut + i);
    if (g < sp.max_nb) jr0 = ld_own<WAY::kRowNt>(l.nbr + nbr_entry(i, g, sp.max_nb));
  }
  // displacement bound of x^step since the last search (half skins): the
  // previous evaluation's bound plus the largest drift of the update since;
  // then the row cut it allows
  int u_cut;
  {
    const double m = sqrt(drift_of(sp, sp.brec + bound_slot(step, 0) * kDriftRec));
    const double acc = sp.bacc[bound_slot(step, -1)] + m;
    if (blockIdx.x == 0 && threadIdx.x < kDriftSpread) {
      sp.brec[bound_slot(step, 2) * kDriftRec + threadIdx.x * kDriftStride] = 0ull;
      if (threadIdx.x == 0) {
        sp.bacc[bound_slot(step, 0)] = acc;
        sp.blog[step & (kDriftLog - 1)] = m;
      }
    }
    u_cut = row_cut(acc);
  }
  len = cut_row(len, cut, u_cut);
  extern __shared__ double4 force_lds[];
  Tile<G> tile;
  tile.rec = force_lds;
  tile.in = reinterpret_cast<int*>(force_lds + 3 * nb);
  tile.lo = b0;
  tile.cnt = sp.n - b0 < nb ? sp.n - b0 : nb;
  tile.stage(in, info, il, g);
  __syncthreads();
  double d = 0.0;
  if (i < sp.n)
    d = force_particle<R, MODE, MODEL, WAY, REC, PAIRS>(
        i, g, sp, inst, ppc, pwc, walls, in, ToBufs<WAY::kStateNt>{out}, info, l, ws, Fo, To, clock,
        step_rel, flags, MODE != 1, xsel, Fx, Tx, tile, len, jr0, pf);
  // this launch's own update produced x^(step + 1)
  if (MODE != 1) raise_drift(sp, sp.brec + bound_slot(step, 1) * kDriftRec, d);
}

// `steps` steps of a context of at most kStepsMax particles in one workgroup:
// the updated states stay in LDS, in two copies that take turns, and the drift
// of a step is reduced there, so that a barrier stands where the end of one
// launch and the start of the next were.  Row entries and histories stay in
// their buffers (a lane reads back only what it wrote).  What is left is one
// particle's chain of loads and arithmetic: 2.7 us per step for 20 spheres,
// where a launch took 4.2 and 1.1 passed between two.  Registers for the two
// wavefronts per SIMD of the largest context.
template <typename R, int MODE, int MODEL, int PAIRS>
__global__ void __launch_bounds__(4 * kStepsMax) __attribute__((amdgpu_waves_per_eu(2)))
k_force_steps(StepParams sp, const InstDev* __restrict__ inst, const PairCoef* __restrict__ ppc,
              const PairCoef* __restrict__ pwc, const WallDev* __restrict__ walls,
              ParticleBufs in, ParticleBufs out, const int* __restrict__ info, NbrList l,
              WallSlots ws, double4* __restrict__ Fo, double4* __restrict__ To,
              const int64_t* __restrict__ clock, int64_t step_rel, int steps,
              const int* __restrict__ flags) {
  typedef WaySmall4 WAY;
  constexpr int G = WAY::kLanes, kPerWave = 64 / G;
  __shared__ double wave_drift[2][4 * kStepsMax / 64];
  extern __shared__ double4 force_lds[];
  const int nb = blockDim.x / G, waves = blockDim.x >> 6, wave = threadIdx.x >> 6;
  const int g = (threadIdx.x & 63) / kPerWave;
  const int i = wave * kPerWave + (threadIdx.x & (kPerWave - 1));
  const int n = sp.n;
  const int64_t step0 = *clock + step_rel;
  int len_all = 0, cut = 0;
  if (i < n) {
    len_all = l.rowlen[i];
    cut = l.rowcut[i];
  }
  double m = sqrt(drift_of(sp, sp.brec + bound_slot(step0, 0) * kDriftRec));
  double acc = sp.bacc[bound_slot(step0, -1)];
  Tile<G> first;
  first.rec = force_lds;
  first.in = reinterpret_cast<int*>(force_lds + 6 * nb);
  first.lo = 0;
  first.cnt = n;
  first.stage(in, info, i, g);
  __syncthreads();
  double largest = 0.0;
#pragma unroll 1
  for (int s = 0; s < steps; ++s) {
    // as k_force does at the start of its launch
    acc = acc + m;
    if (threadIdx.x == 0) sp.blog[(step0 + s) & (kDriftLog - 1)] = m;
    const int len = cut_row(len_all, cut, row_cut(acc));
    TileAll tile;
    tile.rec = force_lds + (s & 1) * 3 * nb;
    tile.in = first.in;
    double d = 0.0;
    if (i < n) {
      int jr0 = 0;
      if (g < sp.max_nb) jr0 = l.nbr[nbr_entry(i, g, sp.max_nb)];
      d = force_particle<R, MODE, MODEL, WAY, false, PAIRS>(
          i, g, sp, inst, ppc, pwc, walls, in, ToRecords{force_lds + (~s & 1) * 3 * nb}, info, l,
          ws, Fo, To, clock, step_rel + s, flags, true, nullptr, nullptr, nullptr, tile, len, jr0,
          nullptr);
    }
    d = wave_max63(d);
    if ((threadIdx.x & 63) == 63) wave_drift[s & 1][wave] = d > 0.0 ? d : 0.0;
    __syncthreads();
    largest = 0.0;
    for (int w = 0; w < waves; ++w) largest = fmax(largest, wave_drift[s & 1][w]);
    m = sqrt(largest);
  }
  // the state, and the displacement bound as the last of `steps` launches
  // leaves it
  if (i < n && g < 3) {
    double4* to = g == 0 ? out.pos : (g == 1 ? out.vel : out.omg);
    to[i] = force_lds[(steps & 1) * 3 * nb + 3 * i + g];
  }
  const int64_t last = step0 + steps - 1;
  if (threadIdx.x < kDriftSpread) {
    sp.brec[bound_slot(last, 1) * kDriftRec + threadIdx.x * kDriftStride] =
        threadIdx.x == 0 ? (unsigned long long)__double_as_longlong(largest) : 0ull;
    sp.brec[bound_slot(last, 2) * kDriftRec + threadIdx.x * kDriftStride] = 0ull;
    if (threadIdx.x == 0) sp.bacc[bound_slot(last, 0)] = acc;
  }
}

// Which way a force launch of n particles takes (us per step with an FP64 law,
// settling beds of 1.8 touching pairs per sphere, one MI355X).
//
// Lanes per particle.  One lane per particle fills the chip's wavefront slots
// (256 compute units x 16 at the kernel's registers) from 262,144 particles
// on; below, the time is that of one particle's chain of dependent loads and
// arithmetic, which more lanes shorten.  4 / 2 / 1 lanes: 1,000 spheres 13.6 /
// 16.0 / 19.4; 8,000 12.5 / 15.0 / 20.2; 30,000 14.5 / 15.5 / 20.1; 50,000
// 17.7 / 18.1 / 19.4; 60,000 in a silo 20.6 / 21.3 / 23.5; 100,000 28.0 / 23.9
// / 25.0; 130,000 - / 27.2 / 27.5; 200,000 - / 44.6 / 41.8.  8 lanes were
// never the best.  The lines hold for the FP32 law too: dense beds that rest,
// FP32 (FP64), 30,000 10.8 / 11.5 / 13.1 (11.2 / 11.8 / 13.9); 50,000 13.9 / 13.7 /
// 15.4 (14.8 / 14.5 / 16.0); 100,000 20.5 / 16.8 / 18.6 (21.6 / 18.2 / 20.2);
// 130,000 25.4 / 23.4 / 21.4 (27.1 / 24.6 / 24.1).
//
// Streaming.  A step touches about 400 bytes per particle (two copies of the
// state, histories, row entries), and the memory-side cache holds 256 MB.
// While all of it fits, nothing streams (WayCached); then the histories stream
// past the state, which keeps fitting (WayMid); and when that does not fit
// either, the histories are the ones to stay between their load and their
// store (WayLarge).  Cached / mid / large: 200,000 41.8 / 46.5 / -; 300,000
// 46.1 / 54.3 / 56.4; 600,000 91.3 / 91.4 / -; 700,000 108.6 / 99.5 / 105.6;
// 1,000,000 149.6 / 137.8 / 145.1; 1,250,000 - / 176.7 / 175.1; 1,400,000 211 /
// 208 / 206; 2,000,000 286 / 293 / 276; 4,300,000 in a silo 748 / 770 / 727.
// (Before, every launch streamed loads and stores alike: 200,000 47.1, 1,000,000
// 147.0, 4,300,000 768.)  Beds that rest, FP32 (FP64): 500,000 60.3 / 63.5 / 69.7
// (62.3 / 66.1 / 71.7); 600,000 82.1 / 79.9 / 85.4 (83.8 / 81.5 / 86.8); 1,000,000
// 140.9 / 124.6 / 135.5 (142.8 / 129.0 / 137.6); 1,400,000 199.6 / 187.9 / 194.2
// (201.1 / 190.2 / 197.1); 2,000,000 273.3 / 262.3 / 266.7 (276.3 / 265.5 / 269.6).
// The upper line is that of beds that move; resting ones would stay with WayMid
// for 1.5 to 3 % up to 2,000,000.
//
// Threads per workgroup, when the caller leaves it open.  Up to 262,144
// particles every workgroup is in flight at once, and the compute unit that got
// the most of them ends last: 200,000 particles are 784 workgroups of 256, four
// for some of the 256 units and three for most, and 3,128 of 64, 13 and 12.
// Above, larger workgroups find more of their neighbours in their own records.
// 256 / 128 / 64 threads, us per step with its share of the search: 1,000
// spheres 11.1 / 10.8 / 10.1; 8,000 12.5 / 12.0 / 12.1; 60,000 18.1 / 17.9 /
// 17.9; 100,000 21.7 / 22.1 / 21.4; 200,000 in a silo 38.7 / 38.4 / 37.2, in a
// mesh 43.0 / 42.5 / 41.8; 400,000 53.6 / 52.6 / 53.3; 1,000,000 139.1 / 140.0
// / 143.4; 4,300,000 742 / 774 / 827.
constexpr int64_t kSmallBlocks = 262144;
constexpr int64_t kAllCached = 600000, kStateCached = 1200000;

enum { kWaySmall4, kWaySmall2, kWayCached, kWayMid, kWayLarge };

static int force_way(int64_t n) {
  if (force_lanes(n) > 1) return force_lanes(n) == 4 ? kWaySmall4 : kWaySmall2;
  if (n <= kAllCached) return kWayCached;
  return n <= kStateCached ? kWayMid : kWayLarge;
}

hipError_t launch_force(int mode, int precision, const StepParams& sp, const InstDev* inst,
                        const PairCoef* pp,
                        const PairCoef* pw, const WallDev* walls, ParticleBufs in,
                        ParticleBufs out, const int* info, NbrList l, WallSlots ws,
                        double4* F, double4* T, const int64_t* clock, int64_t step_rel,
                        const int* flags, const int* xsel, const double4* Fx, const double4* Tx,
                        double* pf, int block, int pair_mode, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  if (block == 0) block = sp.n <= kSmallBlocks ? 64 : kBlock;
  if (block != 64 && block != 128 && block != 256) return hipErrorInvalidValue;
  const int way = pf ? kWayMid : force_way(sp.n);  // the record has one instantiation
  const int per_block = way == kWaySmall4 ? block / 4 : (way == kWaySmall2 ? block / 2 : block);
  const dim3 gr(grid_for(sp.n, per_block)), bl(block);
  const size_t lds = (size_t)per_block * (3 * sizeof(double4) + sizeof(int));
#define DEM_LAUNCH_WAY(RT, M, L, WAY, REC, PAIRS)                                                 \
  hipLaunchKernelGGL((k_force<RT, M, L, WAY, REC, PAIRS>), gr, bl, lds, s, sp, inst, pp, pw,      \
                     walls, in, out, info, l, ws, F, T, clock, step_rel, flags, xsel, Fx, Tx, pf)
#define DEM_LAUNCH_PAIRS(RT, M, L, PAIRS)                                            \
  do {                                                                               \
    if (way == kWaySmall4) DEM_LAUNCH_WAY(RT, M, L, WaySmall4, false, PAIRS);        \
    else if (way == kWaySmall2) DEM_LAUNCH_WAY(RT, M, L, WaySmall2, false, PAIRS);   \
    else if (way == kWayCached) DEM_LAUNCH_WAY(RT, M, L, WayCached, false, PAIRS);   \
    else if (way == kWayMid) DEM_LAUNCH_WAY(RT, M, L, WayMid, false, PAIRS);         \
    else DEM_LAUNCH_WAY(RT, M, L, WayLarge, false, PAIRS);                           \
  } while (0)
#define DEM_LAUNCH(RT, M, L)                                 \
  do {                                                       \
    if (pf) DEM_LAUNCH_WAY(RT, M, L, WayMid, true, 0);       \
    else if (pair_mode == 1) DEM_LAUNCH_PAIRS(RT, M, L, 1);  \
    else if (pair_mode == 2) DEM_LAUNCH_PAIRS(RT, M, L, 2);  \
    else DEM_LAUNCH_PAIRS(RT, M, L, 0);                      \
  } while (0)
#define DEM_LAUNCH_MODE(RT, L)                \
  do {                                        \
    if (mode == 0) DEM_LAUNCH(RT, 0, L);      \
    else if (mode == 1) DEM_LAUNCH(RT, 1, L); \
    else DEM_LAUNCH(RT, 2, L);                \
  } while (0)
  if (precision == 0) {
    if (sp.model == 0) DEM_LAUNCH_MODE(double, 0);
    else DEM_LAUNCH_MODE(double, 1);
  } else {
    if (sp.model == 0) DEM_LAUNCH_MODE(float, 0);
    else DEM_LAUNCH_MODE(float, 1);
  }
#undef DEM_LAUNCH_MODE
#undef DEM_LAUNCH
#undef DEM_LAUNCH_PAIRS
#undef DEM_LAUNCH_WAY
  return hipGetLastError();
}

// Steps of contexts up to kStepsMax particles.  One compute unit does all the
// work then, so the time grows with the particles, while a launch per step
// spreads them; us per step, searches included, several steps in a launch / one
// (an FP64 law, one MI355X): 20 spheres 4.3 / 6.3, 60 in a box 5.2 / 7.3, 128
// 6.5 / 8.3, 250 10.0 / 10.0.
hipError_t launch_force_steps(int mode, int precision, const StepParams& sp, const InstDev* inst,
                              const PairCoef* pp, const PairCoef* pw, const WallDev* walls,
                              ParticleBufs in, ParticleBufs out, const int* info, NbrList l,
                              WallSlots ws, double4* F, double4* T, const int64_t* clock,
                              int64_t step_rel, int steps, const int* flags, int pair_mode,
                              hipStream_t s) {
  if (sp.n <= 0 || steps <= 0) return hipSuccess;
  if (sp.n > kStepsMax || (mode != 0 && mode != 2)) return hipErrorInvalidValue;
  const int nb = (sp.n + 15) / 16 * 16;  // whole wavefronts of 16 particles
  const size_t lds = (size_t)nb * (6 * sizeof(double4) + sizeof(int));
#define DEM_LAUNCH_PAIRS(RT, M, L, PAIRS)                                                         \
  hipLaunchKernelGGL((k_force_steps<RT, M, L, PAIRS>), dim3(1), dim3(4 * nb), lds, s, sp, inst,   \
                     pp, pw, walls, in, out, info, l, ws, F, T, clock, step_rel, steps, flags)
#define DEM_LAUNCH(RT, M, L)                             \
  do {                                                   \
    if (pair_mode == 1) DEM_LAUNCH_PAIRS(RT, M, L, 1);   \
    else if (pair_mode == 2) DEM_LAUNCH_PAIRS(RT, M, L, 2); \
    else DEM_LAUNCH_PAIRS(RT, M, L, 0);                  \
  } while (0)
#define DEM_LAUNCH_MODE(RT, L)           \
  do {                                   \
    if (mode == 0) DEM_LAUNCH(RT, 0, L); \
    else DEM_LAUNCH(RT, 2, L);           \
  } while (0)
  if (precision == 0) {
    if (sp.model == 0) DEM_LAUNCH_MODE(double, 0);
    else DEM_LAUNCH_MODE(double, 1);
  } else {
    if (sp.model == 0) DEM_LAUNCH_MODE(float, 0);
    else DEM_LAUNCH_MODE(float, 1);
  }
#undef DEM_LAUNCH_MODE
#undef DEM_LAUNCH
#undef DEM_LAUNCH_PAIRS
  return hipGetLastError();
}

// ------------------------------------------------------------ mesh contacts
//
// Eight lanes per particle, one for each of its triangle candidates, over the
// list of the particles that have any (in a drum of 200,000 a tenth of them:
// one thread per particle of the context, going through the candidates one
// after the other with a wavefront waiting for its few busy lanes, took 29.7
// us instead of 8.7).
//
// Every candidate reports its closest point and feature.  A face touches
// when the centre is less than R above its plane.  The distance restricted
// to one triangle is convex, so a point on an edge or at a vertex is a local
// minimum of the distance over the surface exactly when every triangle
// around it has it as its closest point: an edge or vertex counts when every
// candidate triangle of the same mesh that contains it reports it, once, in
// the slot of the first candidate reporting it, and touches when closer
// than R.  Slots without a contact restart their tangential overlap at zero.

// acc[c] += the values of the 8 lanes of a particle, slot by slot (lane = 8
// slot + place, so a row of 16 lanes holds two slots)
__device__ __forceinline__ void add_eight(double* acc, const double* v, int n) {
#pragma unroll
  for (int c = 0; c < n; ++c) {
    double a, b, q[4];
    swap32(v[c], a, b);
    swap16(a, q[0], q[1]);
    swap16(b, q[2], q[3]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double o = dpp0<0x128>(q[r]);  // the row rotated by 8 lanes
      const bool upper = (threadIdx.x & 8) != 0;
      acc[c] = (acc[c] + (upper ? o : q[r])) + (upper ? q[r] : o);
    }
  }
}

template <typename R>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
k_mesh(StepParams sp, const PairCoef* __restrict__ pwc, const WallDev* __restrict__ walls,
       MeshTables mt, ParticleBufs in, const int* __restrict__ info, MeshSlots ms,
       double4* __restrict__ Fm, double4* __restrict__ Tm, const int64_t* __restrict__ clock,
       int64_t step_rel, const int* __restrict__ flags) {
  static_assert(kMeshSlots == 8, "a lane per slot, eight particles to a wavefront");
  const int n = sp.n;
  const int count = ms.list[n];
  const int slot = (threadIdx.x & 63) >> 3;
  const int place = ((int)(blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 8 + (threadIdx.x & 7);
  // whole wavefronts go round together: the lanes of a particle exchange
  const int first = (place & ~7), stride = (int)(gridDim.x * blockDim.x >> 6) * 8;
  for (int w0 = first; w0 < count; w0 += stride) {
    const int at = w0 + (threadIdx.x & 7);
    const int i = ms.list[at < count ? at : w0];
    const int inf = info[i];
    const bool on = at < count && !(inf & kInactive) && *flags == 0;
    const double4 xi = in.pos[i], vi = in.vel[i], wi = in.omg[i];
    const double x[3] = {xi.x, xi.y, xi.z};
    const double rad = xi.w;
    const double t = (double)(*clock + step_rel) * sp.dt;
    const int64_t h = (int64_t)(3 * slot) * n + i;
    // the feature that this lane's candidate reports
    const int tr = on ? ms.tri[(int64_t)slot * n + i] : -1;
    int wl = -1, kind = -1, fa = -1, fb = -1, tv0 = -1, tv1 = -1, tv2 = -1;
    bool near = false;  // closer than R (faces: above the plane)
    TriGeo g;
    double n0 = 0.0, n1 = 0.0, n2 = 0.0;  // the triangle's normal
    if (tr >= 0) {
      const TriDev& Tt = mt.tri[tr];
      wl = Tt.wall;
      tri_closest(Tt, walls[wl].vel, t, x, g);
      n0 = Tt.n[0];
      n1 = Tt.n[1];
      n2 = Tt.n[2];
      tv0 = Tt.v[0];
      tv1 = Tt.v[1];
      tv2 = Tt.v[2];
      kind = g.feature;
      near = g.feature == 0 ? g.s < rad : (g.d2 < rad * rad && g.d2 > 0.0);
      const int va = g.a == 0 ? tv0 : (g.a == 1 ? tv1 : tv2);
      const int vb = g.b == 0 ? tv0 : (g.b == 1 ? tv1 : tv2);
      fa = kind == 0 ? tr : (kind == 1 ? (va < vb ? va : vb) : va);
      if (kind == 1) fb = va < vb ? vb : va;
    }
    // does this slot carry a contact
    bool dropped = false, owner = true;
#pragma unroll 1
    for (int j = 0; j < kMeshSlots; ++j) {
      const int from = 8 * j + (threadIdx.x & 7);
      const int o_tri = __shfl(tr, from, 64), o_wl = __shfl(wl, from, 64);
      const int o_kind = __shfl(kind, from, 64), o_fa = __shfl(fa, from, 64);
      const int o_fb = __shfl(fb, from, 64);
      const int o_v0 = __shfl(tv0, from, 64), o_v1 = __shfl(tv1, from, 64),
                o_v2 = __shfl(tv2, from, 64);
      if (o_tri < 0 || o_wl != wl) continue;
      const bool same = o_kind == kind && o_fa == fa && o_fb == fb;
      const bool has_a = o_v0 == fa || o_v1 == fa || o_v2 == fa;
      const bool has_b = o_v0 == fb || o_v1 == fb || o_v2 == fb;
      if (has_a && (kind == 2 || has_b) && !same) dropped = true;
      if (j < slot && same) owner = false;
    }
    bool contact = false;
    double C[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (tr >= 0) {
      const WallDev& W = walls[wl];
      if (t >= W.t_on && t < W.t_off) contact = near && (kind == 0 || (!dropped && owner));
      double dtl[3] = {0.0, 0.0, 0.0};
      if (contact) {
        double gn[3], gdn;
        if (kind == 0) {
          gn[0] = -n0;
          gn[1] = -n1;
          gn[2] = -n2;
          gdn = rad - g.s;
        } else {
          const double dist = sqrt(g.d2);
          gn[0] = (g.q[0] - x[0]) / dist;
          gn[1] = (g.q[1] - x[1]) / dist;
          gn[2] = (g.q[2] - x[2]) / dist;
          gdn = rad - dist;
        }
        const double arm[3] = {g.q[0] - (W.ax[0] + W.vel[0] * t), g.q[1] - (W.ax[1] + W.vel[1] * t),
                               g.q[2] - (W.ax[2] + W.vel[2] * t)};
        dtl[0] = ms.hist[h];
        dtl[1] = ms.hist[h + n];
        dtl[2] = ms.hist[h + 2 * (int64_t)n];
        const int row = ((inf >> kInstShift) * kMaxTypes + (inf & kTypeMask)) * kMaxTypes;
        wall_law<R>(pwc[row + W.material], sp.rolling, sp.model, sp.dt, W, gn, gdn, arm, xi, vi, wi,
                    dtl, C, C + 3);
      }
      ms.hist[h] = dtl[0];
      ms.hist[h + n] = dtl[1];
      ms.hist[h + 2 * (int64_t)n] = dtl[2];
    }
    double FT[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    add_eight(FT, C, 6);
    if (slot == 0 && at < count) {
      Fm[i] = make_double4(FT[0], FT[1], FT[2], 0.0);
      Tm[i] = make_double4(FT[3], FT[4], FT[5], 0.0);
    }
  }
}

hipError_t launch_mesh(int precision, const StepParams& sp, const PairCoef* pw,
                       const WallDev* walls, MeshTables mt, ParticleBufs in, const int* info,
                       MeshSlots ms, double4* Fm, double4* Tm, const int64_t* clock,
                       int64_t step_rel, const int* flags, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  if (precision == 0)
    hipLaunchKernelGGL(k_mesh<double>, dim3(mesh_grid(sp.n)), dim3(kBlock), 0, s, sp, pw, walls,
                       mt, in, info, ms, Fm, Tm, clock, step_rel, flags);
  else
    hipLaunchKernelGGL(k_mesh<float>, dim3(mesh_grid(sp.n)), dim3(kBlock), 0, s, sp, pw, walls,
                       mt, in, info, ms, Fm, Tm, clock, step_rel, flags);
  return hipGetLastError();
}

// ------------------------------------------------------ kick-drift, clock

// first half kick and drift of particle i from the stored forces; returns the
// squared drift in units of half the skin when asked for it
__device__ __forceinline__ double kick_drift_one(int i, const StepParams& sp, const InstDev* __restrict__ inst,
                                 ParticleBufs st, const int* __restrict__ info,
                                 const double4* __restrict__ F,
                                 const double4* __restrict__ T, const bool want_drift) {
  double4 x = st.pos[i], v = st.vel[i], w = st.omg[i];
  double4 f = F[i], tq = T[i];
  const double h = sp.hdt, dt = sp.dt;
  // vel.w = 1/m, omg.w = 1/I
  double a0 = f.x * v.w + sp.g[0], a1 = f.y * v.w + sp.g[1], a2 = f.z * v.w + sp.g[2];
  v.x = v.x + a0 * h;
  v.y = v.y + a1 * h;
  v.z = v.z + a2 * h;
  w.x = w.x + (tq.x * w.w) * h;
  w.y = w.y + (tq.y * w.w) * h;
  w.z = w.z + (tq.z * w.w) * h;
  x.x = x.x + v.x * dt;
  x.y = x.y + v.y * dt;
  x.z = x.z + v.z * dt;
  st.pos[i] = x;
  st.vel[i] = v;
  st.omg[i] = w;
  if (!want_drift) return 0.0;
  return drift2(v, drift_scale(sp, inst, info[i]));
}

__global__ void k_kick_drift(StepParams sp, const InstDev* __restrict__ inst, ParticleBufs st,
                             const int* __restrict__ info, const double4* __restrict__ F,
                             const double4* __restrict__ T,
                             const int64_t* __restrict__ clock, int64_t step_rel) {
  int i = xcd_block() * kBlock + threadIdx.x;
  double d = 0.0;
  if (i < sp.n && !(info[i] & kInactive)) d = kick_drift_one(i, sp, inst, st, info, F, T, true);
  // the displacement bound's record of the update that produced x^step
  const int64_t step = *clock + step_rel;
  raise_drift(sp, sp.brec + bound_slot(step, 0) * kDriftRec, d);
}

hipError_t launch_kick_drift(const StepParams& sp, const InstDev* inst, ParticleBufs st,
                             const int* info, const double4* F, const double4* T,
                             const int64_t* clock, int64_t step_rel, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_kick_drift, dim3(grid_for(sp.n)), dim3(kBlock), 0, s, sp, inst, st, info,
                     F, T, clock, step_rel);
  return hipGetLastError();
}

__global__ void k_tick(int64_t* clock, int64_t k) {
  if (threadIdx.x == 0 && blockIdx.x == 0) clock[0] += k;
}

hipError_t launch_tick(int64_t* clock, int64_t k, hipStream_t s) {
  hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, s, clock, k);
  return hipGetLastError();
}

// -------------------------------------------------------------------- stats

__global__ void k_stats(StepParams sp, const double4* __restrict__ pos,
                        const int* __restrict__ info, NbrList l, WallSlots ws,
                        unsigned long long* out) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  unsigned long long a = 0, e = 0, tch = 0, wc = 0;
  if (i < sp.n && !(info[i] & kInactive)) {
    a = 1;
    double4 xi = pos[i];
    int len = l.rowlen[i];
    e = (unsigned long long)len;
    for (int k = 0; k < len; ++k) {
      int j = l.nbr[nbr_entry(i, k, sp.max_nb)] & 0x7fffffff;
      double4 xj = pos[j];
      double dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
      double d2 = (dx * dx + dy * dy) + dz * dz;
      double rs = xi.w + xj.w;
      if (d2 < rs * rs) ++tch;
    }
    for (int s = 0; s < kWallSlots; ++s)
      if (ws.wid[(int64_t)s * sp.n + i] >= 0) ++wc;
  }
  // wave reduction, then one atomic per wave
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o, 64);
    e += __shfl_down(e, o, 64);
    tch += __shfl_down(tch, o, 64);
    wc += __shfl_down(wc, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&out[0], a);
    atomicAdd(&out[1], e);
    atomicAdd(&out[2], tch);
    atomicAdd(&out[3], wc);
  }
}

hipError_t launch_stats(const StepParams& sp, const double4* pos, const int* info, NbrList l,
                        WallSlots ws, unsigned long long* out, hipStream_t s) {
  if (sp.n <= 0) return hipSuccess;
  unsigned nb = (unsigned)((sp.n + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_stats, dim3(nb), dim3(kBlock), 0, s, sp, pos, info, l, ws, out);
  return hipGetLastError();
}

// ------------------------------------------------------- readout of rows
//
// The input order is found with one scattered 4-byte store per particle; the
// rows are then gathered, so that the results, which may lie in host memory,
// are written in whole lines, one number per thread.  Bound by the gathers (32
// of every 128 bytes fetched are used): about 0.1 ms for the state of a
// million spheres, against 38 ms for copying every array to the host,
// reordering it there and copying it back.

__global__ void k_place(int n, int inst, int gid_base, const int* __restrict__ info,
                        const int* __restrict__ gid, int* __restrict__ at) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p < n && (info[p] >> kInstShift) == inst) at[gid[p] - gid_base] = p;
}

// blockIdx.y: which of the three arrays, 3 the active flags
__global__ void k_rows_out(int64_t n, const int* __restrict__ at, RowsOut r,
                           const int* __restrict__ info) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int a = blockIdx.y;
  if (a == 3) {
    if (r.active && t < n) r.active[t] = (info[at[t]] & kInactive) ? 0 : 1;
    return;
  }
  const double4* __restrict__ src = a == 0 ? r.src[0] : (a == 1 ? r.src[1] : r.src[2]);
  double* __restrict__ out = a == 0 ? r.out[0] : (a == 1 ? r.out[1] : r.out[2]);
  if (!out || t >= 3 * n) return;
  const int64_t g = t / 3;
  out[t] = reinterpret_cast<const double*>(src + at[g])[t - 3 * g];
}

hipError_t launch_place(int n_all, int inst, int gid_base, const int* info, const int* gid,
                        int* at, hipStream_t s) {
  if (n_all <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_place, dim3((unsigned)((n_all + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     n_all, inst, gid_base, info, gid, at);
  return hipGetLastError();
}

hipError_t launch_rows_out(int64_t n, const int* at, const RowsOut& r, const int* info,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rows_out, dim3((unsigned)((3 * n + kBlock - 1) / kBlock), 4), dim3(kBlock),
                     0, s, n, at, r, info);
  return hipGetLastError();
}

// ------------------------------------------------ contact list on the device
//
// The candidate pairs of one instance, each once as (gid_i, gid_j) with
// gid_i < gid_j, written to caller buffers in the sorted order of the first
// particle and then its row order: a per-block count, a scan of the block
// counts, and a fill in which each block recounts its threads' pairs and
// places them after its block's offset.  Only the block counts and their
// scan need memory beyond the outputs.

__device__ __forceinline__ int pairs_of_row(const StepParams& sp, int inst, int p,
                                            const int* __restrict__ info,
                                            const int* __restrict__ gid, const NbrList& l) {
  if (p >= sp.n) return 0;
  const int inf = info[p];
  if ((inf & kInactive) || (inf >> kInstShift) != inst) return 0;
  const int g = gid[p];
  const int len = l.rowlen[p];
  int c = 0;
  for (int k = 0; k < len; ++k) {
    const int q = l.nbr[nbr_entry(p, k, sp.max_nb)] & kIndexMask;
    c += gid[q] > g ? 1 : 0;
  }
  return c;
}

__global__ void k_pairs_count(StepParams sp, int inst, const int* __restrict__ info,
                              const int* __restrict__ gid, NbrList l, int* __restrict__ bcount) {
  __shared__ int sh[4];
  const int p = blockIdx.x * kBlock + threadIdx.x;
  const int c = pairs_of_row(sp, inst, p, info, gid, l);
  int tot;
  block_exclusive_scan(c, sh, &tot);
  if (threadIdx.x == 0) bcount[blockIdx.x] = tot;
}

__global__ void k_pairs_fill(StepParams sp, int inst, int gid_base,
                             const double4* __restrict__ pos, const int* __restrict__ info,
                             const int* __restrict__ gid, NbrList l,
                             const int* __restrict__ bstart, int64_t* __restrict__ pairs,
                             double* __restrict__ delta_t, uint8_t* __restrict__ touching) {
  __shared__ int sh[4];
  const int p = blockIdx.x * kBlock + threadIdx.x;
  const int c = pairs_of_row(sp, inst, p, info, gid, l);
  int tot;
  int64_t o = (int64_t)bstart[blockIdx.x] + block_exclusive_scan(c, sh, &tot);
  if (c == 0) return;
  const int g = gid[p];
  const double4 xp = pos[p];
  const int len = l.rowlen[p];
  for (int k = 0; k < len; ++k) {
    const int64_t e = nbr_entry(p, k, sp.max_nb);
    const int jr = l.nbr[e];
    const int q = jr & kIndexMask;
    const int gq = gid[q];
    if (!(gq > g)) continue;
    if (pairs) {
      pairs[2 * o] = g - gid_base;
      pairs[2 * o + 1] = gq - gid_base;
    }
    if (delta_t) {
      // bit 31: the pair touched at the last evaluation and holds a history
      const bool h = (jr & kTouchedBit) != 0;
      delta_t[3 * o] = h ? l.hist[e] : 0.0;
      delta_t[3 * o + 1] = h ? l.hist[l.cap + e] : 0.0;
      delta_t[3 * o + 2] = h ? l.hist[2 * l.cap + e] : 0.0;
    }
    if (touching) {
      const double4 xq = pos[q];
      const double dx = xq.x - xp.x, dy = xq.y - xp.y, dz = xq.z - xp.z;
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const double rs = xp.w + xq.w;
      touching[o] = d2 < rs * rs ? 1 : 0;
    }
    ++o;
  }
}

int64_t pairs_scratch_ints(int n) {
  const int64_t nb = (n + kBlock - 1) / kBlock;
  return nb + (nb + 2) + ((nb + 1 + kScanTile - 1) / kScanTile + 1);
}

hipError_t launch_pairs_count(const StepParams& sp, int inst, const int* info, const int* gid,
                              NbrList l, int* scratch, hipStream_t s) {
  const int64_t nb = (sp.n + kBlock - 1) / kBlock;
  int* bcount = scratch;
  int* bstart = scratch + nb;
  int* tiles = bstart + nb + 2;
  if (nb > 0)
    hipLaunchKernelGGL(k_pairs_count, dim3((unsigned)nb), dim3(kBlock), 0, s, sp, inst, info,
                       gid, l, bcount);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nb == 0) return launch_fill_i32(bstart, 0, 1, s);
  return launch_scan(bcount, bstart, nb, tiles, s);
}

hipError_t launch_pairs_fill(const StepParams& sp, int inst, int gid_base, const double4* pos,
                             const int* info, const int* gid, NbrList l, const int* scratch,
                             int64_t* pairs, double* delta_t, uint8_t* touching,
                             hipStream_t s) {
  const int64_t nb = (sp.n + kBlock - 1) / kBlock;
  if (nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pairs_fill, dim3((unsigned)nb), dim3(kBlock), 0, s, sp, inst, gid_base,
                     pos, info, gid, l, scratch + nb, pairs, delta_t, touching);
  return hipGetLastError();
}

// -------------------------------------------------- contacts in input order
//
// One thread per particle: a count per gid, a scan, and a fill in which each
// thread writes its pairs in the order of the other gid (a row is short enough
// to rank every entry against the whole row).  The lists used to be copied to
// the host whole (28 bytes for every one of max_nb entries per particle) and
// filtered and sorted there: 35 ms and more for 100,000 spheres; now bound by
// the copy of the results.

int64_t contact_scratch_ints(int64_t n) {
  return n + (n + 2) + ((n + kScanTile - 1) / kScanTile + 1);
}
int* contact_starts(int* scratch, int64_t n) { return scratch + n; }

__global__ void k_contacts_count(StepParams sp, int inst, int gid_base,
                                 const int* __restrict__ info, const int* __restrict__ gid,
                                 NbrList l, int* __restrict__ count) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= sp.n || (info[p] >> kInstShift) != inst) return;
  count[gid[p] - gid_base] = pairs_of_row(sp, inst, p, info, gid, l);
}

__global__ void k_contacts_fill(StepParams sp, int inst, int gid_base,
                                const double4* __restrict__ pos, const int* __restrict__ info,
                                const int* __restrict__ gid, NbrList l,
                                const int* __restrict__ starts, const double* __restrict__ planes,
                                int64_t* __restrict__ pairs, double* __restrict__ values,
                                uint8_t* __restrict__ touching) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= sp.n || (info[p] >> kInstShift) != inst || (info[p] & kInactive)) return;
  const int g = gid[p];
  const int64_t first = starts[g - gid_base];
  if (starts[g - gid_base + 1] == first) return;
  const double4 xp = pos[p];
  const int len = l.rowlen[p];
  for (int k = 0; k < len; ++k) {
    const int64_t e = nbr_entry(p, k, sp.max_nb);
    const int jr = l.nbr[e];
    const int q = jr & kIndexMask;
    const int gq = gid[q];
    if (!(gq > g)) continue;
    int64_t o = first;
    for (int m = 0; m < len; ++m) {
      const int gm = gid[l.nbr[nbr_entry(p, m, sp.max_nb)] & kIndexMask];
      o += gm > g && gm < gq ? 1 : 0;
    }
    if (pairs) {
      pairs[2 * o] = g - gid_base;
      pairs[2 * o + 1] = gq - gid_base;
    }
    if (values) {
      const bool h = (jr & kTouchedBit) != 0;
      for (int a = 0; a < 3; ++a) values[3 * o + a] = h ? planes[a * l.cap + e] : 0.0;
    }
    if (touching) {
      const double4 xq = pos[q];
      const double dx = xq.x - xp.x, dy = xq.y - xp.y, dz = xq.z - xp.z;
      const double d2 = (dx * dx + dy * dy) + dz * dz;
      const double rs = xp.w + xq.w;
      touching[o] = d2 < rs * rs ? 1 : 0;
    }
  }
}

__global__ void k_wall_contacts_count(int n_all, int inst, int gid_base,
                                      const int* __restrict__ info, const int* __restrict__ gid,
                                      WallSlots ws, int* __restrict__ count) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= n_all || (info[p] >> kInstShift) != inst) return;
  int c = 0;
  while (c < kWallSlots && ws.wid[(int64_t)c * n_all + p] >= 0) ++c;
  count[gid[p] - gid_base] = c;
}

// a particle's slots are in the order of the walls
__global__ void k_wall_contacts_fill(int n_all, int inst, int gid_base, int w_begin,
                                     const int* __restrict__ info, const int* __restrict__ gid,
                                     WallSlots ws, const int* __restrict__ starts,
                                     int64_t* __restrict__ pairs, double* __restrict__ delta_t) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= n_all || (info[p] >> kInstShift) != inst) return;
  const int g = gid[p] - gid_base;
  const int64_t o = starts[g];
  const int c = starts[g + 1] - (int)o;
  for (int s = 0; s < c; ++s) {
    if (pairs) {
      pairs[2 * (o + s)] = g;
      pairs[2 * (o + s) + 1] = ws.wid[(int64_t)s * n_all + p] - w_begin;
    }
    if (delta_t)
      for (int a = 0; a < 3; ++a)
        delta_t[3 * (o + s) + a] = ws.hist[(int64_t)(3 * s + a) * n_all + p];
  }
}

static inline dim3 one_per_thread(int64_t n) {
  return dim3((unsigned)std::max<int64_t>((n + kBlock - 1) / kBlock, 1));
}

static hipError_t scan_counts(int64_t n, int* scratch, hipStream_t s) {
  return launch_scan(scratch, scratch + n, n, scratch + n + (n + 2), s);
}

hipError_t launch_contacts_count(const StepParams& sp, int inst, int gid_base, int64_t n,
                                 const int* info, const int* gid, NbrList l, int* scratch,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_contacts_count, one_per_thread(sp.n), dim3(kBlock), 0, s, sp, inst,
                     gid_base, info, gid, l, scratch);
  return scan_counts(n, scratch, s);
}

hipError_t launch_contacts_fill(const StepParams& sp, int inst, int gid_base, const double4* pos,
                                const int* info, const int* gid, NbrList l, const int* starts,
                                const double* planes, int64_t* pairs, double* values,
                                uint8_t* touching, hipStream_t s) {
  hipLaunchKernelGGL(k_contacts_fill, one_per_thread(sp.n), dim3(kBlock), 0, s, sp, inst, gid_base,
                     pos, info, gid, l, starts, planes, pairs, values, touching);
  return hipGetLastError();
}

hipError_t launch_wall_contacts_count(int n_all, int inst, int gid_base, int64_t n,
                                      const int* info, const int* gid, WallSlots ws, int* scratch,
                                      hipStream_t s) {
  hipLaunchKernelGGL(k_wall_contacts_count, one_per_thread(n_all), dim3(kBlock), 0, s, n_all, inst,
                     gid_base, info, gid, ws, scratch);
  return scan_counts(n, scratch, s);
}

hipError_t launch_wall_contacts_fill(int n_all, int inst, int gid_base, int w_begin,
                                     const int* info, const int* gid, WallSlots ws,
                                     const int* starts, int64_t* pairs, double* delta_t,
                                     hipStream_t s) {
  hipLaunchKernelGGL(k_wall_contacts_fill, one_per_thread(n_all), dim3(kBlock), 0, s, n_all, inst,
                     gid_base, w_begin, info, gid, ws, starts, pairs, delta_t);
  return hipGetLastError();
}

// ------------------------------------------------------------ exact resume

__global__ void k_restore_find(StepParams sp, int64_t n, const int* __restrict__ at, NbrList l,
                               SavedPairs v, unsigned long long* __restrict__ bad) {
  const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (m >= v.count) return;
  const int64_t gi = v.pairs[2 * m], gj = v.pairs[2 * m + 1];
  if (gi < 0 || gi >= n || gj < 0 || gj >= n || gi == gj) {
    atomicMin(bad, 2ull * (unsigned long long)m);
    return;
  }
  const int pq[2] = {at[gi], at[gj]};
  for (int side = 0; side < 2; ++side) {
    const int p = pq[side], q = pq[1 - side];
    int64_t e = -1;
    const int len = l.rowlen[p];
    for (int k = 0; k < len && e < 0; ++k) {
      const int64_t t = nbr_entry(p, k, sp.max_nb);
      if ((l.nbr[t] & kIndexMask) == q) e = t;
    }
    v.entry[2 * m + side] = e;
    if (e < 0)
      atomicMin(bad, 2ull * (unsigned long long)m + 1ull);
    else
      atomicMax(v.owner + e, (int)m);
  }
}

// A pair that does not touch at the current positions keeps no history: the
// first force evaluation, here, would restart it at zero (and the row cuts of
// the force kernel may not read its entry until it can touch).
__global__ void k_restore_apply(StepParams sp, const int* __restrict__ at,
                                const double4* __restrict__ pos, NbrList l, SavedPairs v) {
  const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (m >= v.count) return;
  const double4 xp = pos[at[v.pairs[2 * m]]], xq = pos[at[v.pairs[2 * m + 1]]];
  const double dx = xq.x - xp.x, dy = xq.y - xp.y, dz = xq.z - xp.z;
  const double rsum = xp.w + xq.w;
  if (!(((dx * dx + dy * dy) + dz * dz) < rsum * rsum)) return;
  for (int side = 0; side < 2; ++side) {
    const int64_t e = v.entry[2 * m + side];
    if (v.owner[e] != (int)m) continue;
    // history of i -> j, and the exact negative from j's side
    const double sgn = side == 0 ? 1.0 : -1.0;
    l.nbr[e] |= kTouchedBit;
    for (int a = 0; a < 3; ++a) l.hist[a * l.cap + e] = sgn * v.delta[3 * m + a];
  }
}

__global__ void k_restore_find_walls(int n_all, int64_t n, int w_begin, int n_walls,
                                     const int* __restrict__ at, WallSlots ws, SavedPairs v,
                                     unsigned long long* __restrict__ bad) {
  const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (m >= v.count) return;
  const int64_t g = v.pairs[2 * m], w = v.pairs[2 * m + 1];
  if (g < 0 || g >= n || w < 0 || w >= n_walls) {
    atomicMin(bad, 2ull * (unsigned long long)m);
    return;
  }
  int64_t slot = -1;
  for (int s = 0; s < kWallSlots && slot < 0; ++s)
    if (ws.wid[(int64_t)s * n_all + at[g]] == w_begin + (int)w) slot = (int64_t)s * n_all + at[g];
  v.entry[m] = slot;
  if (slot < 0)
    atomicMin(bad, 2ull * (unsigned long long)m + 1ull);
  else
    atomicMax(v.owner + slot, (int)m);
}

__global__ void k_restore_apply_walls(int n_all, WallSlots ws, SavedPairs v) {
  const int64_t m = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (m >= v.count || v.owner[v.entry[m]] != (int)m) return;
  const int64_t s = v.entry[m] / n_all, p = v.entry[m] - s * n_all;
  for (int a = 0; a < 3; ++a) ws.hist[(3 * s + a) * n_all + p] = v.delta[3 * m + a];
}

__global__ void k_restore_clear(StepParams sp, int inst, const int* __restrict__ info, NbrList l,
                                WallSlots ws) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= sp.n || (info[p] >> kInstShift) != inst) return;
  for (int a = 0; a < 3 * kWallSlots; ++a) ws.hist[(int64_t)a * sp.n + p] = 0.0;
  const int len = l.rowlen[p];
  for (int k = 0; k < len; ++k) {
    const int64_t e = nbr_entry(p, k, sp.max_nb);
    const int jr = l.nbr[e];
    if (jr & kTouchedBit) l.nbr[e] = jr & kIndexMask;
  }
}

__global__ void k_rows_in(int64_t n, const int* __restrict__ at, const double* __restrict__ src,
                          double4* __restrict__ dst) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g < n) dst[at[g]] = make_double4(src[3 * g], src[3 * g + 1], src[3 * g + 2], 0.0);
}

hipError_t launch_restore_find(const StepParams& sp, int64_t n, const int* at, NbrList l,
                               const SavedPairs& v, unsigned long long* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_restore_find, one_per_thread(v.count), dim3(kBlock), 0, s, sp, n, at, l, v,
                     bad);
  return hipGetLastError();
}
hipError_t launch_restore_apply(const StepParams& sp, const int* at, const double4* pos,
                                NbrList l, const SavedPairs& v, hipStream_t s) {
  hipLaunchKernelGGL(k_restore_apply, one_per_thread(v.count), dim3(kBlock), 0, s, sp, at, pos, l,
                     v);
  return hipGetLastError();
}
hipError_t launch_restore_find_walls(int n_all, int64_t n, int w_begin, int n_walls,
                                     const int* at, WallSlots ws, const SavedPairs& v,
                                     unsigned long long* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_restore_find_walls, one_per_thread(v.count), dim3(kBlock), 0, s, n_all, n,
                     w_begin, n_walls, at, ws, v, bad);
  return hipGetLastError();
}
hipError_t launch_restore_apply_walls(int n_all, WallSlots ws, const SavedPairs& v,
                                      hipStream_t s) {
  hipLaunchKernelGGL(k_restore_apply_walls, one_per_thread(v.count), dim3(kBlock), 0, s, n_all, ws,
                     v);
  return hipGetLastError();
}
hipError_t launch_restore_clear(const StepParams& sp, int inst, const int* info, NbrList l,
                                WallSlots ws, hipStream_t s) {
  hipLaunchKernelGGL(k_restore_clear, one_per_thread(sp.n), dim3(kBlock), 0, s, sp, inst, info, l,
                     ws);
  return hipGetLastError();
}
hipError_t launch_rows_in(int64_t n, const int* at, const double* src, double4* dst,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_rows_in, one_per_thread(n), dim3(kBlock), 0, s, n, at, src, dst);
  return hipGetLastError();
}

}  // namespace demgpu
