// Device-side data structures and kernel launch interface of the MI355X DEM
// library.  Shared by the HIP kernels (dem_kernels.hip) and the host runtime
// behind the C ABI (dem_api.hip).  Nothing here is visible to library users.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace demgpu {

constexpr int kMaxTypes = 16;
constexpr int kMaxWalls = 32;
constexpr int kWallSlots = 4;   // particle-wall contacts kept per particle
constexpr int kMeshSlots = 8;   // particle-triangle candidates kept per particle
constexpr int kBlock = 256;     // threads per workgroup (4 wave64)
constexpr int kWave = 64;
constexpr int kTypeMask = 0xffff;
constexpr int kInactive = 1 << 16;  // flag bit in the per-particle info word
constexpr int kInstShift = 20;      // info bits 20..30: instance of the particle
// A drift record: up to kDriftSpread words (StepParams::drift_words), each
// kDriftStride words (256 bytes) from the next.  Every wavefront of a step
// raises one of them with an atomic.  Atomics on one cache line run one after
// the other (about 6 ns each): with 32 words side by side on two lines, the
// 15,648 wavefronts of a million spheres took 90 us over them, a floor under
// every step.
constexpr int kDriftSpread = 32;
constexpr int kDriftStride = 32;
constexpr int kDriftRec = kDriftSpread * kDriftStride;  // words from one record to the next
constexpr int kDriftLog = 32;  // steps the drift log reaches back (a power of two)
constexpr int kMaxInstances = 2048;
constexpr int kMaxMeshTriangles = 1 << 24;  // per instance
// Particles per context: while the contact search builds a row, the top three
// bits of each entry carry the pair's gap class, so sorted indices stay below
// 2^29.
constexpr int kClassShift = 29;
constexpr int64_t kMaxParticles = (int64_t)1 << kClassShift;

// Sticky error bits raised by kernels (read once per dem_step call).
enum : int {
  kFlagGuard = 1,         // a particle moved more than skin/2 between searches
  kFlagNonFinite = 2,     // NaN/Inf in the state
  kFlagNbrOverflow = 4,   // a particle had more candidate neighbours than max_nb
  kFlagWallOverflow = 8,  // more wall candidates than kWallSlots
  kFlagMeshOverflow = 16, // more triangle candidates than kMeshSlots
};

// Per material pair constants of the Hertz-Mindlin law (effective-parameter
// table of Sec. 2.1), with Y_e, G_e the effective moduli and
// beta = ln e / sqrt(ln^2 e + pi^2):  kn = 4/3 Y_e, kt = 8 G_e,
// en = -2 sqrt(5/6) beta sqrt(2 Y_e), et = -2 sqrt(5/6) beta sqrt(8 G_e),
// so that k_n = kn q, k_t = kt q, eta_n = en sqrt(m_e q), eta_t = et sqrt(m_e q)
// with q = sqrt(R_e delta_n); mu and mur are the friction coefficients.
// Linear model: kn = kt = (16/15) Y_e (15 V^2 / (16 Y_e))^(1/5) and en = et =
// 2 / sqrt(1 + (pi / ln e)^2), so that k = kn (R_e^2 m_e)^(1/5) and eta = en
// sqrt(m_e k) (Eqs. linearkn, linearetan).
struct PairCoef {
  double kn, kt, en, et, mu, mur, pad0, pad1;
};

// Wall.  kind 0: plane (point p, unit normal nrm into the domain, optional
// rectangular extent along u / vax).  kind 2: cone, as the cylinder with the
// surface at radius + slope s.  kind 1: cylinder (axis point p, unit axis
// nrm, radius, axial range [smin, smax], particles inside or outside).
// kind 3: triangle mesh (its triangles in the triangle table, found through
// a uniform grid over the mesh at time 0; p is its first corner).  Translation with velocity vel: at time t the point and the
// rotation axis sit at p + vel t and ax + vel t.  Surface velocity at a
// contact point x_c: vel + omega x (x_c - ax(t)).  Active for t_on <= t < t_off.
struct WallDev {
  int kind, bounded, inside, material;
  double p[3], nrm[3], u[3], vax[3];
  double hu, hv, radius, smin, smax;
  double omega[3], ax[3];
  double t_on, t_off;
  double skin;  // the owning instance's skin (contact-search margin)
  double slope, q;  // cone: radius + slope s at axial coordinate s; q = sqrt(1 + slope^2)
  double vel[3];
  double axo[3];  // ax - p: the rotation axis moves with the wall
  // mesh: triangles [tri_begin, tri_begin + tri_count); grid cell (cx, cy,
  // cz) = floor((x - vel t - mlo) / mh) lists its triangles at
  // cell_tri[cell[cell_base + c] .. cell[cell_base + c + 1]), c = cx + mnc0
  // (cy + mnc1 cz)
  int tri_begin, tri_count, cell_base, pad;
  int mnc[3], pad2;
  double mlo[3], mh;
};

// One triangle of a mesh wall: corners at time 0 (the particles' side is the
// side of (p1 - p0) x (p2 - p0)), edge vectors e_c = p_{c+1} - p_c, unit
// normal, the mesh's own corner indices (names of its edges and vertices)
// and the owning wall.
struct TriDev {
  double p[3][3];
  double e[3][3];
  double n[3];
  int v[3];
  int wall;
};

// Particle-triangle candidates: slot s of particle i at s * n + i (global
// triangle index or -1), tangential overlaps in 3 * kMeshSlots planes.
// list: the particles that have candidates, in any order, their number at
// list[n] (one copy: a search writes it).
struct MeshSlots {
  int* tri;
  double* hist;
  int* list;
};

// Triangle table and mesh grids (all null when no instance has a mesh).
struct MeshTables {
  const TriDev* tri;
  const int* cell;
  const int* cell_tri;
};

// Uniform cell grid of one instance: cell (cx,cy,cz) = floor((x - lo)/h).
// Cells are ordered along a Morton (Z-order) curve (the bits of the three
// coordinates interleaved; axes with fewer bits drop out of the interleave at
// the top), and a cell's key is its rank in that order among the grid's
// cells: key = ckey[(cz * nc[1] + cy) * nc[0] + cx], 0 .. n_keys - 1, so the
// key space has no unused keys (a power-of-two Morton range would).
struct GridDev {
  double lo[3], hi[3], h;
  int nc[3];
  const uint32_t* ckey;
  int64_t n_keys;  // nc[0] * nc[1] * nc[2]
};

// A block of neighbouring cells that a workgroup of the contact search works
// on: the cells of an instance whose coordinates agree above the low
// StepParams::sb_bits bits.  Its cells are consecutive in Morton order, so its
// particles are consecutive too: the keys [key, key + ncell); (x, y, z) is its
// first cell.
constexpr int kSearchRegion = 1024;  // particles that its LDS stage holds
struct SearchBlock {
  uint32_t key;
  int ncell, inst, x, y, z;
};

// How a contact search finds its rows (us per search of one MI355X: launches,
// sort and row finishing included).
//   kSearchBlocks  a workgroup for every block of cells
//   kSearchListed  the occupied blocks are listed first; a workgroup for each of
//                  them, or, where they hold fewer than kBlockMin particles on
//                  average (known on the device only), a thread per particle
//   kSearchEach    a thread per particle
//
// The list and the launch that it makes room for take 4 to 5 us: 30,000 spheres
// at a packing of 0.5 among 1,000 blocks 87.5 without and 92 with them, among
// 10,000 91 and 96, 300,000 among 20,000 157 and 157.  Where blocks hold few
// particles they gain from some 2,000 blocks on: 10,000 spheres among 857 blocks
// 77 by blocks, 89 each; among 3,906 91 and 85.  A thread per particle is the better one where blocks hold few
// particles: equal spheres in blocks of 4 x 4 x 4 cells, 1,000,000 at a packing of
// 0.2 (54 to a block) 270 by blocks and 240 each, at 0.25 (68) 298 and 288, at
// 0.3 (81) 304 and 321, at 0.5 (130) 345 and 461; at 0.01 (2.7) 1,650 and 590.
// Where the domain has more than one block for two particles, the list costs
// what the blocks could gain: 1,000,000 at a packing of 0.001 7,010 with a list,
// 2,830 without, and dense in a corner of a domain of 216 times their volume
// 1,795 and 1,646.  Where not even the smallest block's region fits the stage in a
// dense bed, nearly all rows would be found without it: 1,000,000 in cells of
// 3 d 1,415 and 1,050, 284,000 small spheres among large ones 3,390 and 2,120;
// contexts of few blocks keep them while the mean region fits (1,000 loose
// spheres 50 and 88).
constexpr int kListedBlocks = 2048;
constexpr int kBlockMin = 64;
enum { kSearchBlocks, kSearchListed, kSearchEach };
inline int search_way(int64_t n, int64_t n_blocks, bool fits) {
  // (eight cells to the smallest block, 64 to its region)
  if (!fits && (n_blocks > kListedBlocks || n > n_blocks * (kSearchRegion / 8))) return kSearchEach;
  if (n_blocks <= kListedBlocks) return kSearchBlocks;
  return 2 * n_blocks <= n ? kSearchListed : kSearchEach;
}
// Workgroups of a search by blocks.  With a list there are n / kBlockMin blocks
// to go through at most, so that their number does not grow with the domain
// and their threads stay below the 2^32 of a launch.
inline unsigned search_workgroups(int64_t n, int64_t n_blocks, int way) {
  const int64_t most = n / kBlockMin;
  return (unsigned)(way == kSearchListed && most < n_blocks ? most : n_blocks);
}

// Lanes to a particle in the force kernel of a context of n (force_way).
constexpr int64_t kFourLanes = 50000, kTwoLanes = 120000;
inline int force_lanes(int64_t n) { return n <= kFourLanes ? 4 : (n <= kTwoLanes ? 2 : 1); }

// Words of a drift record in use: about 64 wavefronts of a force launch to a word
// (0.4 us of atomics, one after the other), one word for the smallest launches,
// whose lanes then read a single line.  Counted by particles instead, 256
// wavefronts of four lanes to a particle shared a word: 4,096 spheres 9.2 us per
// step instead of 8.1, 8,000 10.1 and 8.9, 15,600 11.1 and 9.7, 30,000 12.0 and 11.2.
inline int drift_words_for(int64_t n) {
  int words = 1;
  while (words < kDriftSpread && (int64_t)words * 64 * 64 < n * force_lanes(n)) words *= 2;
  return words;
}

// What a search keeps in LDS per particle, from the mean row of a dense bed:
// lists of 2 bytes an entry that nearly every particle's candidates fit in (those
// of the others are found a slower way), rows of 4 bytes an entry that may spill a
// little.  (A mean row can be anything: a few large spheres among very many small
// ones.)
inline int list_capacity(double row) { return row < 58.0 ? (int)(1.5 * row) + 1 : 88; }
inline int row_capacity(double row, int max_nb) {
  const int r = row < 40.0 ? (int)(1.2 * row) + 2 : 48;
  const int most = max_nb < 48 ? max_nb : 48;
  return r < most ? r : most;
}

// One independent simulation of a batch.  Its cells use the global keys
// [key_base, key_base + grid.n_keys); its walls are walls[wall_begin,
// wall_end); its material-pair constants start at coef_base in the tables.
struct InstDev {
  GridDev grid;
  uint32_t key_base;
  int wall_begin, wall_end;
  int coef_base;
  double rs2;     // squared search radius
  double guard2;  // (skin/2)^2
  double skin;    // r_s - d_max
  double ihs;     // 2 / skin (drift in units of half the skin)
  double ih;      // 1 / cell edge
  float near2;    // (r_s / cell edge)^2 with a margin for the search's FP32 pretest
};

struct StepParams {
  double dt, hdt;
  double g[3];
  int n;           // number of particles of all instances (active + inactive)
  int max_nb;      // neighbour slots per particle
  int rolling;     // 0 none, 1 constant torque, 2 viscous torque
  int model;       // 0 nonlinear (Hertz-Mindlin), 1 linear spring-dashpot
  uint32_t n_keys; // total cell keys; key n_keys collects inactive particles
  int sb_bits[3];  // search block: 2^sb_bits cells along each axis
  bool sb_fits;    // its region fits the search's LDS stage in a dense bed
  int list_cap;    // candidates past the search's pretest kept per particle in LDS
  int row_cap;     // entries of a row sorted in LDS
  int drift_words; // words of a drift record in use (a power of two <= kDriftSpread)
  double drift_scale;  // dt * 2 / skin when every instance has the same skin,
                       // else 0 (then taken per particle from its instance)
  // Displacement bound since the last contact search, in units of half the
  // skin of each particle's instance, for the row cuts (see NbrList): the
  // force evaluation at absolute step s (positions x^s) uses
  // acc(s) = bacc[(s - 1) % 3] + sqrt(max of brec[s % 3]), where brec[s % 3]
  // (drift_words words, non-negative doubles as bits) holds the largest
  // squared drift |v| dt (half skins) of the update that produced x^s.  The
  // evaluation writes bacc[s % 3] = acc(s), raises brec[(s + 1) % 3] with
  // its own update and clears brec[(s + 2) % 3]; a search at step s sets
  // bacc[(s - 1) % 3] and brec[s % 3] to zero.  No particle has moved more
  // than acc(s) half skins from where the last search saw it.  The evaluation
  // also notes the drift of the update that produced its positions, the root
  // of brec[s % 3], in blog[s % kDriftLog] (for the dynamic search trigger).
  double* bacc;             // 3 words
  unsigned long long* brec; // 3 * kDriftRec words
  double* blog;             // kDriftLog words
};

// Particle arrays in sorted (spatial) order.  pos = (x, y, z, R),
// vel = (v, 1/m), omg = (omega, 1/I).
struct ParticleBufs {
  double4* pos;
  double4* vel;
  double4* omg;
};

// Neighbour list, one row per particle in wave-slab column-major layout:
// entry (i, k) lives at ((i / 64) * max_nb + k) * 64 + i % 64.  Bit 31 of a
// neighbour index is set while the pair touches; the stored history of an
// entry without bit 31 is undefined and stands for zero.
//
// A search orders each row by the gap g = d - (R_i + R_j) it found: the
// touching pairs first, then the pairs with g < s/8, g < s/4, g < s/2 and the
// rest (s the skin); rowcut packs the ends of the middle three groups (10
// bits each, 1023 = the whole row).  Two particles that each moved at most
// acc s/2 since the search come at most acc s closer, so while acc < f the
// entries with g >= f s cannot touch and the force evaluation reads the row
// only up to the matching end (f = 1/8, 1/4, 1/2).
struct NbrList {
  int* nbr;      // sorted index of the neighbour
  double* hist;  // 3 planes of tangential overlap (x, y, z), stride cap
  int* rowlen;
  int64_t cap;   // entries per plane
  int* rowcut;   // per particle: the three row cuts
};

// Gap classes of the row cuts: fractions of the skin.
constexpr double kCutFrac[3] = {0.125, 0.25, 0.5};
constexpr int kCutBits = 10;
constexpr int kCutMask = (1 << kCutBits) - 1;  // a stored cut of 1023 means "the whole row"

// Particle-wall slots: slot s of particle i at s * n + i.
struct WallSlots {
  int* wid;      // wall id or -1
  double* hist;  // 3 * kWallSlots planes of n
};

__host__ __device__ inline int64_t nbr_entry(int i, int k, int max_nb) {
  return ((int64_t)(i >> 6) * max_nb + k) * 64 + (i & 63);
}

// ---------------------------------------------------------------- launches
// Every launcher enqueues on `s` and returns the hipError_t of the launch.

hipError_t launch_fill_i32(int* p, int v, int64_t n, hipStream_t s);
hipError_t launch_keys(const InstDev* inst, const StepParams& sp, const double4* pos,
                       const double4* vel, int* info, const double4* xref, int check_guard,
                       uint32_t* keys, int* rank, int* count, int* flags, hipStream_t s);
// exclusive scan of count[0..m) into start[0..m], start[m] = total; with cse
// also cse[key_cell[k]] = (start[k], start[k + 1]) for the keys k < n_cells
hipError_t launch_scan(const int* count, int* start, int64_t m, int* tile_sums, hipStream_t s,
                       const uint32_t* key_cell = nullptr, int2* cse = nullptr,
                       int64_t n_cells = 0);
hipError_t launch_scatter(int n, const uint32_t* keys, const int* rank, const int* start,
                          int* perm0, hipStream_t s);
hipError_t launch_cell_rank(int n, int64_t n_keys, const int* perm0, const uint32_t* keys,
                            const int* start, const int* gid, int* perm, hipStream_t s);
// The whole sort (launch_fill_i32 .. launch_cell_rank) in one workgroup, for
// contexts that small_sort_fits: start, cse and perm as those leave them.
bool small_sort_fits(int n, int64_t n_keys);
hipError_t launch_sort_small(const InstDev* inst, const StepParams& sp, const double4* pos,
                             const double4* vel, int* info, const double4* xref, int check_guard,
                             const int* gid, const uint32_t* key_cell, int2* cse, int* start,
                             int* perm, int* flags, hipStream_t s);
// perm: new -> old index; inv receives old -> new
// The particle-wall and particle-triangle searches take the walls where they
// are at time (*clock + step_rel) dt.
// It also restarts the displacement bound (StepParams) for the force
// evaluation at step *clock + bound_step_rel.
// near_list: n words of scratch for contexts with meshes, whose two counts
// (MeshSlots::list) are to be zero.  *n_occupied is set to zero (launch_search).
hipError_t launch_reorder(const StepParams& sp, const InstDev* inst, const int* perm, int* inv,
                          ParticleBufs src,
                          ParticleBufs dst, const int* gid_src, int* gid_dst,
                          const int* info_src, int* info_dst, double4* xref,
                          WallSlots ws_src, WallSlots ws_dst, const WallDev* walls,
                          MeshTables mt, MeshSlots ms_src, MeshSlots ms_dst, int* near_list,
                          const double4* F_src, const double4* T_src, double4* F_dst,
                          double4* T_dst, const int64_t* clock, int64_t step_rel,
                          int64_t bound_step_rel, int* n_occupied, int* flags, hipStream_t s);
// cse: (start, end) of every cell in sorted order, indexed by the cell's
// position (key_base + (cz * nc[1] + cy) * nc[0] + cx); start: of every key;
// blocks: the search blocks of all instances in key order; occupied: n_blocks +
// 1 words of scratch, the last of them zero
hipError_t launch_search(const InstDev* inst, const StepParams& sp, const SearchBlock* blocks,
                         int n_blocks, int* occupied, const double4* pos, const int* info,
                         const int2* cse, const int* start, const int* perm, const int* inv,
                         NbrList old_l, NbrList new_l, int* flags, hipStream_t s);

// force + integration kernels.  mode: 0 = velocity Verlet fused (second half
// kick of this step, first half kick and drift of the next), 1 = velocity
// Verlet last step of a call (second half kick, forces stored), 2 = explicit
// Euler (forces at the current state, then the update; forces stored).
// xsel (may be null): particles i with xsel[i] >= 0 add the force and torque
// Fx[i] / Tx[i] to their contact sums (the mesh contacts of the same state;
// xsel is the first mesh candidate slot).  pf (may be null): the force of
// every touching pair on the row's particle is also written to entry (i, k)
// of three planes of l.cap doubles (a per-contact record for tests).
// pair_mode: 1 when the batch is one instance whose particles all have type
// 0 (every particle pair takes the pair table's first entry), 2 when every
// particle has type 0 (the first entry of the particle's own row), else 0.
// block: threads per workgroup (64, 128 or 256; 0: by the number of particles).
hipError_t launch_force(int mode, int precision, const StepParams& sp, const InstDev* inst,
                        const PairCoef* pp,
                        const PairCoef* pw, const WallDev* walls, ParticleBufs in,
                        ParticleBufs out, const int* info, NbrList l, WallSlots ws,
                        double4* F, double4* T, const int64_t* clock, int64_t step_rel,
                        const int* flags, const int* xsel, const double4* Fx, const double4* Tx,
                        double* pf, int block, int pair_mode, hipStream_t s);
// `steps` launches of mode 0 or 2 as one, for contexts of at most kStepsMax
// particles without meshes: the state ends in `out`, which may be `in`.
constexpr int kStepsMax = 128;
hipError_t launch_force_steps(int mode, int precision, const StepParams& sp, const InstDev* inst,
                              const PairCoef* pp, const PairCoef* pw, const WallDev* walls,
                              ParticleBufs in, ParticleBufs out, const int* info, NbrList l,
                              WallSlots ws, double4* F, double4* T, const int64_t* clock,
                              int64_t step_rel, int steps, const int* flags, int pair_mode,
                              hipStream_t s);
// Contacts of the particles with triangle candidates at time (*clock +
// step_rel) dt (tangential overlaps updated): their force and torque into
// Fm / Tm (written for those particles only).
hipError_t launch_mesh(int precision, const StepParams& sp, const PairCoef* pw,
                       const WallDev* walls, MeshTables mt, ParticleBufs in, const int* info,
                       MeshSlots ms, double4* Fm, double4* Tm, const int64_t* clock,
                       int64_t step_rel, const int* flags, hipStream_t s);
// first half kick + drift from stored forces (start of a velocity-Verlet call).
// It produces the positions of step *clock + step_rel, whose displacement-bound
// record (StepParams) it raises to its largest squared drift |v| dt, in units
// of half the particle's skin (each wavefront raises one word).
hipError_t launch_kick_drift(const StepParams& sp, const InstDev* inst, ParticleBufs st,
                             const int* info, const double4* F, const double4* T,
                             const int64_t* clock, int64_t step_rel, hipStream_t s);
hipError_t launch_tick(int64_t* clock, int64_t k, hipStream_t s);
// statistics: out[0] active, [1] list entries, [2] touching entries, [3] wall slots
hipError_t launch_stats(const StepParams& sp, const double4* pos, const int* info,
                        NbrList l, WallSlots ws, unsigned long long* out, hipStream_t s);

// Readout in input order.  launch_place: at[gid - gid_base] = sorted index, for
// the particles of instance inst.  launch_rows_out: the first three components
// of row at[g] of each given array (null: skipped) to out[3 g ..], g < n, and
// the active flag to active[g] (null: skipped).
struct RowsOut {
  const double4* src[3];
  double* out[3];
  uint8_t* active;
};
hipError_t launch_place(int n_all, int inst, int gid_base, const int* info, const int* gid,
                        int* at, hipStream_t s);
hipError_t launch_rows_out(int64_t n, const int* at, const RowsOut& r, const int* info,
                           hipStream_t s);

// Contact lists of an instance (n particles, gids from gid_base) in input order.
// scratch: contact_scratch_ints(n) ints.  *_count leaves the pairs' (a wall
// candidate's) first place per gid in contact_starts(scratch, n)[0 .. n], the
// total last; *_fill writes them there, each gid's sorted.  planes: three
// planes of l.cap doubles, whose values an entry with its top bit set stands
// for (else zeros).  Any output may be null.
int64_t contact_scratch_ints(int64_t n);
int* contact_starts(int* scratch, int64_t n);
hipError_t launch_contacts_count(const StepParams& sp, int inst, int gid_base, int64_t n,
                                 const int* info, const int* gid, NbrList l, int* scratch,
                                 hipStream_t s);
hipError_t launch_contacts_fill(const StepParams& sp, int inst, int gid_base, const double4* pos,
                                const int* info, const int* gid, NbrList l, const int* starts,
                                const double* planes, int64_t* pairs, double* values,
                                uint8_t* touching, hipStream_t s);
hipError_t launch_wall_contacts_count(int n_all, int inst, int gid_base, int64_t n,
                                      const int* info, const int* gid, WallSlots ws, int* scratch,
                                      hipStream_t s);
hipError_t launch_wall_contacts_fill(int n_all, int inst, int gid_base, int w_begin,
                                     const int* info, const int* gid, WallSlots ws,
                                     const int* starts, int64_t* pairs, double* delta_t,
                                     hipStream_t s);

// Histories of saved contacts back into the lists (dem_restore).  at: sorted
// index per gid (launch_place); n: particles of the instance.  The find
// kernels look every contact's entries up (entry: two per pair, slot: one per
// wall contact), note the last contact that names an entry in owner (preset to
// -1) and lower *bad (preset to INT64_MAX) to 2 m (out of range) or 2 m + 1
// (not in the lists) for the first contact m that fails; the apply kernels
// write the histories of the owners.
struct SavedPairs {
  int64_t count;
  const int64_t* pairs;
  const double* delta;
  int64_t* entry;
  int* owner;
};
hipError_t launch_restore_find(const StepParams& sp, int64_t n, const int* at, NbrList l,
                               const SavedPairs& v, unsigned long long* bad, hipStream_t s);
hipError_t launch_restore_apply(const StepParams& sp, const int* at, const double4* pos,
                                NbrList l, const SavedPairs& v, hipStream_t s);
hipError_t launch_restore_find_walls(int n_all, int64_t n, int w_begin, int n_walls,
                                     const int* at, WallSlots ws, const SavedPairs& v,
                                     unsigned long long* bad, hipStream_t s);
hipError_t launch_restore_apply_walls(int n_all, WallSlots ws, const SavedPairs& v,
                                      hipStream_t s);
// every entry and wall slot of an instance without history
hipError_t launch_restore_clear(const StepParams& sp, int inst, const int* info, NbrList l,
                                WallSlots ws, hipStream_t s);
// dst[at[g]] = (src[3 g ..], 0), g < n
hipError_t launch_rows_in(int64_t n, const int* at, const double* src, double4* dst,
                          hipStream_t s);

// Candidate pairs of instance inst on the device (see dem_get_contacts_device).
// scratch holds pairs_scratch_ints(sp.n) ints: block counts, their exclusive
// scan (scratch[nb + nb] is the total afterwards) and the scan's tile sums.
int64_t pairs_scratch_ints(int n);
hipError_t launch_pairs_count(const StepParams& sp, int inst, const int* info, const int* gid,
                              NbrList l, int* scratch, hipStream_t s);
hipError_t launch_pairs_fill(const StepParams& sp, int inst, int gid_base, const double4* pos,
                             const int* info, const int* gid, NbrList l, const int* scratch,
                             int64_t* pairs, double* delta_t, uint8_t* touching, hipStream_t s);

}  // namespace demgpu
