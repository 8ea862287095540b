// Internal declarations shared by the kernels (gd_kernels.hip) and the C ABI
// runtime (gd_api.hip). Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace gd {

// Launch geometry. Workgroups have 256 lanes (4 wave64s), except those of the
// teams and of k_sym_force (512), and of the diagnostics' sort (512) and scan (1024).
constexpr int kBlock = 256;
// j particles staged per LDS tile.
constexpr int kTileJ = 256;
// i particles held per lane by the force kernel: kIPerLane, or
// kIPerLaneLarge in contexts of at least kLargeN particles with eps > 0. More
// i per lane give each lane more independent pair chains and each LDS read
// of j more pairs, which long items repay; at smaller N the mid-size blocks
// are faster with 2 (and pools always use 2).
constexpr int kIPerLane = 2;
constexpr int kIPerLaneLarge = 4;
constexpr int kLargeN = 131072;
// Items the force decomposition aims for: slices are added (in powers of
// two) while i tiles times slices stays within kSliceItems, about two items
// per workgroup of the grid.
constexpr int kSliceItems = 2048;
// Fewest work units (i tiles times j tiles, times the i per lane) at which
// the decomposition stops widening the lanes per i.
constexpr int kMinUnits = 1536;
// Upper bound of the force grid: workgroups loop over items beyond it.
constexpr int kForceGrid = 1024;
// Upper bound of the corrector grid.
constexpr int kCorrectGrid = 2048;
// Shortest j slice (one LDS tile): it bounds the number of slice partials a
// particle has (N / kMinSlice). Small blocks shorten each lane's serial
// chain of pair evaluations with more lanes per i instead (LJ up to 64).
constexpr int kMinSlice = kTileJ;
// Smallest log2 of the lanes that share one i: i tiles hold at most
// (kBlock >> kMinLj) * ipl = 32 (or 64) particles, which keeps the number of
// j slices (and so the partial sums to reduce) small for large blocks.
constexpr int kMinLj = 4;
// Energy: i particles per lane from these sizes on (four, two), workgroups of a
// call, and the items it is cut into at least (where slices of kEnergyMinLen j
// allow).
constexpr int kEnergyN4 = 65536;
constexpr int kEnergyN2 = 4096;
constexpr int kEnergyGrid = 2048;
constexpr int kEnergyItems = 8192;
constexpr int kEnergyMinLen = 32;
// Maximum block-step level (dt = dt_max / 2^level).
constexpr int kMaxLevels = 41;

// Bins of the block-size histogram: bin b counts the block steps whose N_act
// lies in [2^b, 2^(b+1)).
constexpr int kNactBins = 32;

// Mass fractions one diagnostics call can take.
constexpr int kMaxDiagFractions = 32;

// Predictor modes.
enum : int { kPredAuto = 0, kPredAll = 1, kPredExplicit = 2 };

// Decomposition of one force launch over (i tile, j slice) items.
//   lj   : log2 of the lanes sharing one i (LJ = 1 << lj, 1..64, in one wave)
//   it   : i particles per workgroup tile = (kBlock >> lj) * ipl
//   nit  : number of i tiles
//   s    : number of j slices; item = itile * s + slice
//   len  : j particles per slice
struct Plan {
  int lj, it, nit, s, len, items;
};

// Device-resident scheduling and bookkeeping record (lives in the workspace).
//
// Block steps replayed from a graph run two kernels each (k_step_force,
// k_step_correct; small ones in a team, see k_team), and the step's parity
// (0/1, a kernel argument) picks one of two active lists: the corrector of a
// step predicts every particle to the speculated next block time and builds
// the next step's list in the other list, and the next force kernel checks the
// speculation (see k_step_force).
struct Sched {
  long long t_now;   // current block time, in dt_min ticks
  long long t_next;  // block time of the step in flight
  long long t_end;   // steps whose t_next would exceed this are skipped
  // The prepared list and j stream: (block time << 1) | list. One 64-bit word,
  // so that a kernel that reads it while another workgroup rewrites it sees
  // either the old pair or the new one.
  long long spec;
  int n_act;         // active particles of the step in flight
  int kthr;          // a particle is active when its level >= kthr
  int done;          // 1: the step in flight is skipped (t_end reached)
  int lcnt[2];       // compaction counters of the two active lists
  int nonfinite;     // set when a non-finite force or jerk is seen
  int bad_input;     // set by input / state validation
  int refill;        // 1: the step in flight rebuilt the list (no force, no correction)
  int fine;          // finest occupied level of the step in flight
  long long block_steps, particle_steps, pairs, clamps;
  long long refills;  // replayed steps that rebuilt their list instead of stepping
  long long nact_hist[kNactBins];  // block steps by floor(log2 N_act)
  Plan plan;                 // force decomposition of the step in flight
  int hist[kMaxLevels + 1];  // particles per level
  // Team kernel (k_team): workgroups that have started, and that have
  // finished (kTeamOff: called off); launches to leave out.
  int team_join, team_vote, team_skip;
  unsigned team_epoch;  // steps published in the exchange lines since they were cleared
};

// The plan depends only on (n_act, n). The kernel that fixes n_act for a
// step (predictor, or the explicit index list) stores it in the Sched record,
// and the force kernel and every slice reduction read that one copy.
// The decomposition with LJ = 2^lj lanes per i, ipl i per lane and at most
// s_req slices of whole LDS tiles (as many as keep each slice's tile count,
// with none empty).
__host__ __device__ inline Plan plan_with(int n_act, int n, int lj, int s_req, int ipl) {
  int tiles = (n + kTileJ - 1) / kTileJ;
  if (tiles < 1) tiles = 1;
  const int s0 = s_req < 1 ? 1 : (s_req > tiles ? tiles : s_req);
  // it and (in make_plan's plans) s0 are powers of two: shifts, not divisions
  const int lg_it = (8 - lj) + __builtin_ctz((unsigned)ipl);  // kBlock = 2^8
  const int tps = (s0 & (s0 - 1)) == 0 ? (tiles + s0 - 1) >> __builtin_ctz((unsigned)s0)
                                       : (tiles + s0 - 1) / s0;  // tiles per slice
  Plan p;
  p.lj = lj;
  p.it = (kBlock >> lj) * ipl;
  p.nit = (n_act + p.it - 1) >> lg_it;
  if (p.nit < 1) p.nit = 1;
  p.s = (tiles + tps - 1) / tps;
  p.len = tps * kTileJ;
  p.items = p.nit * p.s;
  return p;
}

// The decomposition make_plan considers at lj: slice count the largest power
// of two (at most one per tile) for which i tiles times slices stays within
// kSliceItems. *stop tells whether make_plan takes it: enough work units for
// the grid at this lj with i tiles at least half full, or the last
// candidate (LJ = 64).
__host__ __device__ inline Plan plan_for_lj(int n_act, int n, int lj, int ipl, bool* stop) {
  int tiles = (n + kTileJ - 1) / kTileJ;
  if (tiles < 1) tiles = 1;
  const int it = (kBlock >> lj) * ipl;
  int nit = (n_act + it - 1) >> ((8 - lj) + __builtin_ctz((unsigned)ipl));  // it = 2^(8 - lj) * ipl
  if (nit < 1) nit = 1;
  int s = 1;
  while (2 * s <= tiles && 2 * s * nit <= kSliceItems) s *= 2;
  *stop = lj == 6 || ((long long)nit * tiles * ipl >= kMinUnits && 2 * n_act >= nit * it);
  return plan_with(n_act, n, lj, s, ipl);
}

// The first lj from kMinLj up that gives enough work units (or the last one).
__host__ __device__ inline Plan make_plan(int n_act, int n, int ipl) {
  for (int lj = kMinLj;; ++lj) {
    bool stop = false;
    const Plan p = plan_for_lj(n_act, n, lj, ipl, &stop);
    if (stop) return p;
  }
}

// Rows of the partial-force buffer a context of n particles with ipl i per
// lane needs: for every plan, s * n_act <= s * nit * it <= max(nit,
// kSliceItems) * it with it <= (kBlock >> kMinLj) * ipl, and
// s * n_act <= (n / kMinSlice rounded up) * n. More i per lane never needs
// fewer rows.
constexpr long long partial_rows(long long n, int ipl) {
  const long long it_max = (long long)(kBlock >> kMinLj) * ipl;
  const long long by_items = n + it_max + (long long)kSliceItems * it_max;
  const long long by_slices = ((n + kMinSlice - 1) / kMinSlice) * n;
  const long long rows = by_items < by_slices ? by_items : by_slices;
  // Also scratch of the diagnostics (of 6 rows doubles): 4 n + n / 64 + 5 of them.
  return rows > n + 16 ? rows : n + 16;
}

// Energy decomposition: an item is an i tile of kBlock * ipl particles and a
// slice of len j at or right of it (a power-of-two part of the tile). Tile a
// has the slices a * q .. s0 - 1 of the whole row of slices, q to a tile, so
// only pairs that are wanted make items, all of the same size but for those
// on the diagonal.
struct EPlan {
  int ipl, nit, q, s0, len, grid;
  long long items;
};
__host__ __device__ inline long long eplan_before(const EPlan& e, long long a) {  // items of tiles < a
  return a * e.s0 - e.q * (a * (a - 1) / 2);
}
__host__ __device__ inline EPlan make_eplan(int n) {
  EPlan e;
  e.ipl = n >= kEnergyN4 ? 4 : n >= kEnergyN2 ? 2 : 1;
  const int tile = kBlock * e.ipl;
  e.nit = (n + tile - 1) / tile;
  for (e.q = 1;; e.q *= 2) {
    e.len = tile / e.q;
    e.s0 = (n + e.len - 1) / e.len;
    e.items = eplan_before(e, e.nit);
    if (e.items >= kEnergyItems || e.len <= kEnergyMinLen) break;
  }
  e.grid = e.items < kEnergyGrid ? (int)e.items : kEnergyGrid;
  return e;
}

// ---------------------------------------------------------------------------
// Teams: small block steps in one resident kernel (k_team)
// ---------------------------------------------------------------------------
constexpr int kTeamBlock = 512;      // threads of a team's workgroup
constexpr int kTeamWaves = kTeamBlock / 64;
constexpr int kTeamTiles = 4;        // most tiles of owned j
// Most active particles that every owner of all j computes by itself: with 4 or
// 6 the same, with 16 N = 1024 took 5.34 instead of 4.98 ms (two rounds of
// pairs for each wave take what the exchange does).
constexpr int kTeamSolo = 8;
constexpr int kTeamMaxSlots = 64;    // j slices of the one-particle plan (one per lane of a wave)
constexpr int kTeamMaxCap = 256;     // active particles of a step (LDS)
constexpr int kTeamLine = 128;       // bytes of one exchange line (6 sums with their epochs)
constexpr int kTeamPairs = 1 << 22;  // most pairs (n_act * n) of a team's step
constexpr int kTeamSteps = 1024;     // most steps of one launch of a context's team
constexpr unsigned kTeamLastEpoch = 0xFFFF0000u;
constexpr int kTeamOff = 1 << 30;    // in team_join or team_vote: the launch is called off
constexpr int kTeamSkip = 64;        // launches left out after one that did not find room

// A team's workgroups share a cluster: workgroup w + wp * grp owns the j
// slices w, w + width, ... (ks of them), of the one-particle decomposition's s1
// slices in slot order, and computes the active particles grp, grp + g, ...
struct Team {
  int wgs;    // workgroups (wp * g); 0: no team
  int width;  // slots of the slice reduction per ks: correct_lanes(s1) / ks
  int wp;     // owners of slices: min(width, s1)
  int ks;     // slots per owner
  int g;      // groups that share the active particles
  int cap;    // most active particles of a step
};

// Exchange lines: two sets (the parity of the epoch) of rows lines per owner.
__host__ __device__ inline int team_rows(const Team& t) { return t.cap > t.g ? t.cap : t.g; }
__host__ __device__ inline size_t team_line_bytes(const Team& t) {
  return (size_t)2 * team_rows(t) * t.wp * kTeamLine;
}

// LDS of a team's workgroup, laid out for the largest team (constant offsets:
// with a layout per size the kernel ran out of scalar registers).
struct TeamMem {
  double tile[kTeamTiles][7][kTileJ];           // the owned j, predicted, and their masses
  double st[12][kTeamMaxCap + 1];               // the set (last entry: the central particle)
  double ftot[6][kTeamMaxCap];                  // summed forces, by place in the active list
  double psum[2 * kTeamMaxCap][6];              // sums over the owned slices
  int idx[kTeamMaxCap], lev[kTeamMaxCap + 1];
  int act[kTeamMaxCap];                         // entries of the active particles
  int hist[64], wcnt[kTeamWaves];
  int go, clamp, bad, stuck, bh;
  short mem[kTeamTiles * kTileJ];               // entries of the owned j (-1: not in the set)
};

// Device pointers of one context, carved from the caller's workspace.
struct Dev {
  Sched* sc;
  double* m;
  double* jm;                              // j-stream masses (central particle's zeroed)
  double *x, *y, *z, *vx, *vy, *vz;        // corrected state at t_i
  double *ax, *ay, *az, *jx, *jy, *jz;     // acceleration, jerk at t_i
  double *px, *py, *pz, *pvx, *pvy, *pvz;  // predicted j stream
  long long* tick;                         // t_i in dt_min ticks
  unsigned char* lev;                      // dt_i = dt_max / 2^lev
  // Two active lists, list q at offset q * n of each array (positions
  // 0..n_act-1), with the listed particles' predicted state, a and jerk at
  // t_i, and level, by position.
  int* active;
  double *ix, *iy, *iz, *ivx, *ivy, *ivz;
  double *iax, *iay, *iaz, *ijx, *ijy, *ijz;
  int* ilev;
  // tag[q * n + j]: the block time for which particle j was put in list q
  // (-1: never since the state was loaded).
  long long* tag;
  double* part;                            // [6][partial_rows(n)]: position * s + slot
  double* ebuf;                            // energy partials [grid][3]; results of the diagnostics
  int* nact_log;                           // force-timing pass: N_act of each timed step
  char* xch;                               // a team's exchange lines (null: a context without one)
};

// One force evaluation of an index list (gd_force with indices,
// gd_force_noalloc): the host knows the block size, so the decomposition
// comes as an argument, and the force kernel reads the caller's list itself.
struct ListArgs {
  const int32_t* idx;
  int n_act;
  int direct;          // 1: one slice per particle, the kernel writes acc and jerk
  Plan plan;
  double *acc, *jerk;  // (n_act, 3) outputs, either may be null
  // The caller's rows (gd_force_noalloc), else null: the j stream of d.
  const double *x, *v;
  int* bad;            // set when an index is out of range (null: its row is NaN)
};

struct Consts {
  int n;
  int kmax;          // log2(dt_max / dt_min)
  int force_grid;    // workgroups of a force launch
  int correct_grid;  // workgroups of a corrector launch
  int bh;            // index of the central particle, -1 if none
  int mixed;         // 1: pair arithmetic in mixed precision (GD_FLAG_MIXED)
  double dt_min, dt_max, eta, eps2, eps2_bh;
  double inv_dt_min, inv_dt_max;  // exact reciprocals (powers of two)
  // The decomposition of a one-particle block (log2 lanes per i; j slices
  // s1), the force kernel's i count per lane, and the largest block size up
  // to which every block has the one-particle decomposition (at most
  // 65535), packed as lj1 | ipl << 8 | n1 << 16: one field more would split
  // the corrector's kernel-argument loads into two dependent batches (its
  // scalar registers are full).
  int lj1_ipl, s1;
  long long part_cs;  // component stride of the partial-force buffer (partial_rows(n, ipl))
};
__host__ __device__ inline int lj1_of(const Consts& c) { return c.lj1_ipl & 255; }
__host__ __device__ inline int ipl_of(const Consts& c) { return (c.lj1_ipl >> 8) & 255; }
__host__ __device__ inline int n1_of(const Consts& c) { return (int)((unsigned)c.lj1_ipl >> 16); }

// make_plan(n_act, n, ipl_of(c)) for n_act <= n1_of(c): the one-particle
// decomposition with the i tiles that n_act needs (a few shifts, where
// make_plan's search is a long dependent chain).
__host__ __device__ inline Plan one_plan(int n_act, int n, const Consts& c) {
  const int lj = lj1_of(c), ipl = ipl_of(c);
  const int tiles = (n + kTileJ - 1) / kTileJ;
  Plan p;
  p.lj = lj;
  p.it = (kBlock >> lj) * ipl;
  p.nit = (n_act + p.it - 1) >> ((8 - lj) + __builtin_ctz((unsigned)ipl));
  if (p.nit < 1) p.nit = 1;
  p.s = c.s1;
  p.len = ((tiles + c.s1 - 1) / c.s1) * kTileJ;
  p.items = p.nit * p.s;
  return p;
}

// Lanes the corrector gives one active particle: one per j slice of the
// force plan (rounded up to a power of two), at most a wave.
__host__ __device__ inline int correct_lanes(int s) {
  int l = 1;
  while (l < s && l < 64) l <<= 1;
  return l;
}

// The team of a cluster of n particles (wgs == 0: none). Steps run in a team
// have the one-particle decomposition (at most n1 active), one slot per lane
// of the slice reduction, and one owned j per thread (two where every owner has
// all slices).
//   - ks: with slices of one tile and more than 32 of them, two per owner: an
//     exchange among 64 owners took 2.3 us, among 32 2.0 us.
//   - In a context of at most four tiles every owner has all slices. 32 groups
//     share its larger steps (N = 1024: 4.98 ms; 16 groups 5.14, 8 5.57).
//   - g: groups up to 128 workgroups in all share the pairs of a step: one
//     largest step of N = 16384 took 60.6 ms with 32 workgroups (16 at
//     N = 4096: 17.7 ms), 54.6 with 64, 52.3 with 128 (15.0 ms) and 52.3
//     with 256.
//   - cap: with 2^20 pairs as the most of a step instead of 2^22 N = 16384
//     took 1.5 % more; the set's place in LDS ends it at 256 particles. In a
//     pool, 2^14 pairs per workgroup (4.4 us): the others' teams wait for the
//     slowest (2^15 of them: 81.4 instead of 79.6 ms, 48 clusters).
inline Team make_team(int n, int ipl, int n1, bool pool) {
  Team t{};
  const Plan p1 = make_plan(1, n, ipl);
  const int lanes = correct_lanes(p1.s);
  if (p1.lj != 6 || ipl != kIPerLane || p1.s > kTeamMaxSlots || p1.len > kTeamBlock) return t;
  t.ks = p1.len == kTileJ && lanes > (pool ? 1 : 32) ? 2 : 1;
  if (!pool && p1.s * p1.len <= kTeamTiles * kTileJ) t.ks = lanes;
  t.width = lanes / t.ks;
  t.wp = t.width < p1.s ? t.width : p1.s;
  t.g = 1;
  while (!pool && t.g < (t.wp == 1 ? 32 : 8) && 2 * t.g * t.wp <= 128) t.g *= 2;
  t.cap = (pool ? t.wp << 14 : kTeamPairs) / n;
  if (t.cap > kTeamMaxCap) t.cap = kTeamMaxCap;
  if (t.cap > n1) t.cap = n1;
  t.wgs = t.wp * t.g;
  return t;
}

// ---------------------------------------------------------------------------
// The force of all particles, each pair once (k_sym_force)
// ---------------------------------------------------------------------------
constexpr int kSymBlock = 512;  // threads of a workgroup
constexpr int kSymI = 4;        // i particles per lane
constexpr int kSymTile = 512;   // j of an LDS tile
constexpr int kSymSpan = 3;     // most successive d of a launch

struct SymPlan {
  int wi;           // waves along i: blocks of 64 * kSymI * wi particles
  int nb;           // blocks
  int span;         // successive d of a launch
  long long items;  // pairs of blocks (b, b + d): item d * nb + b
};

// Accumulator array k: six components of n sums. The lists' predicted state,
// acceleration and jerk are 24 n doubles in a row; the rest is in the buffer
// of slice partials.
__host__ __device__ inline double* sym_sums(const Dev& d, int n, int k) {
  return k < 4 ? d.ix + (size_t)k * 6 * n : d.part + (size_t)(k - 4) * 6 * n;
}

// Whether a cluster's initial force takes each pair once: FP64 (the mixed
// arithmetic is that of one side, and its rounding is part of its results),
// one softening, and enough pairs of blocks for the chip. gd_reinit with the
// forces one-sided and with this: N = 24576 1.01 and 1.12 ms, 32768 1.72 and
// 1.39, 65536 6.4 and 4.0.
constexpr int kSymN = 32768;
// Blocks of four waves from here, below of two: N = 131072 takes 14.9 ms with
// four and 16.0 with two, N = 100003 10.5 and 9.5.
constexpr int kSymN4 = 131072;
inline bool sym_init(const Consts& c) { return c.n >= kSymN && !c.mixed && c.bh < 0; }

inline SymPlan make_sym_plan(const Consts& c) {
  SymPlan p;
  p.wi = c.n >= kSymN4 ? 4 : 2;
  const int rows = 64 * kSymI * p.wi;
  p.nb = (c.n + rows - 1) / rows;
  p.items = (long long)p.nb * ((p.nb + 1) / 2) + (p.nb % 2 == 0 ? p.nb / 2 : 0);
  // Three d where two leave workgroups idle, if the arrays have room (N =
  // 32768: 192 workgroups instead of 128, 1.39 instead of 2.06 ms).
  const long long arrays = 4 + c.part_cs / c.n;
  for (p.span = 2; p.span < kSymSpan && 2 * (p.span + 1) <= arrays && p.span * p.nb < 256;) ++p.span;
  return p;
}
// Where the launch that begins with item f ends: as many whole turns of the
// chip's workgroups as a d has, at most span d, at most one energy partial
// per item.
inline long long sym_launch_end(const SymPlan& p, long long f) {
  const long long chunk = std::min(kEnergyGrid, 256 * std::max(1, p.nb / 256));
  return std::min(std::min(f + chunk, (f / p.nb + p.span) * p.nb), p.items);
}

// Bytes of exchange lines in a cluster's workspace: those of its context's team.
inline size_t team_room(int n) {
  const Team t = make_team(n, kIPerLane, n, false);
  return t.wgs ? team_line_bytes(t) : 0;
}
// A pool's team t of n particles with g groups.
inline Team pool_team(Team t, int n, int n1, int g) {
  if (t.wp == 1) return t;  // (its steps need no exchange)
  t.g = g;
  t.wgs = t.wp * g;
  t.cap = std::min({(t.wgs << 14) / n, kTeamMaxCap, n1, (int)(team_room(n) / ((size_t)2 * t.wp * kTeamLine))});
  return t;
}

// Launch sizes for a context of n particles: enough workgroups for the
// largest force decomposition and corrector layout over all block sizes
// (sampled), capped; kernels loop over anything beyond the grid.
inline void launch_grids(int n, int ipl, int* force_grid, int* correct_grid) {
  long long fmax = 1, cmax = 1;
  const int step = n > 8192 ? n / 8192 : 1;
  for (int a = 1;; a += step) {
    if (a > n) a = n;
    const Plan p = make_plan(a, n, ipl);
    if (p.items > fmax) fmax = p.items;
    const long long lanes = (long long)a * correct_lanes(p.s);
    const long long wg = (lanes + kBlock - 1) / kBlock;
    if (wg > cmax) cmax = wg;
    if (a == n) break;
  }
  *force_grid = (int)(fmax < kForceGrid ? fmax : kForceGrid);
  *correct_grid = (int)(cmax < kCorrectGrid ? cmax : kCorrectGrid);
}

// ---------------------------------------------------------------------------
// Pools of independent clusters (continuous batching)
// ---------------------------------------------------------------------------
// A pool keeps up to kMaxPool clusters resident; one pool step advances every
// resident cluster by one of its own block steps, with one launch per phase
// (predict, force, correct) for all of them. The tables live in device memory
// at the head of the pool's arena.
constexpr int kMaxPool = 256;

struct PoolSlot {
  Dev d;
  Consts c;
  Team t;
};

// With teams, a replay of a pool is rounds of up to kPoolTeamSteps (or
// kPoolWideSteps) steps in the teams and one of every cluster's in the packed
// launches. All teams have to fit the chip (one workgroup per compute unit, by
// their LDS), and get as many groups as they have room for: with more of them a
// team takes larger steps, and fewer wait for the packed ones. 48 clusters of
// 256 to 8192 to t = 1/8 (one group for most of the time) took 87.9 ms without
// teams, 79.6 with 8 x (3 + 1) steps, 84.2 with 4 x (7 + 1) and 90.9 with
// 16 x (1 + 1). With more groups: 5 clusters of up to 8192 32.2 ms with one,
// 29.7 with four, 25.6 with 4 x (7 + 1) steps as well and 23.7 with 2 x
// (15 + 1); 24 of up to 4096 31.9, 29.7, 26.8 and 28.4; 12 of up to 8192 46.3,
// -, 37.6 and 40.8. (Rounds of a power of two of steps: the clusters' large
// blocks then fall into the packed launches together.)
constexpr int kPoolTeamSteps = 3;
constexpr int kPoolWideSteps = 7;  // with at least kPoolWide groups to a team (2: 24 of up to 8192 51.3 ms, 4: 48.5)
constexpr int kPoolWide = 4;
constexpr int kPoolTeamWgs = 256;
constexpr int kPoolTeamGroups = 8;

struct PoolTable {
  int count;                   // resident clusters
  int order[kMaxPool];         // slot index of each resident cluster
  int pred_off[kMaxPool + 1];  // prefix sum of the clusters' predictor blocks
  int team_off[kMaxPool + 1];  // prefix sum of the teams' workgroups
  int team_g[kMaxPool];        // their groups and largest steps (pool_team)
  int team_cap[kMaxPool];
};

// A cluster's block step as the pool predictor fixed it: block size, block
// time and decomposition (what the force and corrector otherwise read from
// the cluster's record).
struct PoolStep {
  long long t_next;
  int n_act;
  Plan plan;
};

// Work of each resident cluster in the current pool step (by table
// position), written by the pool predictor for the force and corrector
// launches: force items, corrector workgroups (0 once the cluster is done)
// and the step itself.
struct PoolWork {
  int force_n[kMaxPool];
  int correct_n[kMaxPool];
  PoolStep step[kMaxPool];
};

// Per-slot status gathered after each batch of pool steps.
struct PoolStatus {
  long long t_now, block_steps, particle_steps, pairs, clamps;
  int done, nonfinite;
};

// The small block steps that come next of every resident cluster, up to
// steps, in their teams.
hipError_t launch_pool_team(const PoolSlot* slots, const PoolTable* tab, int steps, bool mixed, hipStream_t s);
hipError_t launch_pool_step(const PoolSlot* slots, const PoolTable* tab, PoolWork* work, bool mixed,
                            hipStream_t s);
// Lagrange radii of the ascending fractions frac[0..n_frac) into out[0..n_frac),
// Eq. (5) into out[n_frac], the half-mass radius into out[n_frac + 1].
hipError_t launch_diagnostics(const Dev& d, const Consts& c, const double* frac, int n_frac,
                              double* out, hipStream_t s);
hipError_t launch_pool_status(const PoolSlot* slots, const PoolTable* tab, PoolStatus* out,
                              hipStream_t s);

// Launchers (gd_kernels.hip). Each returns the hipGetLastError() of its launch.
hipError_t launch_load(const Dev& d, const Consts& c, const double* m, const double* x,
                       const double* v, hipStream_t s);
hipError_t launch_predict(const Dev& d, const Consts& c, int mode, double t_explicit, hipStream_t s);
// ev_start/ev_stop (may be null): events that record the launch's own start
// and end (hipExtLaunchKernelGGL), for per-launch timing outside graphs.
hipError_t launch_force(const Dev& d, const Consts& c, hipStream_t s, hipEvent_t ev_start = nullptr,
                        hipEvent_t ev_stop = nullptr);
hipError_t launch_correct(const Dev& d, const Consts& c, hipStream_t s);
// The two kernels of a graph-replayed block step with parity par (see Sched).
hipError_t launch_step_force(const Dev& d, const Consts& c, int par, hipStream_t s,
                             hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
hipError_t launch_step_correct(const Dev& d, const Consts& c, int par, hipStream_t s);
// The small block steps that come next, up to kTeamSteps, in one launch; ends
// before a step of parity par, with its list prepared.
hipError_t launch_team(const Dev& d, const Consts& c, const Team& t, int par, hipStream_t s);
// Clears the exchange lines of a cluster of n particles and its part of the schedule record.
hipError_t launch_team_clear(const Dev& d, int n, hipStream_t s);
// Predicts every particle to the next block time and builds list 0 for it,
// so that a step of parity 0 finds its list prepared.
hipError_t launch_prepare(const Dev& d, const Consts& c, hipStream_t s);
// Copies the N_act of the step in flight (0 if it was skipped or rebuilt its
// list) to *out.
hipError_t launch_log_nact(const Dev& d, int* out, hipStream_t s);
hipError_t launch_init_dt(const Dev& d, const Consts& c, hipStream_t s);
// The force of every particle at t_now, its initial block step, and the energy
// (out as launch_energy's, the third 0): instead of launch_force,
// launch_init_dt and launch_energy.
hipError_t launch_sym_init(const Dev& d, const Consts& c, const SymPlan& p, double* out, hipStream_t s,
                           hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
hipError_t launch_reduce_out(const Dev& d, const Consts& c, double* acc, double* jerk, hipStream_t s);
// The force of an index list, and its outputs. d.sc null: no record of
// non-finite results is kept.
hipError_t launch_list_force(const Dev& d, const Consts& c, const ListArgs& a, hipStream_t s,
                             hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// out: 3 doubles (kinetic, potential, unsoftened potential), memory the GPU can
// write (the pinned result of the caller).
hipError_t launch_energy(const Dev& d, const Consts& c, int unsoft, double* out, hipStream_t s);
hipError_t launch_set_tend(const Dev& d, long long t_end, hipStream_t s);
hipError_t launch_reset_sched(const Dev& d, long long t_now, hipStream_t s);
hipError_t launch_copy_active(const Dev& d, const Consts& c, int32_t* idx, hipStream_t s);
hipError_t launch_get_state(const Dev& d, const Consts& c, double* x, double* v, double* a,
                            double* jerk, double* t_i, double* dt_i, hipStream_t s);
hipError_t launch_set_state(const Dev& d, const Consts& c, const double* x, const double* v,
                            const double* a, const double* jerk, const double* t_i,
                            const double* dt_i, long long t_now, hipStream_t s);

}  // namespace gd
