// Cell binning (counting sort into cell order) and Verlet-list construction
// (Sec. 1.4).  This translation unit is compiled with -ffp-contract=off: the
// wrap and the minimum-image distance are evaluated operation by operation,
// so the neighbour set equals the brute-force definition bit for bit.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "md_internal.h"

namespace {

// Per-atom kernels run 256-thread blocks, each covering 4 work tiles of 64
// atoms (one wavefront per tile).  Logical blocks are remapped per XCD; a block
// strides over logical blocks when the grid is capped.  FOR_ATOMS(i, T) runs
// its body for every atom i of the block's tiles (T the tile).
#define FOR_ATOMS(b, I, T, ...)                                               \
  do {                                                                        \
    const int _nlb = ((b).n_tiles + 3) / 4;                                   \
    const int _lane = threadIdx.x & (MD_WAVE - 1);                            \
    for (int _k = 0;; ++_k) {                                                 \
      const int _lb = md_remap_stride(_nlb, _k);                              \
      if (_lb >= _nlb) break;                                                 \
      const int _t = _lb * 4 + (int)(threadIdx.x / MD_WAVE);                  \
      if (_t >= (b).n_tiles) continue;                                        \
      const md_tile T = (b).tiles[_t];                                        \
      if (_lane >= T.count) continue;                                         \
      const int I = T.first + _lane;                                          \
      __VA_ARGS__                                                             \
    }                                                                         \
  } while (0)

__device__ __forceinline__ bool skip_rebuild(int mode, const md_ctl_dev* ctl) {
  return mode == MD_IF_FLAGGED && ctl->rebuild == 0;
}

__device__ __forceinline__ int cell_coord(double x, double lo, double inv_w, int nc) {
  double q = floor((x - lo) * inv_w);
  if (!(q >= 0.0)) return 0;  // also catches NaN
  if (q >= (double)nc) return nc - 1;
  return (int)q;
}

// ---------------------------------------------------------------------------
// 1. wrap, cell index, histogram.
// ---------------------------------------------------------------------------
// Lanes below this one in mask m.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// x wrapped into the box (x <- x - L floor((x - lo) / L); a result of lo + L goes to lo) and its
// cell; problems are added to bad.
__device__ __forceinline__ int wrap_and_cell(const md_domain& D, double4& p, int& bad) {
  double x[3] = {p.x, p.y, p.z};
  int c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (!isfinite(x[a])) bad |= MD_FLAG_NONFINITE;
    if (D.periodic[a]) {
      double y = x[a] - D.len[a] * floor((x[a] - D.lo[a]) / D.len[a]);
      if (y >= D.lo[a] + D.len[a]) y = D.lo[a];
      x[a] = y;
    } else if (x[a] < D.lo[a] || x[a] > D.lo[a] + D.len[a]) {
      bad |= MD_FLAG_WALL;
    }
    c[a] = cell_coord(x[a], D.lo[a], D.inv_w[a], D.nc[a]);
  }
  p.x = x[0];
  p.y = x[1];
  p.z = x[2];
  return D.cell_off + (c[0] * D.nc[1] + c[1]) * D.nc[2] + c[2];
}

// The wrapped positions, velocities and ids also go to their copies, from which the gather writes
// the sorted arrays: each atom's record is read and written twice.  With the gather writing the
// copies and a fifth launch copying them back (three times each) the three kernels that touch the
// records took 25 + 34 + 21 us for 640,000 atoms and 47 + 86 + 58 us for 2,048,000, now 34 + 26
// and 58 + 84 us.
__global__ __launch_bounds__(MD_ATOM_BLOCK) void k_bin_count(md_batch b, int mode,
                                                             const double4* pos, const double* vel,
                                                             const int* id, int* cell_of,
                                                             int* rank_of, int* counts,
                                                             double4* pos_s, double* vel_s,
                                                             int* id_s, md_ctl_dev* ctl) {
  // The rebuild decision: every block reduces the displacement maxima of the last
  // drift itself (no cross-block communication); block 0 publishes it for the
  // other rebuild kernels of this call.
  const bool go = mode == MD_ALWAYS || md_displacement_exceeded(ctl);
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->rebuild = go ? 1 : 0;
  if (!go) return;
  const int n = b.n_atoms;
  int bad = 0;
  FOR_ATOMS(b, i, T, {
    const md_domain& D = b.domains[T.rep];
    double4 p = pos[i];
    const double v0 = vel[i], v1 = vel[n + i], v2 = vel[2 * n + i];
    const int my = id[i];
    const int cell = wrap_and_cell(D, p, bad);
    pos_s[i] = p;
    vel_s[i] = v0;
    vel_s[n + i] = v1;
    vel_s[2 * n + i] = v2;
    id_s[i] = my;
    cell_of[i] = cell;
    // Histogram with one atomic per run of equal cells among the wavefront's atoms
    // (they are still nearly in cell order from the last rebuild), all runs' atomics
    // in one instruction; each atom keeps the slot it got, so the scatter needs no
    // atomics.  Slot order inside a cell is arbitrary here; the gather ranks by id.
    // The active lanes of a tile are lanes 0 .. count - 1.
    const int lane = threadIdx.x & (MD_WAVE - 1);
    const int prev = __shfl(cell, lane > 0 ? lane - 1 : 0, MD_WAVE);
    const unsigned long long leads = __builtin_amdgcn_ballot_w64(lane == 0 || prev != cell);
    const int start = 63 - __builtin_clzll(leads & ((2ull << lane) - 1));  // this run's first lane
    int base = 0;
    if (lane == start) {
      const unsigned long long later = leads & ~((2ull << lane) - 1);
      const int end = later ? __builtin_ctzll(later) : T.count;
      base = atomicAdd(&counts[cell], end - lane);
    }
    base = __shfl(base, start, MD_WAVE);
    rank_of[i] = base + (lane - start);
  });
  if (bad) md_flag(ctl, bad);
}

// 2. exclusive scan of the histogram into cell_start.  The counts are reset by the scatter, when
// no block reads them any more.
__device__ __forceinline__ int block_incl_scan(int v, int* s_w, int& total) {
  const int lane = threadIdx.x & (MD_WAVE - 1), w = threadIdx.x / MD_WAVE;
  const int nw = blockDim.x / MD_WAVE;
#pragma unroll
  for (int o = 1; o < MD_WAVE; o <<= 1) {
    const int t = __shfl_up(v, o, MD_WAVE);
    if (lane >= o) v += t;
  }
  if (lane == MD_WAVE - 1) s_w[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int q = 0; q < nw; ++q) {
      const int t = s_w[q];
      s_w[q] = run;
      run += t;
    }
    s_w[16] = run;
  }
  __syncthreads();
  v += s_w[w];
  total = s_w[16];
  __syncthreads();  // s_w is reused by the next call
  return v;
}

// A block per 1024 cells, each summing the counts before its own itself: one launch, no block
// waits for another.  For grids of at most MD_SCAN_DIRECT_MAX cells (the last block then reads
// 0.5 MB): 5 us for 37,000 cells, 7 us for 104,000.  One block scanning all cells, a run per
// thread, took 66 us for the first, three launches 15 us for the second.
#define MD_SCAN_DIRECT_MAX 131072
__global__ __launch_bounds__(1024) void k_scan_direct(int n_cells, int mode, const int* counts,
                                                       int* cell_start, md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  __shared__ int s_w[17];
  const int beg = blockIdx.x * 1024, k = beg + threadIdx.x;
  const int v = k < n_cells ? counts[k] : 0;
  int before = 0, carry, total;
  const int4* c4 = reinterpret_cast<const int4*>(counts);
#pragma unroll 4
  for (int q = threadIdx.x; q < beg / 4; q += 1024) {
    const int4 c = c4[q];
    before += c.x + c.y + c.z + c.w;
  }
  block_incl_scan(before, s_w, carry);
  const int incl = block_incl_scan(v, s_w, total);
  if (k < n_cells) cell_start[k] = carry + incl - v;
  if (k == n_cells - 1) {
    cell_start[n_cells] = carry + total;
    ctl->n_rebuilds += 1;
  }
}

// Larger grids: contiguous segments of cells, one 1024-thread block each: segment sums, one
// block scanning the sums, then each block scanning its segment from its offset.
__global__ __launch_bounds__(1024) void k_scan_sums(int n_cells, int seg, int mode,
                                                     const int* counts, int* bsum,
                                                     md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  __shared__ int s_w[17];
  const int beg = blockIdx.x * seg, end = min(n_cells, beg + seg);
  int v = 0;
  for (int k = beg + threadIdx.x; k < end; k += blockDim.x) v += counts[k];
  int total;
  block_incl_scan(v, s_w, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_top(int nb, int n_cells, int mode, int* bsum,
                                                    int* cell_start, md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  __shared__ int s_w[17];
  const int t = threadIdx.x;
  const int v = t < nb ? bsum[t] : 0;
  int total;
  const int incl = block_incl_scan(v, s_w, total);
  if (t < nb) bsum[t] = incl - v;
  if (t == 0) {
    cell_start[n_cells] = total;
    ctl->n_rebuilds += 1;
  }
}

__global__ __launch_bounds__(1024) void k_scan_apply(int n_cells, int seg, int mode, const int* counts,
                                                      const int* bsum, int* cell_start,
                                                      md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  __shared__ int s_w[17];
  const int beg = blockIdx.x * seg, end = min(n_cells, beg + seg);
  int carry = bsum[blockIdx.x];
  for (int c0 = beg; c0 < end; c0 += blockDim.x) {
    const int k = c0 + threadIdx.x;
    const int v = k < end ? counts[k] : 0;
    int total;
    const int incl = block_incl_scan(v, s_w, total);
    if (k < end) cell_start[k] = carry + incl - v;
    carry += total;
  }
}

// 3. scatter atom indices (and their ids) into their cell segments, at the slots
//    the histogram handed out, and reset the histogram.
__global__ __launch_bounds__(MD_ATOM_BLOCK) void k_bin_scatter(md_batch b, int mode,
                                                               const int* cell_of,
                                                               const int* rank_of,
                                                               const int* cell_start,
                                                               const int* id, int* src, int* sid,
                                                               int* counts,
                                                               const md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  FOR_ATOMS(b, i, T, {
    const int dst = cell_start[cell_of[i]] + rank_of[i];
    src[dst] = i;
    sid[dst] = id[i];
  });
  for (int k = blockIdx.x * MD_ATOM_BLOCK + threadIdx.x; k < b.n_cells;
       k += gridDim.x * MD_ATOM_BLOCK)
    counts[k] = 0;
}

// 4. order each cell by atom id (rank sort inside the cell segment) and gather the atom records
//    from their copies; the positions become the displacement reference.
__global__ __launch_bounds__(MD_ATOM_BLOCK) void k_bin_gather(
    md_batch b, int mode, const int* cell_of, const int* cell_start, const int* src,
    const int* sid, const double4* pos_s, const double* vel_s, double4* pos, double* vel,
    int* id, double* pos_ref, md_ctl_dev* ctl) {
  if (skip_rebuild(mode, ctl)) return;
  const int n = b.n_atoms;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->n_dmax = 0;      // displacements now measured afresh
    ctl->rec_stale = 1;   // atoms reordered: carried-over neighbour records are void
  }
  FOR_ATOMS(b, slot, T, {
    const int a = src[slot];
    const double4 p = pos_s[a];
    const double v0 = vel_s[a], v1 = vel_s[n + a], v2 = vel_s[2 * n + a];
    const int c = cell_of[a];
    const int beg = cell_start[c], end = cell_start[c + 1];
    const int my = sid[slot];
    int rank = 0;  // ids are unique: the rank by id is a permutation of the segment
    for (int k = beg; k < end; ++k) rank += sid[k] < my;
    const int dst = beg + rank;
    pos[dst] = p;
    vel[dst] = v0;
    vel[n + dst] = v1;
    vel[2 * n + dst] = v2;
    id[dst] = my;
    pos_ref[dst] = p.x;
    pos_ref[n + dst] = p.y;
    pos_ref[2 * n + dst] = p.z;
  });
}

// Steps 1 to 4 in one block for small batches (atoms in registers, 4 tiles per wavefront;
// histogram in LDS): one launch instead of four.  In a replayed graph 256 atoms take 6.3 us and 12.1
// by the four launches, 864 atoms 7.6 and 13.5, 2048 11.9 and 13.9, 2916 14.9 and 13.8, 4000 17.7
// and 13.2; a call that finds nothing to do (MD_IF_FLAGGED) costs 4.7 us per launch.  Hence up to
// 32 tiles, and up to 64 where the rebuild is conditional.
constexpr int SMALL_TILES = 64, SMALL_TILES_ALWAYS = 32, SMALL_CELLS = 4096;
__global__ __launch_bounds__(1024) void k_bin_small(md_batch b, int mode, double4* pos,
                                                    double* vel, int* id, double* pos_ref,
                                                    int* cell_start, md_ctl_dev* ctl) {
  constexpr int TW = SMALL_TILES / 16;  // tiles per wavefront
  __shared__ int s_cell[SMALL_CELLS];   // counts, then first slots
  __shared__ int s_id[SMALL_TILES * MD_WAVE];
  __shared__ int s_w[17];
  const bool go = mode == MD_ALWAYS || md_displacement_exceeded(ctl);
  if (threadIdx.x == 0) ctl->rebuild = go ? 1 : 0;
  if (!go) return;
  const int n = b.n_atoms, n_cells = b.n_cells;
  const int w = threadIdx.x / MD_WAVE, lane = threadIdx.x & (MD_WAVE - 1);
  for (int k = threadIdx.x; k < n_cells; k += 1024) s_cell[k] = 0;
  __syncthreads();
  double4 p[TW];
  double v[TW][3];
  int my[TW], cell[TW], slot[TW], bad = 0;
#pragma unroll
  for (int u = 0; u < TW; ++u) {
    const int t = w + 16 * u;
    cell[u] = -1;
    if (t >= b.n_tiles) continue;
    const md_tile T = b.tiles[t];
    if (lane >= T.count) continue;
    const int i = T.first + lane;
    p[u] = pos[i];
#pragma unroll
    for (int q = 0; q < 3; ++q) v[u][q] = vel[q * n + i];
    my[u] = id[i];
    cell[u] = wrap_and_cell(b.domains[T.rep], p[u], bad);
    slot[u] = atomicAdd(&s_cell[cell[u]], 1);
  }
  if (bad) md_flag(ctl, bad);
  __syncthreads();
  // exclusive scan: a run of cells per thread
  const int per = (n_cells + 1023) / 1024;
  const int beg = min(n_cells, (int)threadIdx.x * per), end = min(n_cells, beg + per);
  int mine = 0, total;
  for (int k = beg; k < end; ++k) mine += s_cell[k];
  int run = block_incl_scan(mine, s_w, total) - mine;
  for (int k = beg; k < end; ++k) {
    const int c = s_cell[k];
    s_cell[k] = run;
    cell_start[k] = run;
    run += c;
  }
  if (threadIdx.x == 0) {
    cell_start[n_cells] = total;
    ctl->n_rebuilds += 1;
    ctl->n_dmax = 0;      // displacements now measured afresh
    ctl->rec_stale = 1;   // atoms reordered: carried-over neighbour records are void
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TW; ++u)
    if (cell[u] >= 0) s_id[s_cell[cell[u]] + slot[u]] = my[u];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TW; ++u) {
    if (cell[u] < 0) continue;
    const int first = s_cell[cell[u]], last = cell[u] + 1 < n_cells ? s_cell[cell[u] + 1] : total;
    int dst = first;  // ids are unique: the rank by id is a permutation of the segment
    for (int k = first; k < last; ++k) dst += s_id[k] < my[u];
    pos[dst] = p[u];
#pragma unroll
    for (int q = 0; q < 3; ++q) vel[q * n + dst] = v[u][q];
    id[dst] = my[u];
    pos_ref[dst] = p[u].x;
    pos_ref[n + dst] = p[u].y;
    pos_ref[2 * n + dst] = p[u].z;
  }
}

// ---------------------------------------------------------------------------
// Verlet list (Sec. 1.4): the candidates of every atom of a cell are the atoms of
// the (de-duplicated) 3x3x3 block of cells around it, the same set for all atoms
// of the cell.  One block takes one cell: its four wavefronts stage the candidates in
// LDS together and then take the cell's atoms four at a time.  Lists are written in
// candidate order (stencil cell order, then cell order).
// ---------------------------------------------------------------------------
constexpr int CW = 4;                  // wavefronts per block
constexpr int CELL_BLOCK = CW * MD_WAVE;
constexpr int STRIDE_GRID = 8192;      // most blocks of k_build_strided
constexpr int GRID_CELLS = 1 << 23;    // most cells that get a block each
constexpr int SEG_MAX = 64;            // most candidates per four-lane segment (16 segments)
constexpr int LSLOT = 130;             // list slots per atom in LDS (a stride of 65 banks)

// LDS of a block besides the candidates.
struct CellLds {
  unsigned short list[CW][4 * LSLOT];      // the lists of a wavefront's four atoms, as candidates
  int beg[33];                             // cell_lists: stencil ranges' first candidates,
  unsigned start[32];                      // atoms and images
  // found by the first wavefront: runs of stencil cells that follow one another in memory with
  // one image (the z-neighbours where they do not wrap)
  int n_runs, C, own, a0, na, img, fixed, rep, out;
  int run_v[28], run_j[27];                // first candidate and first atom
  double run_off[27][3];                   // L k + cell centre
  double ctr[3], edge[3];                  // the cell's centre, 1.5 cell edges
};
// The candidates, in dynamic LDS for `seg` per segment: records {-2 u, |u|^2} by segment (rows
// of 4 mod 8 records, so that 64 lanes' reads meet no bank twice), then their atoms.  The FP64
// form keeps 64 positions per wavefront there.
static inline size_t candidate_lds(int seg) {
  return std::max<size_t>(16 * (seg + 4) * 16 + 16 * seg * 4, CW * 3 * MD_WAVE * sizeof(double));
}

// What a build only reads, in the constant address space: uniform reads are scalar loads also
// after stores (in the loop of k_build_strided).
#define MD_CONST __attribute__((address_space(4)))
using Domain = const md_domain MD_CONST;

using f32x4 = float __attribute__((ext_vector_type(4)));

// LDS written by this wavefront's other lanes is read next.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Stencil cell t (0..2) along one axis for an atom in cell c: the cell index, or -1
// when there is none (outside a non-periodic box, or a duplicate when nc < 3), and
// the image k = rint(d / L) that a candidate in it has (d = x_j - x_i): +1 for a
// cell reached by wrapping below 0, -1 by wrapping above nc - 1.
__device__ __forceinline__ int stencil_cell(int c, int t, int nc, int periodic, int& k) {
  k = 0;
  if (periodic && nc < 3) return t < nc ? t : -1;
  int q = c + t - 1;
  if (q < 0) {
    if (!periodic) return -1;
    q += nc;
    k = 1;
  } else if (q >= nc) {
    if (!periodic) return -1;
    q -= nc;
    k = -1;
  }
  return q;
}

struct Cand {
  double x, y, z;     // candidate position
  int j;              // candidate index
  unsigned image;     // of its stencil cell (image_code)
  bool valid;
};

// The images k of a stencil cell along the axes as a number below 27.  A range's first atom
// (below 2^27) and its image share a word: LDS beyond 20 KB would cost a block its place on the CU.
__device__ __forceinline__ unsigned image_code(const int (&k)[3]) {
  return (unsigned)((k[0] + 1) * 9 + (k[1] + 1) * 3 + k[2] + 1);
}
constexpr int IMAGE_BIT = 27;
static_assert(MD_MAX_ATOMS < 1 << IMAGE_BIT, "a range's first atom and its image share a word");

// Entry `slot` of atom ia: row slot / lanes, column ia * lanes + slot % lanes.
__device__ __forceinline__ int* entry(int* neigh, int ia, int slot, int lanes_log2,
                                      unsigned row) {
  const unsigned lanes = 1u << lanes_log2;
  return neigh + (size_t)ia * lanes + (size_t)((unsigned)slot >> lanes_log2) * row +
         ((unsigned)slot & (lanes - 1));
}

// Candidate c against atom k of the cell (position in s_p, index ia): with FIXED by its stencil
// cell's image (shift = L k), else with the minimum image per candidate.
template <bool FIXED>
__device__ __forceinline__ bool accept_pair(const Cand& c, const double (&shift)[3],
                                            double (*s_p)[MD_WAVE], int k, int ia,
                                            const double* len, const double* inv, const int* per,
                                            double rns2) {
  double dx = c.x - s_p[0][k], dy = c.y - s_p[1][k], dz = c.z - s_p[2][k];
  if (FIXED) {
    dx = dx - shift[0];
    dy = dy - shift[1];
    dz = dz - shift[2];
  } else {
    if (per[0]) dx = dx - len[0] * rint(dx * inv[0]);
    if (per[1]) dy = dy - len[1] * rint(dy * inv[1]);
    if (per[2]) dz = dz - len[2] * rint(dz * inv[2]);
  }
  const double r2 = (dx * dx + dy * dy) + dz * dz;
  return c.valid & (c.j != ia) & (r2 < rns2);
}

// v of lane `src` (all lanes on).
__device__ __forceinline__ int from_lane(int src, int v) {
  return __builtin_amdgcn_ds_bpermute(src << 2, v);
}

// Overflow flag and longest list of a wavefront's atoms.  The longest list is one word for all
// wavefronts: only those that raise it touch it with an atomic (one atomicMax per wavefront, all
// to one address, took 10 ns each one after the other and set the whole build's time: 118 us on
// 131k Cu atoms whatever the rest of the kernel did).
__device__ __forceinline__ void publish_counts(int lane, int over, int most, md_ctl_dev* ctl) {
  if (__any(over)) {
    if (lane == 0) md_flag(ctl, MD_FLAG_NEIGH_OVERFLOW);
  }
#pragma unroll
  for (int o = MD_WAVE / 2; o > 0; o >>= 1) most = max(most, from_lane(lane ^ o, most));
  if (lane == 0 &&
      most > __hip_atomic_load(&ctl->max_nneigh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&ctl->max_nneigh, most);
}

// The lists of a cell by FP64 tests: for cells with more candidates than a block stages (FIXED),
// and for grids whose cells hold several images of a pair (two cells on a periodic axis) and cells
// with positions outside their places, which take the minimum image of each candidate.  Bound by
// FP64 issue: by the stencil's images 131,072 Cu atoms at 7.8 A (1290 candidates) 217 us, at 9 A
// (2048) 306-332, by a rounding per candidate and axis 281 and 410; one wavefront per cell that
// loads its candidates once, with a same-address atomic, 251 and 490.
template <bool FIXED>
__device__ __forceinline__ void cell_lists(int lane, Domain& D, int a0, int na, int C,
                                           const int* s_beg, const unsigned* s_start,
                                           double (*s_p)[MD_WAVE],
                                           const double4* __restrict__ pos, int* neigh,
                                           int* nneigh, int max_neigh, int lanes_log2, int npad,
                                           double rns2, bool img, int& over, int& most) {
  const unsigned row = (unsigned)npad << lanes_log2;  // ints per list row
  double len[3], inv[3];
  int per[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    len[q] = D.len[q];
    inv[q] = D.inv_len[q];
    per[q] = D.periodic[q];
  }
  // candidate v of the flattened stencil: range r = the last with s_beg[r] <= v
  auto make = [&](int v) {
    Cand c;
    c.valid = v < C;
    int r = 0;
#pragma unroll
    for (int st = 16; st > 0; st >>= 1)
      if (s_beg[r + st] <= v) r += st;
    const unsigned range = s_start[r];
    c.j = c.valid ? (int)(range & ((1u << IMAGE_BIT) - 1)) + (v - s_beg[r]) : a0;
    const double4 q = pos[c.j];
    c.x = q.x;
    c.y = q.y;
    c.z = q.z;
    c.image = FIXED ? range >> IMAGE_BIT : 0u;
    return c;
  };
  for (int g0 = 0; g0 < na; g0 += MD_WAVE) {
    const int gc = min(MD_WAVE, na - g0);
    if (lane < gc) {
      const double4 q = pos[a0 + g0 + lane];
      s_p[0][lane] = q.x;
      s_p[1][lane] = q.y;
      s_p[2][lane] = q.z;
    }
    __builtin_amdgcn_wave_barrier();
    int tot = 0;  // lane k: accepted candidates of atom g0 + k so far
    Cand nx = make(lane);
    for (int v0 = 0; v0 < C; v0 += MD_WAVE) {
      const Cand c = nx;
      if (v0 + MD_WAVE < C) nx = make(v0 + MD_WAVE + lane);  // next chunk in flight
      double sh[3] = {0.0, 0.0, 0.0};
      if (FIXED) {
        const int kx = c.image / 9, ky = c.image / 3 % 3, kz = c.image % 3;
        sh[0] = (double)(kx - 1) * len[0];
        sh[1] = (double)(ky - 1) * len[1];
        sh[2] = (double)(kz - 1) * len[2];
      }
      // two atoms per trip: their distance chains overlap
      for (int k = 0; k < gc; k += 2) {
        const int k1 = min(k + 1, gc - 1);  // gc odd: the last trip tests atom k twice
        const bool ok0 = accept_pair<FIXED>(c, sh, s_p, k, a0 + g0 + k, len, inv, per, rns2);
        const bool ok1 = accept_pair<FIXED>(c, sh, s_p, k1, a0 + g0 + k1, len, inv, per, rns2) &&
                         k1 != k;
        const unsigned long long m0 = __builtin_amdgcn_ballot_w64(ok0);
        const unsigned long long m1 = __builtin_amdgcn_ballot_w64(ok1);
        const int base0 = __builtin_amdgcn_readlane(tot, k);
        const int base1 = __builtin_amdgcn_readlane(tot, k1);
        const int slot0 = base0 + lanes_below(m0), slot1 = base1 + lanes_below(m1);
        if (ok0 && slot0 < max_neigh)
          *entry(neigh, a0 + g0 + k, slot0, lanes_log2, row) = c.j;
        if (ok1 && slot1 < max_neigh)
          *entry(neigh, a0 + g0 + k1, slot1, lanes_log2, row) = c.j;
        tot = lane == k ? base0 + (int)__popcll(m0) : tot;
        tot = lane == k1 && k1 != k ? base1 + (int)__popcll(m1) : tot;
      }
    }
    if (lane < gc) {
      nneigh[a0 + g0 + lane] = (tot < max_neigh ? tot : max_neigh) | (img ? MD_NN_IMG : 0);
      over |= tot > max_neigh;
      most = max(most, tot);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// The value of a lane of the same group of four (CTRL: two bits per lane), and of the lane N
// below in the same row of 16 (0 if there is none).
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int N>
__device__ __forceinline__ int row_shr(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x110 + N, 0xF, 0xF, true);
}

// v / S for 0 <= v < 1024, 4 <= S <= 64 (the reciprocal is uniform).
__device__ __forceinline__ int segment_of(int v, int S) {
  return (int)((unsigned)v * (((1u << 20) + S - 1) / S) >> 20);
}

// The lists of four atoms of a cell by matrix instructions: squared distances
//   r_ij^2 - r_ns^2 = (|u_i|^2 - r_ns^2) + |u_j|^2 - 2 u_i . u_j
// (u relative to the cell's centre) of four candidates {-2 u_j, |u_j|^2} and the four atoms
// {u_i, 1} come from four v_mfma_f32_4x4x1 (16 such blocks at once), and the sign of each
// element decides its pair.  Lane 4 b + i takes atom i and the b-th of 16 equal segments of the
// candidates: it shifts the four signs it gets per step into bit masks and then lists its
// segment's accepted candidates one by one, its first slot being the number accepted in the
// segments below: candidate order, as from cell_lists.  The four lists are put together in LDS
// and written row by row.
//
// The decisions are those of the FP64 test, bit for bit.  With A = max |u_i|, a pair with
// |u_j| <= A + 1.05 r_ns is formed with an error of at most tau = 2^-20 ((2 A + 1.05 r_ns)^2 +
// r_ns^2) (inputs, norms and four accumulations, each within 2 x 2^-24 of the sum of
// magnitudes), and one farther out has r^2 - r_ns^2 > 0.09 r_ns^2, far more than its error.  If
// any element is within tau of zero (about 1 % of the four-atom groups of a thermal crystal),
// the group's accepted candidates, with tau added to r_ns^2, are tested again in FP64
// (accept_pair's operations: d - L k with the image k of the candidate's stencil cell).
__device__ __forceinline__ void atom_lists(int lane, Domain& D, int a0, int na, int t,
                                           int S, int own, CellLds& s,
                                           const float (*recs)[4], const int* cand, int w,
                                           const double4* __restrict__ pos, int* neigh,
                                           int* nneigh, int max_neigh, int lanes_log2,
                                           unsigned row, double rns2, bool img, int& over,
                                           int& most) {
  const int col = lane & 3, seg = lane >> 2;
  const int pad = (S & 4) ? 0 : 4;  // rows of 4 mod 8 records: the LDS reads meet no bank twice
  const int S1 = S + pad;
  const int ia = t + col;           // this lane's atom of the cell
  const float rns2f = (float)rns2;
  // the atom's own record, as a candidate
  float u[4] = {0.0f, 0.0f, 0.0f, 0.0f}, cv = 1e30f, a2 = 0.0f;
  const int v_own = own + min(ia, na - 1);
  if (ia < na) {
    const f32x4 q = *reinterpret_cast<const f32x4*>(recs[v_own + pad * segment_of(v_own, S)]);
#pragma unroll
    for (int k = 0; k < 3; ++k) u[k] = -0.5f * q[k];
    u[3] = 1.0f;
    a2 = q[3];
    cv = a2 - rns2f;
  }
  a2 = fmaxf(a2, __int_as_float(quad_perm<0xB1>(__float_as_int(a2))));
  a2 = fmaxf(a2, __int_as_float(quad_perm<0x4E>(__float_as_int(a2))));
  const float reach = 2.0f * __builtin_amdgcn_sqrtf(a2) + 1.05f * __builtin_amdgcn_sqrtf(rns2f);
  const float tau = 9.6e-7f * (reach * reach + rns2f);  // (2^-20, rounded up)
  // signs of the segment's two parts (first candidate in the highest bit), and the least
  // magnitude, with cv as the part of the distance that the atom contributes
  const int H[2] = {((S / 2) + 3) & ~3, S - (((S / 2) + 3) & ~3)};
  unsigned m[2];
  auto signs = [&](float c) {
    float least = 1e30f;
    m[0] = m[1] = 0u;
    const float(*rec)[4] = recs + seg * S1 + col;
    auto step = [&](int h, int q) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(rec[q + h * H[0]]);
      f32x4 d = {c, c, c, c};
#pragma unroll
      for (int k = 0; k < 4; ++k) d = __builtin_amdgcn_mfma_f32_4x4x1f32(a[k], u[k], d, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        m[h] = __builtin_amdgcn_alignbit(m[h], __float_as_uint(d[e]), 31);
        least = __builtin_amdgcn_fmed3f(fabsf(d[e]), least, 0.0f);  // the smaller
      }
    };
    int q = 0;
#pragma unroll 2
    for (; q < H[1]; q += 4) {
      step(0, q);
      step(1, q);
    }
    if (q < H[0]) step(0, q);
    m[0] <<= 32 - H[0];
    m[1] = H[1] ? m[1] << (32 - H[1]) : 0u;
    return least;
  };
  const float least = signs(cv);
  const int v0 = seg * S;
  const int self = v_own - v0;  // the atom itself is no neighbour of its own
  auto drop_self = [&]() {
    if (self >= 0 && self < H[0]) m[0] &= ~(0x80000000u >> self);
    if (self >= H[0] && self < S) m[1] &= ~(0x80000000u >> (self - H[0]));
  };
  if (__any(!(least >= tau))) {
    signs(cv - tau);
    drop_self();
    const double4 pi = pos[a0 + min(ia, na - 1)];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      unsigned left = m[h];
      while (left) {
        const int z = __clz(left);
        const unsigned bit = 0x80000000u >> z;
        left ^= bit;
        const int v = v0 + h * H[0] + z;
        const f32x4 r = *reinterpret_cast<const f32x4*>(recs[v + pad * seg]);
        const double4 q = pos[cand[v]];
        const double x[3] = {q.x, q.y, q.z}, xi[3] = {pi.x, pi.y, pi.z};
        double d[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          // x_j - L k = centre + u: the image is what the record was staged with
          const double im = rint(((x[k] - s.ctr[k]) + 0.5 * (double)r[k]) * D.inv_len[k]);
          d[k] = (x[k] - xi[k]) - im * D.len[k];
        }
        const double r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
        if (!(r2 < rns2)) m[h] ^= bit;
      }
    }
  } else {
    drop_self();
  }
  // slots: the segments' counts in turn
  const int n0 = __popc(m[0]), mine = n0 + __popc(m[1]);
  // (within the four rows of 16 lanes, then across them)
  int incl = mine;
  incl += row_shr<4>(incl);
  incl += row_shr<8>(incl);
  const int r0 = from_lane(12 + col, incl), r1 = from_lane(28 + col, incl);
  const int r2 = from_lane(44 + col, incl), r3 = from_lane(60 + col, incl);
  incl += (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
  const int tot = r0 + r1 + r2 + r3;
  // the two parts side by side, an entry of each per trip
  const int lim = min(LSLOT, max_neigh);
  unsigned short* list = s.list[w];
  int slot[2] = {incl - mine, incl - mine + n0};
  wave_sync();
  if (!__any(tot > lim)) {
    unsigned short* to[2] = {list + col * LSLOT + slot[0], list + col * LSLOT + slot[1]};
    while (m[0] | m[1]) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (m[h] != 0u) {
          const int z = __builtin_clz(m[h]);
          *to[h]++ = (unsigned short)(v0 + h * H[0] + z);
          m[h] &= 0x7fffffffu >> z;
        }
      }
    }
  } else {  // entries past the LDS slots go straight to memory, those past max_neigh nowhere
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      for (; m[h] != 0u; ++slot[h]) {
        const int z = __builtin_clz(m[h]), v = v0 + h * H[0] + z;
        m[h] &= 0x7fffffffu >> z;
        if (slot[h] < lim) list[col * LSLOT + slot[h]] = (unsigned short)v;
        else if (slot[h] < max_neigh) *entry(neigh, a0 + ia, slot[h], lanes_log2, row) = cand[v];
      }
    }
  }
  wave_sync();
  if (lane < 4 && ia < na) {
    nneigh[a0 + ia] = (tot < max_neigh ? tot : max_neigh) | (img ? MD_NN_IMG : 0);
    over |= tot > max_neigh;
    most = max(most, tot);
  }
  // rows: the four atoms' entries of a row are contiguous; a lane keeps its place in the row
  // (W = 4 lanes ints, a divisor of 64) and steps over rows
  const int W = 4 << lanes_log2, c = lane & (W - 1), i = c >> lanes_log2;
  const int last = from_lane(i, min(ia < na ? tot : 0, lim));
  int q = lane / W, at = (q << lanes_log2) + (c & ((1 << lanes_log2) - 1));
  const int step = MD_WAVE / W;
  int* to = neigh + ((size_t)(a0 + t) << lanes_log2) + (size_t)q * row + c;
  for (; at < last; at += step << lanes_log2, to += (size_t)step * row)
    *to = cand[list[i * LSLOT + at]];
  wave_sync();
}

// The lists of one cell, by a block.  The fixed image of a stencil cell is the minimum image of every pair
// that can be closer than r_ns when each periodic axis has at least three cells of edge w >
// r_ns, the cell's own atoms lie within w / 2 of its centre and every candidate's image within
// 1.5 w of it per axis: the other images are then 3 w - 2 w > r_ns away or farther.  Both are
// checked while staging (not so if positions changed since the binning, left a wall or are not
// finite).
// Cells for which either fails, or with more candidates than LDS holds, take the FP64 form,
// their atoms shared among the wavefronts; by the fixed images too where only the LDS lacks.
//
// Bound by latency: of 66 us for 131k Cu atoms (78 of 515 candidates accepted per atom, 41
// MB of lists, an 8 us write) the vector units are busy for 46; finding the runs takes about 20,
// the staging 10, the tests 20 and the entries the rest, much of it overlapped by the eight
// blocks of a CU (59 VGPRs; 20 KB of LDS each at 640 candidates).  Before: one wavefront per cell
// testing 64 candidates against one atom at a time in FP64, 118-126 us (98 us without its
// same-address atomics, see publish_counts); 864,000 argon atoms 305 us, 551 before.  Measured at
// 69 us for the Cu build: entries stored one by one as they are found (scattered words,
// 11 per instruction) took 44 us of such a build, and 16 atoms per matrix instruction (two
// groups for the 19 atoms of a cell, the second nearly empty) left the lanes a fifth full while
// listing: 114 us; three wavefronts per block 76 us, two 78, five 88.
__device__ __forceinline__ void build_cell(Domain* domains, int n_rep, int cell, int tid,
                                           CellLds& s, double* s_dyn,
                                           const double4* __restrict__ pos,
                                           const int* __restrict__ cell_start, int* neigh,
                                           int* nneigh, int max_neigh, int lanes_log2, int npad,
                                           double rns2, int seg, md_ctl_dev* ctl) {
  float(*recs)[4] = reinterpret_cast<float(*)[4]>(s_dyn);
  int* cand = reinterpret_cast<int*>(recs + 16 * (seg + 4));
  const int w = __builtin_amdgcn_readfirstlane(tid / MD_WAVE);
  const int lane = tid & (MD_WAVE - 1);
  if (w == 0) {
    const int MD_CONST* range = (const int MD_CONST*)cell_start + cell;
    const int a0 = range[0], na = range[1] - a0;
    // the box of this cell: the last domain whose cells start at or before it
    int lo = 0, hi = n_rep - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (domains[mid].cell_off <= cell) lo = mid; else hi = mid - 1;
    }
    Domain& D = domains[lo];
    const int local = cell - D.cell_off;
    const int cc[3] = {local / (D.nc[2] * D.nc[1]), (local / D.nc[2]) % D.nc[1], local % D.nc[2]};
    // lane t < 27 takes stencil cell (t / 9, t / 3 % 3, t % 3): its atom range and image
    int cnt = 0, start = 0, k[3] = {0, 0, 0};
    if (lane < 27) {
      const int qx = stencil_cell(cc[0], lane / 9, D.nc[0], D.periodic[0], k[0]);
      const int qy = stencil_cell(cc[1], (lane / 3) % 3, D.nc[1], D.periodic[1], k[1]);
      const int qz = stencil_cell(cc[2], lane % 3, D.nc[2], D.periodic[2], k[2]);
      if (qx >= 0 && qy >= 0 && qz >= 0) {
        const int q = D.cell_off + (qx * D.nc[1] + qy) * D.nc[2] + qz;
        start = cell_start[q];
        cnt = cell_start[q + 1] - start;
      }
    }
    // exclusive prefix of the range sizes over the lanes
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const int u = from_lane(lane - o, incl);
      if (lane >= o) incl += u;
    }
    const int C = __builtin_amdgcn_readlane(incl, 31);
    const int beg = incl - cnt;
    // the block wraps (image flag for the force passes)
    bool img = false, fixed = true;
    double off[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      double width = __builtin_amdgcn_rcp(D.inv_w[q]);  // 1 / inv_w, refined once
      width = fma(width, fma(-D.inv_w[q], width, 1.0), width);
      const double ctr = D.lo[q] + (cc[q] + 0.5) * width;
      off[q] = (double)k[q] * D.len[q] + ctr;
      if (lane == 0) {
        s.ctr[q] = ctr;
        s.edge[q] = 1.5 * width * (1.0 + 1e-6);
      }
      if (D.periodic[q]) {
        img |= (D.nc[q] < 3) || cc[q] == 0 || cc[q] == D.nc[q] - 1;
        // two cells hold both images of a pair; cells no wider than r_ns leave none to rounding
        fixed &= D.nc[q] >= 3 && width * width > rns2 * (1.0 + 1e-4);
      }
    }
    const int key = (int)image_code(k);
    // (both exchanges before any test: a shuffle from a lane that && switched off reads 0)
    const int prev_end = from_lane(lane - 1, start + cnt), prev_key = from_lane(lane - 1, key);
    const bool joins = lane > 0 && lane < 27 && prev_end == start && prev_key == key;
    const unsigned long long heads = __builtin_amdgcn_ballot_w64(lane < 27 && !joins);
    if (lane < 27 && !joins) {
      const int r = lanes_below(heads);
      s.run_v[r] = beg;
      s.run_j[r] = start;
#pragma unroll
      for (int q = 0; q < 3; ++q) s.run_off[r][q] = off[q];
    }
    if (lane < 32) {
      s.beg[lane] = lane < 27 ? beg : C;
      s.start[lane] = (unsigned)start | image_code(k) << IMAGE_BIT;
    }
    if (lane == 13) s.own = beg;
    if (lane == 0) {
      s.beg[32] = C;
      s.n_runs = (int)__popcll(heads);
      s.run_v[(int)__popcll(heads)] = C;
      s.C = C;
      s.a0 = a0;
      s.na = na;
      s.img = img;
      s.fixed = fixed;
      s.out = 0;  // a candidate outside its place
      s.rep = lo;
    }
  }
  __syncthreads();
  auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int na = uniform(s.na);
  if (na == 0) return;
  const int a0 = uniform(s.a0), C = uniform(s.C);
  Domain& D = domains[uniform(s.rep)];
  const bool img = uniform(s.img) != 0;
  bool fixed = uniform(s.fixed) != 0;
  int over = 0, most = 0;
  const bool staged = fixed && C <= 16 * seg;
  const int S = (C + 63) / 64 * 4;  // candidates per segment
  if (fixed) {
    const int pad = (S & 4) ? 0 : 4, n_runs = uniform(s.n_runs);
    const double ex = s.edge[0], ey = s.edge[1], ez = s.edge[2];
    bool bad = false;
    auto visit = [&](auto store) {
      for (int r = w; r < n_runs; r += CW) {
        const int v0 = uniform(s.run_v[r]), n = uniform(s.run_v[r + 1]) - v0;
        const int j0 = uniform(s.run_j[r]);
        const double ox = s.run_off[r][0], oy = s.run_off[r][1], oz = s.run_off[r][2];
        for (int q = lane; q < n; q += MD_WAVE) {
          const double4 p = pos[j0 + q];
          const double ux = p.x - ox, uy = p.y - oy, uz = p.z - oz;
          const double m = (unsigned)(j0 + q - a0) < (unsigned)na ? 3.0 : 1.0;  // the cell's own
          bad |= !(m * fabs(ux) <= ex && m * fabs(uy) <= ey && m * fabs(uz) <= ez);
          if constexpr (decltype(store)::value) {
            const float x = (float)ux, y = (float)uy, z = (float)uz;
            const int v = v0 + q;
            *reinterpret_cast<f32x4*>(recs[v + pad * segment_of(v, S)]) =
                f32x4{-2.0f * x, -2.0f * y, -2.0f * z, x * x + y * y + z * z};
            cand[v] = j0 + q;
          }
        }
      }
    };
    if (staged) {
      visit(std::true_type{});
      for (int v = C + tid; v < 16 * S; v += CELL_BLOCK)  // past the last: far away
        *reinterpret_cast<f32x4*>(recs[v + pad * segment_of(v, S)]) =
            f32x4{0.0f, 0.0f, 0.0f, 1e30f};
    } else {
      visit(std::false_type{});
    }
    if (__any(bad) && lane == 0) s.out = 1;
    __syncthreads();
    fixed = s.out == 0;
  }
  if (fixed && staged) {
    const int own = uniform(s.own);
    for (int t = 4 * w; t < na; t += 4 * CW)
      atom_lists(lane, D, a0, na, t, S, own, s, recs, cand, w, pos, neigh, nneigh, max_neigh,
                 lanes_log2, (unsigned)npad << lanes_log2, rns2, img, over, most);
  } else {
    const int per = (na + CW - 1) / CW, first = min(na, w * per), n = min(na, first + per) - first;
    auto lists = [&](auto fixed_tag) {
      cell_lists<decltype(fixed_tag)::value>(lane, D, a0 + first, n, C, s.beg, s.start,
                                             (double(*)[MD_WAVE])s_dyn + 3 * w, pos, neigh, nneigh,
                                             max_neigh, lanes_log2, npad, rns2, img, over, most);
    };
    if (n > 0) {
      if (fixed) lists(std::true_type{});
      else lists(std::false_type{});
    }
  }
  publish_counts(lane, over, most, ctl);
}

struct BuildArgs {
  md_batch b;
  int mode, max_neigh, lanes_log2, npad, seg, chunk, n_chunks;
  const double4* pos;
  const int* cell_start;
  int *neigh, *nneigh;
  double rns2;
  md_ctl_dev* ctl;
};

// A block per cell.
__global__ __launch_bounds__(CELL_BLOCK, 8) void k_build(BuildArgs A) {
  if (skip_rebuild(A.mode, A.ctl)) return;
  extern __shared__ double s_dyn[];
  __shared__ CellLds s;
  const int cell = md_remap_block(A.b.n_cells);
  if (cell >= A.b.n_cells) return;
  build_cell((Domain*)A.b.domains, A.b.n_rep, cell, threadIdx.x, s, s_dyn, A.pos, A.cell_start,
             A.neigh, A.nneigh, A.max_neigh, A.lanes_log2, A.npad, A.rns2, A.seg, A.ctl);
}

// The same with a limited grid: a block strides over chunks of up to 64 cells and takes the cells
// of a chunk that hold atoms one after the other.
//
// The arguments are read again for each cell and the thread index is made opaque: kept across the
// loop, addresses and lane indexes cost registers that the cell needs (18 spilled, 864,000 argon
// atoms 493 us; now as many registers as k_build, 342 us against its 305).
__global__ __launch_bounds__(CELL_BLOCK, 8) void k_build_strided(BuildArgs) {
  using Args = const BuildArgs MD_CONST;
  extern __shared__ double s_dyn[];
  __shared__ CellLds s;
  Args* ka = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
  if (skip_rebuild(ka->mode, ka->ctl)) return;
  for (int k = 0;; ++k) {
    const int at = md_remap_stride(ka->n_chunks, k), chunk = ka->chunk;
    if (at >= ka->n_chunks) break;
    const int first = at * chunk, last = min(first + chunk, ka->b.n_cells);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int c = first + (tid & (MD_WAVE - 1));
    const bool some = c < last && ka->cell_start[c + 1] > ka->cell_start[c];
    for (unsigned long long left = __builtin_amdgcn_ballot_w64(some); left; left &= left - 1) {
      const int cell = first + __builtin_ctzll(left);
      Args* a = ka;
      asm volatile("" : "+s"(a));
      asm volatile("" : "+v"(tid));
      build_cell((Domain*)a->b.domains, a->b.n_rep, cell, tid, s, s_dyn, a->pos, a->cell_start,
                 a->neigh, a->nneigh, a->max_neigh, a->lanes_log2, a->npad, a->rns2, a->seg, a->ctl);
      __syncthreads();  // the LDS is the next cell's
    }
  }
}

}  // namespace

extern "C" int md_bin_cells(const md_batch* b, md_rebuild_mode mode, double* pos, double* vel,
                            int* id, double* pos_ref, int* cell_start, void* ws, void* ctl,
                            void* stream) {
  if (!md_batch_ok(b) || !pos || !vel || !id || !pos_ref || !cell_start || !ws || !ctl)
    return MD_ERR_ARG;
  if (mode != MD_ALWAYS && mode != MD_IF_FLAGGED) return MD_ERR_ARG;
  if (b->n_atoms == 0) return MD_OK;
  const md_ws_layout L = md_ws_plan(b);
  char* w = (char*)ws;
  int* cell_of = (int*)(w + L.cell_of);
  int* rank_of = (int*)(w + L.rank);
  int* src = (int*)(w + L.src);
  int* sid = (int*)(w + L.sid);
  int* counts = (int*)(w + L.counts);
  double4* pos_s = (double4*)(w + L.pos_s);
  double* vel_s = (double*)(w + L.vel_s);
  int* id_s = (int*)(w + L.id_s);
  md_ctl_dev* c = (md_ctl_dev*)ctl;
  hipStream_t st = (hipStream_t)stream;
  if (b->n_tiles <= (mode == MD_ALWAYS ? SMALL_TILES_ALWAYS : SMALL_TILES) &&
      b->n_cells <= SMALL_CELLS) {
    MD_LAUNCH_TIMED(MD_KERNEL_BIN_COUNT, k_bin_small, dim3(1), dim3(1024), 0, st, *b, (int)mode,
                    (double4*)pos, vel, id, pos_ref, cell_start, c);
    MD_LAUNCH_CHECK();
    return MD_OK;
  }
  const dim3 grid(md_atom_grid(b->n_tiles)), block(MD_ATOM_BLOCK);
  MD_LAUNCH_TIMED(MD_KERNEL_BIN_COUNT, k_bin_count, grid, block, 0, st, *b, (int)mode,
                  (const double4*)pos, vel, id, cell_of, rank_of, counts, pos_s, vel_s, id_s, c);
  MD_LAUNCH_CHECK();
  if (b->n_cells <= MD_SCAN_DIRECT_MAX) {
    hipLaunchKernelGGL(k_scan_direct, dim3((b->n_cells + 1023) / 1024), dim3(1024), 0, st,
                       b->n_cells, (int)mode, counts, cell_start, c);
    MD_LAUNCH_CHECK();
  } else {
    const int nb = std::min(MD_SCAN_BLOCKS, (b->n_cells + 1023) / 1024);
    const int seg = (b->n_cells + nb - 1) / nb;
    int* bsum = (int*)(w + L.scan);
    hipLaunchKernelGGL(k_scan_sums, dim3(nb), dim3(1024), 0, st, b->n_cells, seg, (int)mode,
                       counts, bsum, c);
    MD_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, nb, b->n_cells, (int)mode, bsum,
                       cell_start, c);
    MD_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(1024), 0, st, b->n_cells, seg, (int)mode,
                       counts, bsum, cell_start, c);
    MD_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_bin_scatter, grid, block, 0, st, *b, (int)mode, cell_of, rank_of,
                     cell_start, id_s, src, sid, counts, c);
  MD_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_bin_gather, grid, block, 0, st, *b, (int)mode, cell_of, cell_start, src,
                     sid, pos_s, vel_s, (double4*)pos, vel, id, pos_ref, c);
  MD_LAUNCH_CHECK();
  return MD_OK;
}

extern "C" int md_build_neighbors(const md_batch* b, md_rebuild_mode mode, const double* pos,
                                  const int* cell_start, const md_nlist* nl, void* ctl,
                                  void* stream) {
  if (!md_batch_ok(b) || !pos || !cell_start || !nl || !nl->neigh || !nl->nneigh || !ctl)
    return MD_ERR_ARG;
  if (mode != MD_ALWAYS && mode != MD_IF_FLAGGED) return MD_ERR_ARG;
  int lg = -1;
  for (int k = 0; k <= 4; ++k)
    if (nl->lanes == (1 << k)) lg = k;
  if (lg < 0 || nl->max_neigh < nl->lanes || nl->max_neigh % nl->lanes) return MD_ERR_ARG;
  if (!(b->r_ns > 0.0)) return MD_ERR_ARG;
  if (b->n_atoms == 0) return MD_OK;
  // LDS for 1.2 times the average number of candidates, at least 640 (eight blocks then share a
  // CU) and at most 1024; cells with more take the FP64 form.  1.6 times in a batch of several
  // boxes, whose cells may differ more: 64 cubes of 4^3 to 12^3 cells at several densities (182,276
  // atoms, 365 to 1690 candidates, 542 on average) take 104 us, 141 at 1.2 times; over a wider
  // range of densities 141 and 247.  Equal boxes pay for it with 3 to 5 % (16 of 8,788 atoms
  // 75 and 72 us, 512 of 500 atoms 120 and 114): the host does not know the boxes.
  const double avg = 27.0 * b->n_atoms / b->n_cells;
  const double room = b->n_rep > 1 ? 1.6 : 1.2;
  const int seg = std::min(SEG_MAX, std::max(40, (int)(room * avg / 16.0 + 4.0) / 4 * 4));
  BuildArgs A{*b, (int)mode, nl->max_neigh, lg, md_npad(b->n_atoms), seg, 1, 0, (const double4*)pos,
              cell_start, nl->neigh, nl->nneigh, b->r_ns * b->r_ns, (md_ctl_dev*)ctl};
  const dim3 block(CELL_BLOCK);
  const hipStream_t st = (hipStream_t)stream;
  // A block per cell, or 8192 blocks that take the cells in turn.  Rebuilds that may find nothing
  // to do: a block per cell costs 9.6 us then for 36,000 cells and 24.6 for 107,000, the strided
  // form 3.6 and 3.7 (and 263 against 236 us where 640,000 Al atoms are rebuilt: half a round of
  // blocks is left over).  Grids of fewer atoms than cells: 125,000 cells with 0.5, 1 and 2 atoms
  // each take 216, 267 and 317 us by a block per cell and 167, 256 and 340 by the strided form,
  // 8.4 million cells with 100,000 atoms 8600 and 311 us.  And a launch holds less than 2^32
  // threads: 2^24 blocks.
  if (b->n_cells > STRIDE_GRID &&
      (mode == MD_IF_FLAGGED || b->n_atoms < b->n_cells || b->n_cells > GRID_CELLS)) {
    A.chunk = std::min(MD_WAVE, (b->n_cells + STRIDE_GRID - 1) / STRIDE_GRID);
    A.n_chunks = (b->n_cells + A.chunk - 1) / A.chunk;
    MD_LAUNCH_TIMED(MD_KERNEL_BUILD, k_build_strided,
                    dim3(std::min(STRIDE_GRID, md_grid_blocks(A.n_chunks))), block,
                    candidate_lds(seg), st, A);
  } else {
    MD_LAUNCH_TIMED(MD_KERNEL_BUILD, k_build, dim3(md_grid_blocks(b->n_cells)), block,
                    candidate_lds(seg), st, A);
  }
  MD_LAUNCH_CHECK();
  return MD_OK;
}
