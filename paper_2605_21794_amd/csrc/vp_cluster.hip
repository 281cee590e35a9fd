// HIP kernels (gfx950) for the decorated-particle initialisation of arXiv 2605.21794,
// Algorithm 1 ("Decorated Particle Initialization") with the periodic moments of the torus
// subsection: k-means of marker particles in (q, p), then one decorated particle per
// non-empty cluster.
//
// Design:
//  * nearest centre: the centres are binned into a uniform (q, p) grid of about one centre
//    per cell (rebuilt every iteration) and copied in cell order, so the cells of one grid
//    row are one contiguous run of centres; each marker searches its own cell and the ring
//    around it, leaves out the cells that lie farther than its best distance (from its previous
//    centre at first), and goes on, grid row by grid row, only if that distance reaches beyond
//    the ring.  The result is the exact nearest centre, ties to the lowest centre index, whatever order the cells
//    list their centres in.
//  * labels: the centres are renumbered once, in the cell order of their starting markers, so
//    that markers which are neighbours in the visiting order count on, and read, neighbouring
//    clusters.  Ties and outputs go by the caller's numbering (origid).
//  * per-cluster sums: every cluster's members are summed in increasing marker order by one
//    thread, so the sums are those of a sequential pass over the markers, bit for bit, and the
//    centres, the assignments and the moments are reproducible run to run.  Members are
//    gathered into segments by counting, in any order, and put in marker order in LDS
//    (k_group), or, for large clusters, by a stable radix sort of all marker indices.
//  * every index that reaches memory is clamped or counted exactly: cell coordinates are
//    clamped into the grid, group positions come from exact integer counts.

#include "vp_internal.h"

#include <mutex>

#include <math.h>

namespace vpk {

namespace {

constexpr double kTwoPi = 6.283185307179586;

// Cells of the search grid per centre over the markers' bounding box (1.5, 2 and 3: whole calls
// 2 to 25% slower, with more empty cells to read the bounds of).
constexpr double kCellsPerCentre = 1.0;

struct Grid {
  int gx, gp;
  double sx, sp, pmin;  // cell width in q, height in p, lower edge in p
};

__device__ __forceinline__ int grid_cell(const Grid& g, double q, double p, int* cx, int* cy) {
  double fx = floor(q / g.sx);
  double fy = floor((p - g.pmin) / g.sp);
  int x = !(fx >= 0.0) ? 0 : (fx >= (double)(g.gx - 1) ? g.gx - 1 : (int)fx);
  int y = !(fy >= 0.0) ? 0 : (fy >= (double)(g.gp - 1) ? g.gp - 1 : (int)fy);
  *cx = x;
  *cy = y;
  return y * g.gx + x;
}

// A marker as the passes visit it: in cell order, 32 bytes, so that placing one and fetching one
// out of order each touch a single 32-byte sector (as four arrays they touched four).
struct alignas(32) Marker {
  double q, p, w;
  int id;  // marker index (position in the batch)
  int pad;
};

// ---------------------------------------------------------------- small helpers
__global__ void k_fill_int(int* p, long long n, int v) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Per-block min / max of p (the markers' velocity range), then one block folds them.
__global__ __launch_bounds__(256) void k_minmax_partial(const double* __restrict__ p, long long m,
                                                        double* __restrict__ part) {
  __shared__ double smin[256], smax[256];
  double lo = INFINITY, hi = -INFINITY;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    const double v = p[i];
    lo = fmin(lo, v);
    hi = fmax(hi, v);
  }
  smin[threadIdx.x] = lo;
  smax[threadIdx.x] = hi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = smin[0];
    part[2 * blockIdx.x + 1] = smax[0];
  }
}

__global__ __launch_bounds__(256) void k_minmax_final(const double* __restrict__ part, int nb,
                                                      double* __restrict__ out) {
  __shared__ double smin[256], smax[256];
  double lo = INFINITY, hi = -INFINITY;
  for (int i = threadIdx.x; i < nb; i += 256) {
    lo = fmin(lo, part[2 * i]);
    hi = fmax(hi, part[2 * i + 1]);
  }
  smin[threadIdx.x] = lo;
  smax[threadIdx.x] = hi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = smin[0];
    out[1] = smax[0];
  }
}

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_incl(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  return v;
}

// Exclusive sum over the 1024 threads of a workgroup (*total: the whole sum); wt: 16 ints of
// LDS, free again after the caller's next barrier.
__device__ __forceinline__ int block_excl(int v, int* wt, int* total) {
  const int incl = wave_incl(v), w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) wt[w] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int x = wt[i];
    before += i < w ? x : 0;
    all += x;
  }
  *total = all;
  return before + incl - v;
}

// Exclusive scans of n ints into out[0..n] (out[n] = total).  Each thread takes PER consecutive
// ints.  ZERO: the counters are cleared once read, so the next count starts from zero without a
// fill of its own.
// One launch up to kScanOne ints (one workgroup); above, tile sums and then every tile scanned
// on its own, offset by the sums before it: each workgroup adds those itself while there are
// at most kScanSelf tiles (a handful of loads per thread), else a third launch scans them.
// These arrays are small (a few MB at most), so what a scan costs is its launches, 4 to 5 us
// each: 2 launches instead of 3 for 16385 .. 2^24 ints, 1 instead of 3 from 4097 to 16384.
constexpr int kScanOne = 16384;   // 1024 threads x 16
constexpr int kScanTile = 4096;   // 1024 threads x 4
constexpr int kScanSelf = 4096;

template <int PER, bool ZERO>
__device__ __forceinline__ void scan_tile(int* __restrict__ in, int n, long long base, int run0,
                                          int* __restrict__ out, int* wt, int* total) {
  int x[PER], t = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    x[u] = base + u < n ? in[base + u] : 0;
    t += x[u];
  }
  int run = run0 + block_excl(t, wt, total);
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (base + u < n) {
      out[base + u] = run;
      run += x[u];
      if (ZERO) in[base + u] = 0;
    }
}

template <int PER, bool ZERO>
__global__ __launch_bounds__(1024) void k_scan_one(int* __restrict__ in, int n,
                                                   int* __restrict__ out) {
  __shared__ int wt[16];
  int total;
  scan_tile<PER, ZERO>(in, n, (long long)PER * threadIdx.x, 0, out, wt, &total);
  if (threadIdx.x == 0) out[n] = total;
}

__global__ __launch_bounds__(1024) void k_scan_tile_sums(const int* __restrict__ in, int n,
                                                         int* __restrict__ sums) {
  __shared__ int wt[16];
  const long long base = (long long)blockIdx.x * kScanTile + 4LL * threadIdx.x;
  int v = 0, total;
  for (int u = 0; u < 4; ++u)
    if (base + u < n) v += in[base + u];
  block_excl(v, wt, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One workgroup walking the array in chunks of kScanTile with a running carry (the tile sums
// of very large scans).
__global__ __launch_bounds__(1024) void k_scan_walk(int* __restrict__ in, int n,
                                                    int* __restrict__ out) {
  __shared__ int wt[16];
  int carry = 0;
  for (int base = 0; base < n; base += kScanTile) {
    int total;
    scan_tile<4, false>(in, n, base + 4LL * threadIdx.x, carry, out, wt, &total);
    carry += total;
    __syncthreads();  // wt is free for the next chunk
  }
  if (threadIdx.x == 0) out[n] = carry;
}

// SELF: sums holds the tiles' own sums; else tile_off their exclusive scan.
template <bool SELF, bool ZERO>
__global__ __launch_bounds__(1024) void k_scan_tiles(int* __restrict__ in, int n,
                                                     const int* __restrict__ sums,
                                                     int* __restrict__ out) {
  __shared__ int wt[16], wt2[16];
  int before = 0, total;
  if constexpr (SELF) {
    int v = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += 1024) v += sums[b];
    block_excl(v, wt2, &before);
  } else {
    before = sums[blockIdx.x];
  }
  scan_tile<4, ZERO>(in, n, (long long)blockIdx.x * kScanTile + 4LL * threadIdx.x, before, out,
                     wt, &total);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = before + total;
}

// ---------------------------------------------------------------- k-means
// Count a centre on its cell; the count before it is its place in the cell's list.
__device__ __forceinline__ int bin_centre(const Grid& g, double q, double p,
                                          int* __restrict__ ccnt) {
  int cx, cy;
  return atomicAdd(ccnt + grid_cell(g, q, p, &cx, &cy), 1);
}

__global__ void k_init_bin(const double* __restrict__ q, const double* __restrict__ p,
                           const int* __restrict__ init_idx, int k, Grid g,
                           int* __restrict__ ccnt, int* __restrict__ cslot) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= k) return;
  const int i = init_idx[a];  // checked against [0, m) on the host
  cslot[a] = bin_centre(g, q[i], p[i], ccnt);
}

// Labels in cell order: centre a of the caller becomes label l, its place in the cell lists,
// which are then in label order themselves.
__global__ void k_init_labels(const double* __restrict__ q, const double* __restrict__ p,
                              const int* __restrict__ init_idx, int k, Grid g,
                              const int* __restrict__ coff, const int* __restrict__ cslot,
                              double* __restrict__ cq, double* __restrict__ cp,
                              int* __restrict__ origid, double2* __restrict__ cc,
                              int* __restrict__ clab, int* __restrict__ lab0) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= k) return;
  const int i = init_idx[a];
  const double qa = q[i], pa = p[i];
  int cx, cy;
  const int l = coff[grid_cell(g, qa, pa, &cx, &cy)] + cslot[a];
  cq[l] = qa;
  cp[l] = pa;
  cc[l] = make_double2(qa, pa);
  clab[l] = l;
  origid[l] = a;
  if (a == 0) *lab0 = l;
}

// The centres in cell order (their counts scanned into coff).
__global__ void k_cell_fill(const double* __restrict__ cq, const double* __restrict__ cp, int k,
                            Grid g, const int* __restrict__ coff, const int* __restrict__ cslot,
                            double2* __restrict__ cc, int* __restrict__ clab) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= k) return;
  const double qa = cq[l], pa = cp[l];
  int cx, cy;
  const int s = coff[grid_cell(g, qa, pa, &cx, &cy)] + cslot[l];
  cc[s] = make_double2(qa, pa);
  clab[s] = l;
}

// Markers in cell order (any order within a cell: it changes no result): count, then, after
// the scan, place.  idx: marker indices, gridDim.y batches of m (NULL: the markers themselves);
// each batch has cell counts of its own, one behind the other, so one scan orders them all.
__global__ void k_marker_count(const double* __restrict__ q, const double* __restrict__ p,
                               const int* __restrict__ idx, long long m, Grid g,
                               int* __restrict__ cnt, int* __restrict__ slot) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m) return;
  slot += blockIdx.y * m;
  cnt += (long long)blockIdx.y * g.gx * g.gp;
  if (idx) idx += blockIdx.y * m;
  const long long i = idx ? idx[t] : t;  // batch indices are checked on the device before
  slot[t] = bin_centre(g, q[i], p[i], cnt);
}

// RUNS: the markers' records in cell order; else perm[place] = t, and for a batch (idx) its
// copies of q, p, w at t.
template <bool RUNS>
__global__ void k_marker_place(const double* __restrict__ q, const double* __restrict__ p,
                               const double* __restrict__ w, const int* __restrict__ idx,
                               long long m, Grid g, const int* __restrict__ off,
                               const int* __restrict__ slot, Marker* __restrict__ rec,
                               int* __restrict__ perm, double* __restrict__ bq,
                               double* __restrict__ bp, double* __restrict__ bw) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m) return;
  slot += blockIdx.y * m;
  off += (long long)blockIdx.y * g.gx * g.gp;
  if (idx) idx += blockIdx.y * m;
  const long long i = idx ? idx[t] : t;
  const double qi = q[i], pi = p[i];
  int cx, cy;
  const int at = off[grid_cell(g, qi, pi, &cx, &cy)] + slot[t];
  if constexpr (RUNS) {
    rec[at] = Marker{qi, pi, w[i], (int)t, 0};
  } else {
    perm[at] = (int)t;
    if (idx) {
      bq[t] = qi;
      bp[t] = pi;
      bw[t] = w[i];
    }
  }
}

// The label of the centre nearest to (qi, pi).  prev: the marker's label before, or -1; the
// distance to that label's centre, as moved since, bounds the search from the start (the centre
// itself is found again in the lists).
// The search: the own cell and the ring around it, less the cells beyond the best distance; where
// the ring's outer edge is nearer than that distance, every further grid row the circle reaches,
// as one run of cells (an empty cell costs nothing in a run, and the markers in the thin tails of
// the velocity distribution have circles of thousands of empty cells: taken cell by cell, their
// wavefronts alone held a pass at 1069 us).
__device__ __forceinline__ int nearest_centre(
    double qi, double pi, int prev, const double* __restrict__ cq, const double* __restrict__ cp,
    const Grid& g, const int* __restrict__ coff, const double2* __restrict__ cc,
    const int* __restrict__ clab, const int* __restrict__ origid, const int* __restrict__ lab0,
    int k) {
  int cx, cy;
  grid_cell(g, qi, pi, &cx, &cy);
  // list bounds of the own row and its neighbours, cells cx-1 .. cx+1 (all loads at once)
  const int xl = max(cx - 1, 0), xr = min(cx + 1, g.gx - 1);
  int o[3][4];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int y = min(max(cy + (j == 2 ? -1 : j), 0), g.gp - 1);
    const int* row = coff + (long long)y * g.gx;
    o[j][0] = row[xl];
    o[j][1] = row[cx];
    o[j][2] = row[cx + 1];
    o[j][3] = row[xr + 1];
  }
  double lim = INFINITY;
  if (prev >= 0) {
    const int l = prev;
    const double dq = qi - cq[l], dp = pi - cp[l];
    const double d0 = dq * dq + dp * dp;
    if (d0 < INFINITY) lim = d0;
  }
  double best = INFINITY;
  int bs = -1;
  auto take = [&](double2 c, int s) {
    const double dq = qi - c.x, dp = pi - c.y;
    const double d2 = dq * dq + dp * dp;
    const bool less = d2 < best;
    if (!less && d2 == best) {  // a tie goes to the lower centre (rare)
      if (bs < 0 || origid[clab[s]] < origid[clab[bs]]) bs = s;
    }
    best = less ? d2 : best;
    bs = less ? s : bs;
  };
  auto scan = [&](int s, int e) {  // the centres s .. e-1 of the cell lists
    for (; s + 4 <= e; s += 4) {
      const double2 c0 = cc[s], c1 = cc[s + 1], c2 = cc[s + 2], c3 = cc[s + 3];
      take(c0, s);
      take(c1, s + 1);
      take(c2, s + 2);
      take(c3, s + 3);
    }
    for (; s < e; ++s) take(cc[s], s);
    lim = fmin(lim, best);
  };
  // Distances to cell edges are taken smaller by a millionth of a cell, far above the rounding
  // of the cell coordinates: a cell is left out only when it lies farther for certain.  (Also
  // where pmin is so large that pmin + y sp rounds by more: rounding is monotone, so the rounded
  // edge still has each row's centres, which are doubles, on its side.)
  const double mx = 1e-6 * g.sx, my = 1e-6 * g.sp;
  auto low = [](double d, double margin) { return fmax(0.0, d - margin); };
  auto row_gap = [&](int y) {
    return y < cy ? low(pi - (g.pmin + (y + 1) * g.sp), my)
                  : y > cy ? low(g.pmin + y * g.sp - pi, my) : 0.0;
  };
  const double gl = low(qi - cx * g.sx, mx), gr = low((cx + 1) * g.sx - qi, mx);
#pragma unroll
  for (int j = 0; j < 3; ++j) {  // own row first
    const int y = cy + (j == 2 ? -1 : j);
    if (y < 0 || y >= g.gp) continue;
    const double gy = row_gap(y), gy2 = gy * gy;
    if (gy2 > lim) continue;
    scan(gl * gl + gy2 <= lim ? o[j][0] : o[j][1], gr * gr + gy2 <= lim ? o[j][3] : o[j][2]);
  }
  // everything outside the square of radius r lies beyond one of its four edges (an edge on
  // the grid's border has nothing beyond it)
  auto edge = [&](int r) {
    double d = INFINITY;
    if (cx - r > 0) d = fmin(d, low(qi - (cx - r) * g.sx, mx));
    if (cx + r < g.gx - 1) d = fmin(d, low((cx + r + 1) * g.sx - qi, mx));
    if (cy - r > 0) d = fmin(d, low(pi - (g.pmin + (cy - r) * g.sp), my));
    if (cy + r < g.gp - 1) d = fmin(d, low(g.pmin + (cy + r + 1) * g.sp - pi, my));
    return d;
  };
  const double d1 = edge(1);
  if (lim == INFINITY && d1 < INFINITY) {
    // nothing to go by: the centres before and after the (empty) own cell in cell order, one of
    // which is in the own row where that holds any
    const int s = o[0][1];
    if (s > 0) take(cc[s - 1], s - 1);
    if (s < k) take(cc[s], s);
    lim = fmin(lim, best);
  }
  if (d1 < INFINITY && !(lim < d1 * d1)) {
    // rows cy, then cy + 1, cy - 1, cy + 2, ... four at a time: their list bounds are loaded
    // together (in the tails a circle takes dozens of rows, mostly empty, and the loads of one
    // after another were the pass's longest chain)
    for (int k0 = 0;; k0 += 4) {
      int s0[4], s1[4];
      bool reached = false;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u, dy = (k + 1) >> 1, y = (k & 1) ? cy + dy : cy - dy;
        s0[u] = s1[u] = 0;
        if (y < 0 || y >= g.gp) continue;
        const double gy = row_gap(y), rest = lim - gy * gy;
        if (rest < 0.0) continue;
        reached = true;
        const double hw = sqrt(rest) * (1.0 + 1e-9) + mx;
        const double fa = floor((qi - hw) / g.sx), fb = floor((qi + hw) / g.sx);
        const int xa = fa > 0.0 ? (int)fmin(fa, (double)(g.gx - 1)) : 0;
        const int xb = fb < (double)(g.gx - 1) ? (int)fmax(fb, 0.0) : g.gx - 1;
        const int* row = coff + (long long)y * g.gx;
        s0[u] = row[min(xa, cx)];
        s1[u] = row[max(xb, cx) + 1];
      }
      if (!reached) break;
#pragma unroll
      for (int u = 0; u < 4; ++u) scan(s0[u], s1[u]);
    }
  }
  // every centre is binned, so the whole grid holds one, unless every distance was NaN
  // (non-finite or zero-weight input): keep the index in range even then
  return bs < 0 ? *lab0 : clab[bs];
}

// Nearest centre of each marker, taken in cell order, so that neighbouring lanes search the same
// cells.  RUNS: from the records, assign is in that order too, the marker also counts on its
// cluster (cnt), and slot receives the count before it; else q, p and assign are in marker order,
// reached through perm.  prev: assign holds the previous iteration's labels.
// Bound by the latency of the list and centre loads from L2 (finer grids, with fewer centres to
// compare, are no faster).  4194304 markers and 419430 centres, ten markers a centre: 140 us a
// pass, against 1515 us with cell lists read through two indirections, square rings searched cell
// by cell and the clusters counted in a pass of their own (159 us).
// RUNS: a workgroup counts its markers per label in an LDS table and adds each label's count to
// the global counter once (neighbouring markers share labels; one device atomic per marker, 26
// per ns over the whole chip, took 150 us of the pass).  ccnt: ncells counters to clear (the next
// binning's, see k_scan_cells).  over: set once a cluster did not fit a run; the results are void
// then (cluster_run), and neither labels nor counts change any more.
constexpr int kAssignThreads = 256;  // 512 the same within 2%, 1024 5% slower
template <bool RUNS>
__global__ __launch_bounds__(kAssignThreads) void k_assign(
    const Marker* __restrict__ rec, const double* __restrict__ q, const double* __restrict__ p,
    long long m, const int* __restrict__ perm, const double* __restrict__ cq,
    const double* __restrict__ cp, Grid g, const int* __restrict__ coff,
    const double2* __restrict__ cc, const int* __restrict__ clab, const int* __restrict__ origid,
    const int* __restrict__ lab0, int prev, int* __restrict__ assign, int* __restrict__ cnt,
    int* __restrict__ slot, int* __restrict__ ccnt, int ncells, int k,
    const int* __restrict__ over) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if constexpr (!RUNS) {
    if (t >= m) return;
    const int i = perm[t];
    assign[i] = nearest_centre(q[i], p[i], prev ? assign[i] : -1, cq, cp, g, coff, cc, clab,
                               origid, lab0, k);
  } else {
    constexpr int kTable = 2 * kAssignThreads;  // twice the labels a workgroup can meet
    __shared__ int key[kTable], num[kTable];
    const int stop = *over;  // used behind the barrier below, which hides the load
    for (long long j = t; j < ncells; j += (long long)gridDim.x * kAssignThreads) ccnt[j] = 0;
    for (int j = threadIdx.x; j < kTable; j += kAssignThreads) {
      key[j] = -1;
      num[j] = 0;
    }
    __syncthreads();
    int h = 0, mine = 0;
    const bool on = t < m && !stop;
    if (on) {
      const int l = nearest_centre(rec[t].q, rec[t].p, prev ? assign[t] : -1, cq, cp, g, coff, cc,
                                   clab, origid, lab0, k);
      assign[t] = l;
      h = (int)(((unsigned)l * 2654435761u) >> 16) & (kTable - 1);
      for (;;) {  // at most half of the places are taken: an empty one is met
        const int was = atomicCAS(key + h, -1, l);
        if (was == -1 || was == l) break;
        h = (h + 1) & (kTable - 1);
      }
      mine = atomicAdd(num + h, 1);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < kTable; j += kAssignThreads)
      if (key[j] >= 0) num[j] = atomicAdd(cnt + key[j], num[j]);
    __syncthreads();
    if (on) slot[t] = num[h] + mine;
  }
}

// Members of each cluster, in any order: mem[off[label] + slot] = place of the marker.  (Nothing
// once `over` is set: assign may then hold no labels.)
__global__ void k_member_fill(const int* __restrict__ assign, const int* __restrict__ slot,
                              long long m, const int* __restrict__ off, int* __restrict__ mem,
                              const int* __restrict__ over) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m) return;
  const int a = assign[t], at = slot[t], stop = *over;  // one latency for the three
  if (!stop) mem[off[a] + at] = (int)t;
}

// The scan of the counters and the fill that needs it as one launch, for up to kFusedScan
// counters: every workgroup scans all of them into LDS for itself (they lie in L2), the first
// writes the offsets out, and the counters are cleared by the next kernel that may.  A pass over a
// small marker set is bound by its launches; 40960 markers in 4096 clusters took 7 us for each
// scan and 3 for each fill.
constexpr int kFusedScan = 8192;  // 1024 threads x 8

__device__ __forceinline__ void scan_lds(const int* __restrict__ in, int n, int* sh, int* wt,
                                         int* __restrict__ out) {
  constexpr int PER = kFusedScan / 1024;
  const int base = PER * threadIdx.x;
  int x[PER], t = 0, total;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    x[u] = base + u < n ? in[base + u] : 0;
    t += x[u];
  }
  int run = block_excl(t, wt, &total);
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (base + u < n) {
      sh[base + u] = run;
      if (blockIdx.x == 0) out[base + u] = run;
      run += x[u];
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = total;
  __syncthreads();
}

__global__ __launch_bounds__(1024) void k_scan_members(const int* __restrict__ cnt, int k,
                                                       int* __restrict__ off,
                                                       const int* __restrict__ assign,
                                                       const int* __restrict__ slot, long long m,
                                                       int* __restrict__ mem,
                                                       const int* __restrict__ over) {
  __shared__ int sh[kFusedScan], wt[16];
  const int stop = *over;
  scan_lds(cnt, k, sh, wt, off);
  if (stop) return;  // as k_member_fill
  const long long stride = (long long)gridDim.x * 1024;
  for (long long t = (long long)blockIdx.x * 1024 + threadIdx.x; t < m; t += stride)
    mem[sh[assign[t]] + slot[t]] = (int)t;
}

__global__ __launch_bounds__(1024) void k_scan_cells(const int* __restrict__ ccnt, int ncells,
                                                     int* __restrict__ coff,
                                                     const double* __restrict__ cq,
                                                     const double* __restrict__ cp, int k, Grid g,
                                                     const int* __restrict__ cslot,
                                                     double2* __restrict__ cc,
                                                     int* __restrict__ clab) {
  __shared__ int sh[kFusedScan], wt[16];
  scan_lds(ccnt, ncells, sh, wt, coff);
  const int stride = gridDim.x * 1024;
  for (int l = blockIdx.x * 1024 + threadIdx.x; l < k; l += stride) {
    const double qa = cq[l], pa = cp[l];
    int cx, cy;
    const int s = sh[grid_cell(g, qa, pa, &cx, &cy)] + cslot[l];
    cc[s] = make_double2(qa, pa);
    clab[s] = l;
  }
}

// Where a kernel of one thread per cluster leaves a centre that moved (or, without members,
// did not): bound for the next search.
struct CentreOut {
  double* cq;
  double* cp;
  double* v;     // mini-batch: the weight each centre has absorbed
  int* ccnt;     // centres per cell, counted for the next search
  int* cslot;
};

// Per-cluster work of one pass, on members gathered by k_member_fill.  A workgroup takes
// `per` consecutive labels, in runs whose members fit kGroupCap; each member's rank in its
// cluster is the number of members with a smaller marker index (markers are unique), which
// puts the run's q, p, w into marker order in LDS; one thread per cluster then adds its terms
// in that order.  A single cluster above kGroupCap is not taken: `over` is set, the passes that
// follow find no members, and the caller runs everything again with the radix sort.
//   kGroupMean   the centre moves to the weighted mean; a cluster with no members keeps it
//   kGroupBatch  the mini-batch update (see k_minibatch_update)
//   kGroupMoments the decorated particle (see k_moments)
// Bound by latency (dependent gathers of members, LDS round trips), not bytes: 44 B a member.
// At 4194304 markers in 419430 clusters 64 us (moments 123 us), with 14 us for the member lists.
// It replaces three passes of a stable radix sort (430 us), the counting of the clusters in
// marker order (159 us) and one thread per cluster gathering from the markers at random
// (251 us; 687 us for the moments).
constexpr int kGroupCap = 512;  // 1024: 3 to 5% slower (fewer workgroups to a CU)
constexpr int kGroupThreads = 256;
// Mean members per cluster up to which the runs are used: a member compares itself with its
// whole cluster, and a cluster has to fit a run with room for uneven ones.
constexpr int kGroupMeanMax = 96;
enum GroupWork { kGroupMean = 0, kGroupBatch = 1, kGroupMoments = 2 };

struct MomentOut {
  double* Q;
  double* P;
  double* qs;
  double* ps;
  double* psi;
  int* flag;
};

template <int WORK>
__global__ __launch_bounds__(kGroupThreads) void k_group(
    const Marker* __restrict__ rec, const int* __restrict__ assign, const int* __restrict__ off,
    const int* __restrict__ mem, int k, int per, Grid g, double L, CentreOut co, MomentOut mo,
    const int* __restrict__ origid, int* __restrict__ over, int* __restrict__ cnt) {
  constexpr int kSlots = kGroupCap / kGroupThreads;
  __shared__ int soff[kGroupThreads + 1];
  __shared__ int sidx[kGroupCap];
  __shared__ double lq[kGroupCap], lp[kGroupCap], lw[kGroupCap];
  __shared__ double ld[WORK == kGroupMoments ? kGroupCap : 1];
  __shared__ double zq[WORK == kGroupMoments ? kGroupThreads : 1];
  __shared__ double zp[WORK == kGroupMoments ? kGroupThreads : 1];
  const int tid = threadIdx.x;
  const int a0 = (int)blockIdx.x * per, na = min(per, k - a0);
  if (cnt && tid < na) cnt[a0 + tid] = 0;  // counted out by k_scan_members
  if (tid <= na) soff[tid] = off[a0 + tid];
  if (tid == 0 && na == kGroupThreads) soff[na] = off[a0 + na];
  __syncthreads();
  for (int c = 0; c < na;) {
    const int base = soff[c];
    const int e = c + __syncthreads_count(tid >= c && tid < na && soff[tid + 1] - base <= kGroupCap);
    if (e == c) {  // one cluster too large for a run
      if (tid == 0) {
        *over = 1;
        const int l = a0 + c;
        if constexpr (WORK == kGroupMoments) mo.flag[origid[l]] = 0;
        else co.cslot[l] = bin_centre(g, co.cq[l], co.cp[l], co.ccnt);
      }
      ++c;
      continue;
    }
    const int n = soff[e] - base;
    Marker mk[kSlots];
    int lab[kSlots];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int j = u * kGroupThreads + tid;
      if (j < n) {
        const int at = mem[base + j];
        mk[u] = rec[at];
        lab[u] = assign[at];
        sidx[j] = mk[u].id;
      }
    }
    __syncthreads();
    int pos[kSlots], own[kSlots];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int j = u * kGroupThreads + tid;
      pos[u] = own[u] = 0;
      if (j < n) {
        const int l = lab[u] - a0, i = mk[u].id;
        const int b = soff[l] - base, f = soff[l + 1] - base;
        int r = b;
        for (int x = b; x < f; ++x) r += sidx[x] < i;
        own[u] = l;
        pos[u] = r;
        lq[r] = mk[u].q;
        lp[r] = mk[u].p;
        lw[r] = mk[u].w;
      }
    }
    __syncthreads();
    const bool mine = tid >= c && tid < e;
    const int b = mine ? soff[tid] - base : 0, f = mine ? soff[tid + 1] - base : 0;
    const int l = a0 + tid;
    double W = 0.0, SQ = 0.0, SP = 0.0;
    for (int x = b; x < f; ++x) {
      W += lw[x];
      SQ += lw[x] * lq[x];
      SP += lw[x] * lp[x];
    }
    if constexpr (WORK != kGroupMoments) {
      if (mine) {
        double nq = co.cq[l], np = co.cp[l];
        if (f > b) {
          if constexpr (WORK == kGroupBatch) {
            const double vo = co.v[l], vn = vo + W;
            nq = (nq * vo + SQ) / vn;
            np = (np * vo + SP) / vn;
            co.v[l] = vn;
          } else {
            nq = SQ / W;
            np = SP / W;
          }
          co.cq[l] = nq;
          co.cp[l] = np;
        }
        co.cslot[l] = bin_centre(g, nq, np, co.ccnt);
      }
    } else {
      if (mine && f > b) {
        zq[tid] = SQ / W;
        zp[tid] = SP / W;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kSlots; ++u)
        if (u * kGroupThreads + tid < n) {
          const double dq = lq[pos[u]] - zq[own[u]], dp = lp[pos[u]] - zp[own[u]];
          ld[pos[u]] = dq * dq + dp * dp;
        }
      __syncthreads();
      if (mine && f > b) {  // the member nearest the mean, the first on ties
        double best = INFINITY;
        int x0 = b;
        for (int x = b; x < f; ++x)
          if (ld[x] < best) {
            best = ld[x];
            x0 = x;
          }
        zq[tid] = lq[x0];
        zp[tid] = lp[x0];
      }
      __syncthreads();
      const double half_len = L / kTwoPi;
#pragma unroll
      for (int u = 0; u < kSlots; ++u)
        if (u * kGroupThreads + tid < n) {
          const int x = pos[u];
          const double wi = lw[x];
          lq[x] = wi * (half_len * sin(kTwoPi * (zq[own[u]] - lq[x]) / L));
          lp[x] = wi * (zp[own[u]] - lp[x]);
        }
      __syncthreads();
      if (mine) {
        const int o = origid[l];
        mo.flag[o] = f > b;
        if (f > b) {
          double sps = 0.0, sqs = 0.0;
          for (int x = b; x < f; ++x) {
            sps += lq[x];
            sqs += lp[x];
          }
          mo.Q[o] = zq[tid];
          mo.P[o] = zp[tid];
          mo.ps[o] = sps;
          mo.qs[o] = -sqs;
          mo.psi[o] = W;
        }
      }
    }
    __syncthreads();  // LDS is free for the next run
    c = e;
  }
}

__global__ void k_group_count(const int* __restrict__ assign, long long m, int* __restrict__ cnt) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) atomicAdd(cnt + assign[i], 1);
}

// Stable LSD radix sort of (key, value) pairs by 8-bit digits: per-chunk digit counts, a
// digit-major scan of them, then a stable scatter in which each chunk keeps its elements in
// order.  Chunks of kRadixChunk elements, one 256-thread workgroup each.
__global__ __launch_bounds__(256) void k_radix_hist(const int* __restrict__ keys, long long m,
                                                    int shift, int nb, int* __restrict__ hist) {
  __shared__ int cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const long long b0 = (long long)blockIdx.x * kRadixChunk;
  const long long e0 = b0 + kRadixChunk < m ? b0 + kRadixChunk : m;
  for (long long i = b0 + threadIdx.x; i < e0; i += 256)
    atomicAdd(cnt + ((keys[i] >> shift) & 255), 1);
  __syncthreads();
  hist[(long long)threadIdx.x * nb + blockIdx.x] = cnt[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_radix_scatter(const int* __restrict__ kin,
                                                       const int* __restrict__ vin, long long m,
                                                       int shift, int nb,
                                                       const int* __restrict__ hoff,
                                                       int* __restrict__ kout,
                                                       int* __restrict__ vout) {
  __shared__ int run[256];
  __shared__ int dig[256];
  run[threadIdx.x] = hoff[(long long)threadIdx.x * nb + blockIdx.x];
  const long long b0 = (long long)blockIdx.x * kRadixChunk;
  const long long e0 = b0 + kRadixChunk < m ? b0 + kRadixChunk : m;
  for (long long s0 = b0; s0 < e0; s0 += 256) {
    const long long i = s0 + threadIdx.x;
    const bool valid = i < e0;
    const int key = valid ? kin[i] : 0;
    const int d = valid ? ((key >> shift) & 255) : -1;
    __syncthreads();  // run[] settled, dig[] free
    dig[threadIdx.x] = d;
    __syncthreads();
    int rank = 0, total = 0;
    for (int t = 0; t < 256; ++t) {
      const int same = dig[t] == d;
      rank += (t < (int)threadIdx.x) & same;
      total += same;
    }
    if (valid) {
      const int pos = run[d] + rank;
      kout[pos] = key;
      vout[pos] = vin[i];
    }
    __syncthreads();  // every thread has read run[d]
    if (valid && rank + 1 == total) run[d] += total;  // the batch's last element of digit d
  }
}

__global__ void k_iota(int* __restrict__ v, long long m) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) v[i] = (int)i;
}

// New centre of each cluster: weighted mean of its members, summed in marker order; a
// cluster with no members keeps its centre.
__global__ void k_centres(const double* __restrict__ q, const double* __restrict__ p,
                          const double* __restrict__ w, const int* __restrict__ off,
                          const int* __restrict__ order, int k, Grid g, CentreOut co) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= k) return;
  const int b = off[a], e = off[a + 1];
  double nq = co.cq[a], np = co.cp[a];
  if (b < e) {
    double W = 0.0, SQ = 0.0, SP = 0.0;
    for (int t = b; t < e; ++t) {
      const int i = order[t];
      W += w[i];
      SQ += w[i] * q[i];
      SP += w[i] * p[i];
    }
    co.cq[a] = nq = SQ / W;
    co.cp[a] = np = SP / W;
  }
  co.cslot[a] = bin_centre(g, nq, np, co.ccnt);
}

// Mini-batch k-means, the weighted batched form of Sculley's update ("Web-scale k-means
// clustering", 2010): move each centre that received members of this batch to the weighted
// mean of every batch member it has received, its old value standing in for the earlier
// ones: v <- v + W, centre <- (centre v_old + S) / v.  W and S are summed over the members
// in batch order, so the result is that of a sequential pass.

// Count the batch indices outside [0, m) (host check before any use).
__global__ void k_count_bad(const int* __restrict__ idx, long long n, long long m,
                            int* __restrict__ bad) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n && (idx[t] < 0 || (long long)idx[t] >= m)) atomicAdd(bad, 1);
}

__global__ void k_minibatch_update(const double* __restrict__ bq, const double* __restrict__ bp,
                                   const double* __restrict__ bw, const int* __restrict__ off,
                                   const int* __restrict__ order, int k, Grid g, CentreOut co) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= k) return;
  const int b = off[a], e = off[a + 1];
  double nq = co.cq[a], np = co.cp[a];
  if (b < e) {
    double W = 0.0, SQ = 0.0, SP = 0.0;
    for (int t = b; t < e; ++t) {
      const int i = order[t];
      W += bw[i];
      SQ += bw[i] * bq[i];
      SP += bw[i] * bp[i];
    }
    const double vo = co.v[a], vn = vo + W;
    co.cq[a] = nq = (nq * vo + SQ) / vn;
    co.cp[a] = np = (np * vo + SP) / vn;
    co.v[a] = vn;
  }
  co.cslot[a] = bin_centre(g, nq, np, co.ccnt);
}

// The decorated particle of each non-empty cluster (Algorithm 1): weight, centre member
// nearest the weighted mean (first in marker order on ties), periodic spatial moment and
// velocity moment, all summed in marker order.  flag = 1 for a non-empty cluster.  Written at
// the caller's number of the cluster.
__global__ void k_moments(const double* __restrict__ q, const double* __restrict__ p,
                          const double* __restrict__ w, const int* __restrict__ off,
                          const int* __restrict__ order, int k, double L,
                          const int* __restrict__ origid, MomentOut mo) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= k) return;
  const int b = off[a], e = off[a + 1], o = origid[a];
  mo.flag[o] = b < e;
  if (b == e) return;
  double W = 0.0, SQ = 0.0, SP = 0.0;
  for (int t = b; t < e; ++t) {
    const int i = order[t];
    W += w[i];
    SQ += w[i] * q[i];
    SP += w[i] * p[i];
  }
  const double zq = SQ / W, zp = SP / W;
  double best = INFINITY;
  int a0 = order[b];
  for (int t = b; t < e; ++t) {
    const int i = order[t];
    const double dq = q[i] - zq, dp = p[i] - zp;
    const double d2 = dq * dq + dp * dp;
    if (d2 < best) {
      best = d2;
      a0 = i;
    }
  }
  const double Qa = q[a0], Pa = p[a0];
  const double half_len = L / kTwoPi;
  double sps = 0.0, sqs = 0.0;
  for (int t = b; t < e; ++t) {
    const int i = order[t];
    sps += w[i] * (half_len * sin(kTwoPi * (Qa - q[i]) / L));
    sqs += w[i] * (Pa - p[i]);
  }
  mo.Q[o] = Qa;
  mo.P[o] = Pa;
  mo.ps[o] = sps;
  mo.qs[o] = -sqs;
  mo.psi[o] = W;
}

// res[0] = number of decorated particles, res[1] = a run was too large (`over`): nothing is
// written then, here and in the two kernels below, so that the caller's arrays, which may be the
// inputs', are as they were for the second take.
__global__ void k_compact(const int* __restrict__ pos, int k, MomentOut mo,
                          double* __restrict__ Q, double* __restrict__ P,
                          double* __restrict__ qs, double* __restrict__ ps,
                          double* __restrict__ psi, const int* __restrict__ over,
                          int* __restrict__ res) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a == 0) {
    res[0] = pos[k];
    res[1] = *over;
  }
  if (a >= k || !mo.flag[a] || *over) return;
  const int j = pos[a];
  Q[j] = mo.Q[a];
  P[j] = mo.P[a];
  qs[j] = mo.qs[a];
  ps[j] = mo.ps[a];
  psi[j] = mo.psi[a];
}

// The caller's cluster number of each marker (rec NULL: assign is in marker order).
__global__ void k_assign_out(const int* __restrict__ assign, const Marker* __restrict__ rec,
                             const int* __restrict__ origid, long long m,
                             int* __restrict__ out, const int* __restrict__ over) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < m && *over == 0) out[rec ? rec[t].id : t] = origid[assign[t]];
}

__global__ void k_absorbed_out(const double* __restrict__ v, const int* __restrict__ origid,
                               int k, double* __restrict__ out, const int* __restrict__ over) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l < k && *over == 0) out[origid[l]] = v[l];
}

__global__ void k_copy_int(const int* __restrict__ in, long long n, int* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i];
}

unsigned blocks_for(long long n, int tpb) {
  long long b = (n + tpb - 1) / tpb;
  return (unsigned)(b < 1 ? 1 : b);
}

hipError_t fill_int(int* p, long long n, int v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  long long b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_fill_int, dim3((unsigned)b), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Exclusive scan of n ints into out[0..n]; tmp holds 2 * (n / kScanTile + 2) ints.  ZERO: in is
// cleared.
template <bool ZERO>
hipError_t scan_int(int* in, int n, int* out, int* tmp, hipStream_t s) {
  if (n <= kScanOne) {
    if (n <= 4096) hipLaunchKernelGGL((k_scan_one<4, ZERO>), dim3(1), dim3(1024), 0, s, in, n, out);
    else hipLaunchKernelGGL((k_scan_one<16, ZERO>), dim3(1), dim3(1024), 0, s, in, n, out);
    return hipGetLastError();
  }
  const int nt = (n - 1) / kScanTile + 1;
  int* sums = tmp;
  int* toff = tmp + nt + 1;
  hipLaunchKernelGGL(k_scan_tile_sums, dim3(nt), dim3(1024), 0, s, in, n, sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nt <= kScanSelf) {
    hipLaunchKernelGGL((k_scan_tiles<true, ZERO>), dim3(nt), dim3(1024), 0, s, in, n, sums, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_scan_walk, dim3(1), dim3(1024), 0, s, sums, nt, toff);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL((k_scan_tiles<false, ZERO>), dim3(nt), dim3(1024), 0, s, in, n, toff, out);
  return hipGetLastError();
}

// Ints of scan scratch for scans of up to n elements.
long long scan_tmp_ints(long long n) { return 2 * (n / kScanTile + 2); }

}  // namespace

// What either grouping of the members needs (the runs 40 bytes a marker, the radix sort 22) lies
// over what the other needs: a call that is taken again by the radix sort starts afresh.  The
// mini-batches' cell counts lie over the moments of the last pass.
ClusterWs cluster_layout(long long m, int k, int batch, bool runs) {
  ClusterWs w{};
  const long long gmax = cluster_max_cells(k);
  const size_t nb = batch > 0 ? (size_t)batch : 0;
  size_t o = 0;
  w.cq = o;      o = a256(o + (size_t)k * sizeof(double));
  w.cp = o;      o = a256(o + (size_t)k * sizeof(double));
  w.assign = o;  o = a256(o + (size_t)m * sizeof(int));
  w.cnt = o;     o = a256(o + (size_t)k * sizeof(int));
  w.off = o;     o = a256(o + (size_t)(k + 1) * sizeof(int));
  w.origid = o;  o = a256(o + (size_t)k * sizeof(int));
  w.ccnt = o;    o = a256(o + (size_t)gmax * sizeof(int));
  w.coff = o;    o = a256(o + (size_t)(gmax + 1) * sizeof(int));
  w.cc = o;      o = a256(o + (size_t)gmax * sizeof(int));  // >= 16 k bytes
  w.clist = o;   o = a256(o + (size_t)k * sizeof(int));
  w.mm = o;      o = a256(o + (size_t)(2 * kClusterMinMaxBlocks + 2) * sizeof(double));
  w.bcnt = o;    // batches (batch <= m): cells counted, and scanned, before the moments are used
  w.boff = a256(w.bcnt + (size_t)gmax * sizeof(int));
  w.tQ = o;      o = a256(o + (size_t)k * sizeof(double));
  w.tP = o;      o = a256(o + (size_t)k * sizeof(double));
  w.tqs = o;     o = a256(o + (size_t)k * sizeof(double));
  w.tps = o;     o = a256(o + (size_t)k * sizeof(double));
  w.tpsi = o;    o = a256(o + (size_t)k * sizeof(double));
  if (batch > 0) {
    const size_t cells = a256(w.boff + (size_t)(gmax + 1) * sizeof(int));
    o = o < cells ? cells : o;
  }
  w.flag = o;    o = a256(o + (size_t)k * sizeof(int));  // the centres' places in their cells before
  w.pos = o;     o = a256(o + (size_t)(k + 1) * sizeof(int));
  {
    long long nmax = 256 * radix_blocks(m);
    if (nmax < k) nmax = k;
    if (nmax < gmax) nmax = gmax;
    if (runs && nmax < m) nmax = m;  // several batches' cells at once
    w.scan = o;  o = a256(o + (size_t)scan_tmp_ints(nmax) * sizeof(int));
  }
  w.v = o;       o = a256(o + (batch > 0 ? (size_t)k : 0) * sizeof(double));
  w.bad = o;     o = a256(o + 8 * sizeof(int));
  const size_t o0 = o;
  w.perm = o;    o = a256(o + (size_t)m * sizeof(int));
  w.keys_a = o;  o = a256(o + (size_t)m * sizeof(int));
  w.vals_a = o;  o = a256(o + (size_t)m * sizeof(int));
  w.keys_b = o;  o = a256(o + (size_t)m * sizeof(int));
  w.vals_b = o;  o = a256(o + (size_t)m * sizeof(int));
  w.hist = o;    o = a256(o + (size_t)256 * radix_blocks(m) * sizeof(int));
  w.hoff = o;    o = a256(o + ((size_t)256 * radix_blocks(m) + 1) * sizeof(int));
  w.bq = o;      o = a256(o + nb * sizeof(double));
  w.bp = o;      o = a256(o + nb * sizeof(double));
  w.bw = o;      o = a256(o + nb * sizeof(double));
  w.bperm = o;   o = a256(o + nb * sizeof(int));
  w.total = o;
  if (runs) {
    o = o0;
    w.slot = o;  o = a256(o + (size_t)m * sizeof(int));
    w.mem = o;   o = a256(o + (size_t)m * sizeof(int));
    w.rec = o;   o = a256(o + (size_t)m * sizeof(Marker));
    w.brec = o;  o = a256(o + nb * sizeof(Marker));
    w.total = w.total < o ? o : w.total;
  }
  return w;
}

// Up to here a workspace may grow for the runs' sake (their records make it about 1.7 times the
// radix sort's): a sixteenth of the card.  Beyond, marker sets that fill the card keep the
// smaller one, and the radix sort.
constexpr size_t kRunsBytesMax = size_t(16) << 30;

bool cluster_runs(long long m, int k, int batch) {
  return m <= (long long)kGroupMeanMax * k && cluster_layout(m, k, batch, true).total <= kRunsBytesMax;
}

// Never less for more markers, clusters or batch markers, though the runs are left at both of
// their bounds: a workspace of the largest call serves every smaller one.
size_t cluster_bytes(long long m, int k, int batch) {
  const size_t radix = cluster_layout(m, k, batch, false).total;
  const long long mr = m < (long long)kGroupMeanMax * k ? m : (long long)kGroupMeanMax * k;
  const size_t wide = cluster_layout(mr, k, batch, true).total;
  const size_t most = wide < kRunsBytesMax ? wide : kRunsBytesMax;
  return radix < most ? most : radix;
}

// ---------------------------------------------------------------- allocation-free workspace
// The workspace of vp_cluster_markers_static.  A file-scope device array: each device the
// library runs on holds its own copy for the life of the process.  In host code the array's
// name is only a stand-in for the symbol, never a device address: its address on a device
// comes from hipGetSymbolAddress, taken once per device with that device current and kept.
static __device__ __align__(256) unsigned char scratch[VP_CLUSTER_STATIC_BYTES];

hipError_t cluster_static_workspace(void** ptr_out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptrs[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptrs[dev] = p;
  }
  *ptr_out = ptrs[dev];
  return hipSuccess;
}

hipError_t cluster_check_inputs(const double* p, long long m, const int* init_idx, int k,
                                const int* batch_idx, long long nbatch_idx, void* ws,
                                const ClusterWs& w, ClusterCheck* host, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  double* part = reinterpret_cast<double*>(base + w.mm);
  double* res = part + 2 * kClusterMinMaxBlocks;
  int* bad = reinterpret_cast<int*>(base + w.bad);
  hipError_t e = fill_int(bad, 2, 0, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_count_bad, dim3(blocks_for(k, 256)), dim3(256), 0, s, init_idx,
                     (long long)k, m, bad);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (nbatch_idx > 0) {
    hipLaunchKernelGGL(k_count_bad, dim3(blocks_for(nbatch_idx, 256)), dim3(256), 0, s, batch_idx,
                       nbatch_idx, m, bad + 1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  long long nb = (m + 255) / 256;
  if (nb > kClusterMinMaxBlocks) nb = kClusterMinMaxBlocks;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_minmax_partial, dim3((unsigned)nb), dim3(256), 0, s, p, m, part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_minmax_final, dim3(1), dim3(256), 0, s, part, (int)nb, res);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(host->minmax, res, sizeof host->minmax, hipMemcpyDeviceToHost, s)) !=
      hipSuccess)
    return e;
  if ((e = hipMemcpyAsync(host->bad, bad, sizeof host->bad, hipMemcpyDeviceToHost, s)) != hipSuccess)
    return e;
  return hipStreamSynchronize(s);
}

// Stable sort of the marker indices 0..m-1 by keys (values below 2^bits) with 8-bit LSD
// passes; keys_a holds the keys on entry (overwritten).  *out = the sorted indices (one of
// vals_a / vals_b).
static hipError_t sort_indices(long long m, int bits, int* keys_a, int* vals_a, int* keys_b,
                               int* vals_b, int* hist, int* hoff, int* stmp, int** out,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_iota, dim3(blocks_for(m, 256)), dim3(256), 0, s, vals_a, m);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nb = (int)((m + kRadixChunk - 1) / kRadixChunk);
  for (int shift = 0; shift < bits; shift += 8) {
    hipLaunchKernelGGL(k_radix_hist, dim3(nb), dim3(256), 0, s, keys_a, m, shift, nb, hist);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = scan_int<false>(hist, 256 * nb, hoff, stmp, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_radix_scatter, dim3(nb), dim3(256), 0, s, keys_a, vals_a, m, shift, nb,
                       hoff, keys_b, vals_b);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int* t = keys_a; keys_a = keys_b; keys_b = t;
    t = vals_a; vals_a = vals_b; vals_b = t;
  }
  *out = vals_a;
  return hipSuccess;
}

static int key_bits(long long nkeys) {
  int bits = 1;
  while (bits < 31 && (1LL << bits) < nkeys) ++bits;
  return bits;
}

// Group the markers by their assignment: counts (cnt: zero on entry and on return) and segment
// offsets per cluster, and the marker indices sorted by cluster (stable, so in marker order
// within each cluster).
static hipError_t group_markers(long long m, int k, const int* assign, int* cnt, int* off,
                                int* keys_a, int* vals_a, int* keys_b, int* vals_b, int* hist,
                                int* hoff, int* stmp, int** order_out, hipStream_t s) {
  hipLaunchKernelGGL(k_group_count, dim3(blocks_for(m, 256)), dim3(256), 0, s, assign, m, cnt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = scan_int<true>(cnt, k, off, stmp, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_copy_int, dim3(blocks_for(m, 256)), dim3(256), 0, s, assign, m, keys_a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return sort_indices(m, key_bits(k), keys_a, vals_a, keys_b, vals_b, hist, hoff, stmp,
                      order_out, s);
}

hipError_t cluster_run(const double* q, const double* p, const double* w, long long m, int k,
                       const int* init_idx, const int* batch_idx, int batch, int nbatch,
                       int iters, double L, double pmin, double pmax, void* ws,
                       const ClusterWs& lay, bool runs, double* Q, double* P, double* qs,
                       double* ps, double* psi, int* assign_out, double* absorbed_out,
                       int* host_res, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  auto ints = [&](size_t o) { return reinterpret_cast<int*>(base + o); };
  auto doubles = [&](size_t o) { return reinterpret_cast<double*>(base + o); };
  int* assign = ints(lay.assign);
  int* cnt = ints(lay.cnt);
  int* off = ints(lay.off);
  int* perm = ints(lay.perm);
  int *keys_a = ints(lay.keys_a), *vals_a = ints(lay.vals_a);
  int *keys_b = ints(lay.keys_b), *vals_b = ints(lay.vals_b);
  int *hist = ints(lay.hist), *hoff = ints(lay.hoff), *stmp = ints(lay.scan);
  int *ccnt = ints(lay.ccnt), *coff = ints(lay.coff), *clab = ints(lay.clist);
  int* origid = ints(lay.origid);
  int* pos = ints(lay.pos);
  int* lab0 = ints(lay.bad) + 2;
  int* over = ints(lay.bad) + 3;
  int* res = ints(lay.bad) + 4;
  double2* cc = reinterpret_cast<double2*>(base + lay.cc);
  Marker* rec = reinterpret_cast<Marker*>(base + lay.rec);
  Marker* brec = reinterpret_cast<Marker*>(base + lay.brec);
  int *slot = ints(lay.slot), *mem = ints(lay.mem);
  const CentreOut co{doubles(lay.cq), doubles(lay.cp), doubles(lay.v), ccnt, ints(lay.flag)};
  const MomentOut mo{doubles(lay.tQ), doubles(lay.tP), doubles(lay.tqs), doubles(lay.tps),
                     doubles(lay.tpsi), ints(lay.flag)};
  int* order = nullptr;

  // grid over [0, L) x [pmin, pmax] (see kCellsPerCentre)
  Grid g{};
  const double span = pmax > pmin ? pmax - pmin : 1.0;
  const long long gmax = cluster_max_cells(k);
  double cell = sqrt(L * span / (kCellsPerCentre * (double)k));
  for (;;) {
    const double gx = ceil(L / cell), gp = ceil(span / cell);
    if (gx * gp <= (double)gmax) {
      g.gx = (int)(gx < 1 ? 1 : gx);
      g.gp = (int)(gp < 1 ? 1 : gp);
      break;
    }
    cell *= 1.25;
  }
  g.sx = L / g.gx;
  g.sp = span / g.gp;
  g.pmin = pmin;
  const int G = g.gx * g.gp;

  const dim3 tb(256), mb(blocks_for(m, 256)), kb(blocks_for(k, 256));
  const dim3 ta(kAssignThreads), ma(blocks_for(m, kAssignThreads));
  hipError_t e = hipSuccess;
#define VP_LAUNCH(kernel, grid, block, ...)                                     \
  do {                                                                         \
    hipLaunchKernelGGL(kernel, grid, block, 0, s, __VA_ARGS__);                \
    if ((e = hipGetLastError()) != hipSuccess) return e;                       \
  } while (0)
#define VP_CALL(expr)                             \
  do {                                            \
    if ((e = (expr)) != hipSuccess) return e;     \
  } while (0)

  VP_CALL(fill_int(ccnt, G, 0, s));
  VP_CALL(fill_int(cnt, k, 0, s));
  VP_CALL(fill_int(over, 1, 0, s));
  // the markers in grid-cell order (the grid stays fixed): the assignment's visiting order
  auto order_markers = [&](int* count, int* offset) -> hipError_t {  // count: cleared
    VP_LAUNCH(k_marker_count, mb, tb, q, p, (const int*)nullptr, m, g, count, assign);
    VP_CALL(scan_int<true>(count, G, offset, stmp, s));
    if (runs)
      VP_LAUNCH(k_marker_place<true>, mb, tb, q, p, w, (const int*)nullptr, m, g, offset, assign,
                rec, perm, nullptr, nullptr, nullptr);
    else
      VP_LAUNCH(k_marker_place<false>, mb, tb, q, p, w, (const int*)nullptr, m, g, offset, assign,
                rec, perm, nullptr, nullptr, nullptr);
    return hipSuccess;
  };
  // after the batches, whose records take the markers' place until then
  if (nbatch == 0) VP_CALL(order_markers(ccnt, coff));
  // the centres, renumbered in cell order
  VP_LAUNCH(k_init_bin, kb, tb, q, p, init_idx, k, g, ccnt, co.cslot);
  VP_CALL(scan_int<true>(ccnt, G, coff, stmp, s));
  VP_LAUNCH(k_init_labels, kb, tb, q, p, init_idx, k, g, coff, co.cslot, co.cq, co.cp, origid, cc,
            clab, lab0);
  const bool fused = runs && k <= kFusedScan && G <= kFusedScan;
  int* const cnt0 = fused ? cnt : nullptr;  // cleared by k_group
  const int cells0 = fused ? G : 0;         // cleared by k_assign
  auto bin_centres = [&]() -> hipError_t {  // counted by the kernel that moved the centres
    if (fused) {
      VP_LAUNCH(k_scan_cells, dim3(blocks_for(k, 1024)), dim3(1024), ccnt, G, coff, co.cq, co.cp, k,
                g, co.cslot, cc, clab);
      return hipSuccess;
    }
    VP_CALL(scan_int<true>(ccnt, G, coff, stmp, s));
    VP_LAUNCH(k_cell_fill, kb, tb, co.cq, co.cp, k, g, coff, co.cslot, cc, clab);
    return hipSuccess;
  };
  // labels per workgroup of k_group: about three quarters of a run, 256 at most
  auto per_group = [&](long long n) {
    const long long a = (3LL * kGroupCap / 4) * k / (n > 0 ? n : 1);
    return (int)(a < 1 ? 1 : (a > kGroupThreads ? kGroupThreads : a));
  };
  auto group_runs = [&](long long n) -> hipError_t {  // counts and slots are in place
    if (fused) {
      const unsigned nb = blocks_for(n, 1024);
      VP_LAUNCH(k_scan_members, dim3(nb < 512 ? nb : 512), dim3(1024), cnt, k, off, assign, slot, n,
                mem, over);
      return hipSuccess;
    }
    VP_CALL(scan_int<true>(cnt, k, off, stmp, s));
    VP_LAUNCH(k_member_fill, dim3(blocks_for(n, 256)), tb, assign, slot, n, off, mem, over);
    return hipSuccess;
  };
  const int per_m = per_group(m), per_b = per_group(batch);
  const dim3 gm(blocks_for(k, per_m)), gb(blocks_for(k, per_b)), gt(kGroupThreads);

  if (nbatch > 0) {
    // mini-batch updates; the batch's assignment and grouping use the marker arrays (b <= m)
    double *bq = doubles(lay.bq), *bp = doubles(lay.bp), *bw = doubles(lay.bw);
    int *bperm = ints(lay.bperm), *bcnt = ints(lay.bcnt), *boff = ints(lay.boff);
    const dim3 ba(blocks_for(batch, kAssignThreads));
    const long long nb = batch;
    VP_CALL(launch_fill_zero(co.v, (size_t)k * sizeof(double), s));
    // A batch is visited in grid-cell order (a random batch in its own order would send the lanes
    // of a wavefront to unrelated cells); the order does not change any result.  It depends on no
    // centre, so with runs as many batches as fit are ordered at once: their records where the
    // markers' go later, their counts and offsets where a batch's slots and members go after.  Eight batches of 162500 among 1.3 million markers, 130000 cells: 326 us one at a
    // time (four launches each, most of them too small to fill the card), 156 us at once.
    long long several = 1;
    if (runs) {
      several = m / nb < (m - 1) / G ? m / nb : (m - 1) / G;  // offsets: several * G + 1 ints
      several = several < nbatch ? several : nbatch;
      several = several < 1 ? 1 : (several > 32768 ? 32768 : several);
    }
    int* const ocnt = several > 1 ? slot : bcnt;
    int* const ooff = several > 1 ? mem : boff;
    Marker* const orec = several > 1 ? rec : brec;
    for (long long t0 = 0; t0 < nbatch; t0 += several) {
      const int n = (int)(nbatch - t0 < several ? nbatch - t0 : several);
      const int* idx = batch_idx + t0 * batch;
      const dim3 bb(blocks_for(batch, 256), (unsigned)n);
      if (t0 == 0 || several > 1) VP_CALL(fill_int(ocnt, (long long)n * G, 0, s));
      // the places: in assign, which holds a batch's labels only once they are used
      VP_LAUNCH(k_marker_count, bb, tb, q, p, idx, nb, g, ocnt, assign);
      VP_CALL(scan_int<true>(ocnt, n * G, ooff, stmp, s));
      if (runs)
        VP_LAUNCH(k_marker_place<true>, bb, tb, q, p, w, idx, nb, g, ooff, assign, orec, bperm, bq,
                  bp, bw);
      else
        VP_LAUNCH(k_marker_place<false>, bb, tb, q, p, w, idx, nb, g, ooff, assign, orec, bperm, bq,
                  bp, bw);
      for (int t = 0; t < n; ++t) {
        const Marker* const r = orec + (size_t)t * batch;
        if (runs) {
          VP_LAUNCH(k_assign<true>, ba, ta, r, bq, bp, nb, bperm, co.cq, co.cp, g, coff, cc, clab,
                    origid, lab0, 0, assign, cnt, slot, ccnt, cells0, k, over);
          VP_CALL(group_runs(nb));
          VP_LAUNCH(k_group<kGroupBatch>, gb, gt, r, assign, off, mem, k, per_b, g, L, co, mo,
                    origid, over, cnt0);
        } else {
          VP_LAUNCH(k_assign<false>, ba, ta, r, bq, bp, nb, bperm, co.cq, co.cp, g, coff, cc, clab,
                    origid, lab0, 0, assign, cnt, slot, ccnt, cells0, k, over);
          VP_CALL(group_markers(nb, k, assign, cnt, off, keys_a, vals_a, keys_b, vals_b, hist, hoff,
                                stmp, &order, s));
          VP_LAUNCH(k_minibatch_update, dim3(blocks_for(k, 64)), dim3(64), bq, bp, bw, off, order,
                    k, g, co);
        }
        VP_CALL(bin_centres());
      }
    }
    VP_CALL(fill_int(bcnt, G, 0, s));
    VP_CALL(order_markers(bcnt, boff));
  }
  for (int it = 0; it <= iters; ++it) {
    const bool last = it == iters;  // the last pass only assigns, and gives the moments
    if (runs) {
      VP_LAUNCH(k_assign<true>, ma, ta, rec, q, p, m, perm, co.cq, co.cp, g, coff, cc, clab, origid,
                lab0, it > 0 ? 1 : 0, assign, cnt, slot, ccnt, cells0, k, over);
      VP_CALL(group_runs(m));
      if (last)
        VP_LAUNCH(k_group<kGroupMoments>, gm, gt, rec, assign, off, mem, k, per_m, g, L, co, mo,
                  origid, over, cnt0);
      else
        VP_LAUNCH(k_group<kGroupMean>, gm, gt, rec, assign, off, mem, k, per_m, g, L, co, mo,
                  origid, over, cnt0);
    } else {
      VP_LAUNCH(k_assign<false>, ma, ta, rec, q, p, m, perm, co.cq, co.cp, g, coff, cc, clab, origid,
                lab0, it > 0 ? 1 : 0, assign, cnt, slot, ccnt, cells0, k, over);
      VP_CALL(group_markers(m, k, assign, cnt, off, keys_a, vals_a, keys_b, vals_b, hist, hoff,
                            stmp, &order, s));
      if (last)
        VP_LAUNCH(k_moments, dim3(blocks_for(k, 64)), dim3(64), q, p, w, off, order, k, L, origid,
                  mo);
      else
        VP_LAUNCH(k_centres, dim3(blocks_for(k, 64)), dim3(64), q, p, w, off, order, k, g, co);
    }
    if (!last) VP_CALL(bin_centres());
  }
  VP_CALL(scan_int<false>(mo.flag, k, pos, stmp, s));
  VP_LAUNCH(k_compact, kb, tb, pos, k, mo, Q, P, qs, ps, psi, over, res);
  if (nbatch > 0 && absorbed_out)
    VP_LAUNCH(k_absorbed_out, kb, tb, co.v, origid, k, absorbed_out, over);
  if (assign_out)
    VP_LAUNCH(k_assign_out, mb, tb, assign, runs ? rec : (const Marker*)nullptr, origid, m,
              assign_out, over);
#undef VP_LAUNCH
#undef VP_CALL
  if ((e = hipMemcpyAsync(host_res, res, 2 * sizeof(int), hipMemcpyDeviceToHost, s)) != hipSuccess)
    return e;
  return hipStreamSynchronize(s);
}

}  // namespace vpk
