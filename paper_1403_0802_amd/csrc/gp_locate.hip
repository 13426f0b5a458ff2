// Locator: the grid's exact per-point index, and the queries that read it.
//
// The paper's refinement tests every point of a cell against every edge of the cell's
// candidates (Sec. III.B-C).  For a resident feature set most of those tests have the
// same outcome for every point of the cell, or of a small part of it, so the grid build
// settles them once: each cell is cut into k x k subcells (k a power of two, per cell),
// and a subcell keeps only what can still differ between its points.
//
//   PIP   per candidate polygon, in id order, the parity of everything that is constant
//         over the subcell, the edges whose crossing predicate is not, and the vertices
//         where a chain of edges right of the subcell begins or ends inside its y band.
//         Polygons with nothing left are either skipped or end the list (the subcell lies
//         inside them).  Most subcells have a single answer and no list.
//   P2P   the segments that can be the nearest within D of some point of the subcell.
//
// A query is one kernel: a point per lane finds its subcell and evaluates the few entries
// left with the FP64 predicates in the definition's operation order, so ids and distances
// are those of the definition, whatever the precision form.  No sort, no work items and no
// scattered result stores: the kernel reads 16 bytes and writes 4 or 12 per point in the
// caller's order, and is bound by the gathers of the index.
//
// Every bound of the build is conservative: boxes are padded by more than the rounding of
// a point's cell and subcell, thresholds by more than the rounding of the FP64 predicates,
// and comparisons keep an entry when a bound is NaN.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "gp_internal.h"

namespace gp {

#define GP_WAVE 64

namespace {

__device__ __forceinline__ uint64_t ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }
__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << lane_id()) - 1ull; }
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// *p = max(*p, v): an atomic only where the value seen is smaller.
__device__ __forceinline__ void raise_to(unsigned long long *p, unsigned long long v) {
  if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, v);
}

unsigned blocks_for(int64_t n, int64_t per, int64_t cap) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + per - 1) / per, cap));
}

// Place of cell c in the order of the index: tiles of 16 x 16 cells, row by row, and the
// cells of a tile row by row.  A neighbourhood of cells then lies in few pages, as the
// address translation of a compute unit needs where points cluster.
__device__ __forceinline__ int32_t tiled_rank(int32_t c, int32_t nx, int32_t ny) {
  const int32_t x = c % nx, y = c / nx;
  const int32_t tx = x & ~15, ty = y & ~15;
  const int32_t w = nx - tx < 16 ? nx - tx : 16, h = ny - ty < 16 ? ny - ty : 16;
  return ty * nx + tx * h + (y - ty) * w + (x - tx);
}

// What the first passes of the build visit: the edges of every cell's candidate polygons, or
// the segments of its candidates' near ranges (`near`, P2P).  out[0] += their number over all
// cells, out[1] = max(that of a cell).  One wave per cell; an atomic per workgroup.
__global__ __launch_bounds__(256) void k_loc_work(const int32_t *cand_off, const int32_t *cand_id,
                                                  const int32_t *eoff, const int2 *near,
                                                  int32_t ncells, unsigned long long *out) {
  __shared__ unsigned long long part[2][256 / GP_WAVE];
  const int32_t nw = (int32_t)(gridDim.x * (blockDim.x / GP_WAVE));
  unsigned long long all = 0, most = 0;
  for (int32_t c = uniform((int32_t)(blockIdx.x * (blockDim.x / GP_WAVE) + threadIdx.x / GP_WAVE));
       c < ncells; c += nw) {
    const int32_t k1 = cand_off[c + 1];
    unsigned long long t = 0;
    for (int32_t k = cand_off[c] + (int32_t)lane_id(); k < k1; k += GP_WAVE) {
      const int32_t f = cand_id[k];
      t += (unsigned long long)(near ? near[k].y - near[k].x : eoff[f + 1] - eoff[f]);
    }
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, GP_WAVE);
    all += t;
    most = most > t ? most : t;
  }
  if (lane_id() == 0) {
    part[0][threadIdx.x / GP_WAVE] = all;
    part[1][threadIdx.x / GP_WAVE] = most;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / GP_WAVE; ++w) {
      all += part[0][w];
      most = most > part[1][w] ? most : part[1][w];
    }
    if (all) {
      atomicAdd(out, all);
      atomicMax(out + 1, most);
    }
  }
}

// ------------------------------------------------------------------------- PIP build

// x of the stand-ins for chains of edges right of a subcell: far right of any point (the
// build refuses coordinates of 1e150 and more), so such an edge's crossing is its straddle
// lo.y <= p.y < hi.y alone: (p.x - X) * h < 0 * (p.y - lo.y) holds for every h > 0,
// infinity included.
constexpr double kFarX = 1e300;

enum { LOC_NEVER = 0, LOC_RIGHT = 1, LOC_GUARD = 2 };

struct Box {
  double x0, y0, x1, y1;
};

// What edge e = (lo.x, lo.y, hi.x, hi.y) does for the points of box b: NEVER crosses;
// RIGHT: the x part of the predicate holds for every point, so the crossing is the
// straddle of p.y; GUARD: anything else.  The x part, (p.x - lo.x) h < w (p.y - lo.y), is
// the sign of a function linear in p, so its extremes over the box are at the corners; tol
// is over 50 times the rounding of the operations that evaluate it, here and at any point
// of the box (and never 0, so a sign lost to underflow is GUARD).
__device__ __forceinline__ int loc_class(const double4 e, const Box &b) {
  if (e.w <= b.y0 || e.y > b.y1) return LOC_NEVER;
  if (e.x >= 0.5 * kFarX) return LOC_RIGHT;
  if (e.y == e.w) return fmin(e.x, e.z) > b.x1 ? LOC_RIGHT : LOC_NEVER;
  const double h = e.w - e.y, w = e.z - e.x;
  const double ax = (b.x0 - e.x) * h, bx = (b.x1 - e.x) * h;
  const double ay = w * (b.y0 - e.y), by = w * (b.y1 - e.y);
  const double lo = ax - fmax(ay, by), hi = bx - fmin(ay, by);
  const double tol = 0x1p-44 * (fmax(fabs(ax), fabs(bx)) + fmax(fabs(ay), fabs(by))) + 0x1p-900;
  if (hi < -tol) return LOC_RIGHT;
  if (lo > tol) return LOC_NEVER;
  return LOC_GUARD;
}

// Ring predecessor of every vertex (edge v joins vertex v and its ring successor).
__global__ void k_loc_ring_prev(const int32_t *rvo, int32_t nr, int32_t *prev) {
  for (int32_t r = blockIdx.x; r < nr; r += gridDim.x) {
    const int32_t v0 = rvo[r], v1 = rvo[r + 1];
    for (int32_t v = v0 + (int32_t)threadIdx.x; v < v1; v += blockDim.x)
      prev[v] = v == v0 ? v1 - 1 : v - 1;
  }
}

__device__ __forceinline__ Box cell_box(uint32_t cell, int32_t nx, double x0, double y0,
                                        double cs, double pad) {
  const double bx = x0 + (double)(cell % (uint32_t)nx) * cs;
  const double by = y0 + (double)(cell / (uint32_t)nx) * cs;
  return Box{bx - pad, by - pad, bx + cs + pad, by + cs + pad};
}

// Elements of every (cell, candidate polygon) pair, one wave per pair, lanes over the
// polygon's vertices in ring order: the guarded edges, and each vertex in the cell's y band
// with exactly one RIGHT edge.  The straddle of an edge (a, b) is [a.y <= y] xor [b.y <= y],
// so over a chain of RIGHT edges the inner vertices cancel and its two ends remain; a
// vertex v is kept as the far edge (v.y, +inf), whose straddle is [v.y <= y].  Ends below
// the band are 1 for every point and go into the pair's parity.
template <bool EMIT>
__global__ __launch_bounds__(256) void k_loc_pip_pairs(
    const uint32_t *pair_cell, const int32_t *cand_id, int32_t npairs, const int32_t *eoff,
    const double4 *edge64, const double *vy, const int32_t *prev, double x0, double y0,
    double cs, int32_t nx, double pad, uint32_t *cnt, uint8_t *par, double4 *elem) {
  const uint64_t lt = lanemask_lt();
  const int32_t nw = (int32_t)(gridDim.x * (blockDim.x / GP_WAVE));
  for (int32_t k = uniform((int32_t)(blockIdx.x * (blockDim.x / GP_WAVE) + threadIdx.x / GP_WAVE));
       k < npairs; k += nw) {
    const Box b = cell_box(pair_cell[k], nx, x0, y0, cs, pad);
    const int32_t f = cand_id[k], e1 = eoff[f + 1];
    uint32_t n = EMIT ? cnt[k] : 0u;  // EMIT: cnt holds the pairs' first elements
    uint32_t odd = 0;
    for (int32_t base = eoff[f]; base < e1; base += GP_WAVE) {
      const int32_t v = base + (int32_t)lane_id();
      bool guard = false, end = false, below = false;
      double4 e;
      double y = 0.0;
      if (v < e1) {
        e = edge64[v];
        y = vy[v];
        const int c = loc_class(e, b), cp = loc_class(edge64[prev[v]], b);
        guard = c == LOC_GUARD;
        const bool brk = (c == LOC_RIGHT) != (cp == LOC_RIGHT);
        below = brk && y <= b.y0;
        end = brk && y > b.y0 && y <= b.y1;
      }
      const uint64_t mg = ballot(guard), me = ballot(end);
      odd ^= (uint32_t)__popcll(ballot(below)) & 1u;
      if constexpr (EMIT) {
        uint32_t at = n + (uint32_t)(__popcll(mg & lt) + __popcll(me & lt));
        if (end) elem[at++] = make_double4(kFarX, y, kFarX, INFINITY);
        if (guard) elem[at] = e;
      }
      n += (uint32_t)(__popcll(mg) + __popcll(me));
    }
    if (!EMIT && lane_id() == 0) {
      cnt[k] = n;
      par[k] = (uint8_t)odd;
    }
  }
}

// Elements of every cell up to the first polygon that contains the whole cell, and the
// cell's answer when there are none.  eoffs[k] are the pairs' first elements.  shape
// [c] = log2 k, or LOC_CONST; cost[0] += subcells, cost[1] += subcells * elements,
// cost[2] += groups of the list builder, cost[3] = max(elements).
constexpr uint32_t LOC_CONST = 0xffu;

// A wave of the list builders takes a group of subcells: an 8 x 8 block, or the whole of a
// cell with fewer.
__device__ __forceinline__ uint32_t group_count(uint32_t m) {
  return m > 3 ? 1u << (2 * (m - 3)) : 1u;
}

// log2 of the subdivision for a cell with E elements: about E / 4 subcells along a side, so
// that a boundary crossing the cell leaves a few elements in the subcells it meets.  At
// half the limits 50M points of the region map take 0.89 instead of 0.92 ms with 28% more
// memory and a 7% longer build, at 2.5 times the limits 1.02 ms with 23% less memory.
__device__ __forceinline__ uint32_t pip_shape(uint32_t E, uint32_t cap) {
  const uint32_t m = E <= 4 ? 2u : E <= 24 ? 3u : E <= 96 ? 4u : E <= 384 ? 5u : 6u;
  return m < cap ? m : cap;
}

__global__ __launch_bounds__(256) void k_loc_pip_cells(const int32_t *cand_off,
                                                       const int32_t *cand_id, int32_t nx,
                                                       int32_t ny, const uint32_t *eoffs, const uint8_t *par,
                                                       uint32_t cap, uint32_t *nsub,
                                                       LocCell *cell,
                                                       unsigned long long *cost) {
  const int32_t ncells = nx * ny;
  unsigned long long s0 = 0, s1 = 0, s2 = 0, most = 0;
  for (int32_t c = blockIdx.x * blockDim.x + threadIdx.x; c <= ncells;
       c += gridDim.x * blockDim.x) {
    uint32_t E = 0;
    int32_t ans = -1;
    if (c < ncells) {
      const int32_t k1 = cand_off[c + 1];
      for (int32_t k = cand_off[c]; k < k1; ++k) {
        const uint32_t n = eoffs[k + 1] - eoffs[k];
        E += n;
        if (n == 0 && par[k]) {
          ans = cand_id[k];
          break;
        }
      }
      const uint32_t m = pip_shape(E, cap);
      const uint32_t q = E ? 1u << (2 * m) : 0u;
      nsub[tiled_rank(c, nx, ny)] = q;
      cell[c] = LocCell{(uint32_t)ans, E ? m : LOC_CONST};
      s0 += q;
      s1 += (unsigned long long)q * E;
      s2 += E ? group_count(m) : 0u;
      most = most > E ? most : E;
    } else {
      nsub[c] = 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off, GP_WAVE);
    s1 += __shfl_xor(s1, off, GP_WAVE);
    s2 += __shfl_xor(s2, off, GP_WAVE);
    const unsigned long long o = __shfl_xor(most, off, GP_WAVE);
    most = most > o ? most : o;
  }
  if (lane_id() == 0 && s1) {
    atomicAdd(cost, s0);
    atomicAdd(cost + 1, s1);
    atomicAdd(cost + 2, s2);
    raise_to(cost + 3, most);
  }
}

// Subcell base of every divided cell, from the scan of nsub.
template <class Cell>
__global__ void k_loc_cell_base(const uint32_t *base, int32_t nx, int32_t ny, Cell *cell) {
  for (int32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < nx * ny; c += gridDim.x * blockDim.x)
    if (cell[c].m != LOC_CONST) cell[c].base = base[tiled_rank(c, nx, ny)];
}

// The groups (cell, block), in no particular order.  One atomic per wave.
template <class Cell>
__global__ __launch_bounds__(256) void k_loc_groups(const Cell *cell, int32_t ncells,
                                                    uint32_t *n, int2 *group) {
  for (int32_t c0 = blockIdx.x * blockDim.x; c0 < ncells; c0 += gridDim.x * blockDim.x) {
    const int32_t c = c0 + (int32_t)threadIdx.x;
    const uint32_t m = c < ncells ? cell[c].m : LOC_CONST;
    const uint32_t q = m == LOC_CONST ? 0u : group_count(m);
    uint32_t inc = q;
#pragma unroll
    for (int off = 1; off < GP_WAVE; off <<= 1) {
      const uint32_t u = __shfl_up(inc, off, GP_WAVE);
      if (lane_id() >= (uint32_t)off) inc += u;
    }
    uint32_t o = 0;
    if (lane_id() == GP_WAVE - 1 && inc) o = atomicAdd(n, inc);
    o = (uint32_t)__builtin_amdgcn_readlane((int32_t)o, GP_WAVE - 1) + inc - q;
    for (uint32_t k = 0; k < q; ++k) group[o + k] = make_int2(c, (int32_t)k);
  }
}

// The lane's subcell of a group: column, row and whether it exists; the group's columns and
// rows start at gx, gy and it is gw subcells wide.
struct GroupLane {
  int32_t gx, gy, gw, sx, sy;
  bool act;
};
__device__ __forceinline__ GroupLane group_lane(uint32_t m, int32_t block) {
  GroupLane g;
  g.gw = m > 3 ? 8 : 1 << m;
  const int32_t bw = m > 3 ? 1 << (m - 3) : 1;  // blocks along a side
  g.gx = block % bw * 8;
  g.gy = block / bw * 8;
  const int32_t l = (int32_t)lane_id();
  g.act = l < g.gw * g.gw;
  g.sx = g.gx + l % g.gw;
  g.sy = g.gy + (l / g.gw) % g.gw;  // idle lanes repeat the active ones' places
  return g;
}

// A subcell's list: per polygon a header slot (int4 x 2: id, elements << 1 | parity, 1 if
// another polygon follows, the id that ends the list or -1) and its elements.
struct alignas(32) LocHead {
  int32_t f, npar, more, last, pad[4];
};
static_assert(sizeof(LocHead) == sizeof(double4), "a header takes one slot");

// Lists of the subcells, one wave per group, lanes over its subcells.  The cell's elements
// pass 64 at a time, a lane each, and those that cannot cross anywhere in the group are
// dropped; the rest are broadcast through LDS.  Elements that are RIGHT for a subcell are
// merged along their chains: a run is the far edge {ra, rb} standing for the edges merged
// so far, and an edge that shares an end with it (by y, which is all its straddle depends
// on) extends it.  Ends outside the subcell's band count as -inf or +inf, so a chain that
// leaves the band and returns merges too, and one that passes through it becomes a constant.
// EMIT = false: slots per subcell in cnt (0: a single answer).  EMIT: cnt holds the first
// slots; writes the lists and sub[s] = answer (>= -1) or -(first slot + 2).
template <bool EMIT>
__global__ __launch_bounds__(256) void k_loc_pip_sub(
    const int32_t *cand_off, const int32_t *cand_id, const int2 *group, uint32_t ngroups,
    const uint32_t *eoffs, const uint8_t *par, const double4 *elem, const LocCell *cell,
    double x0, double y0, double cs, int32_t nx, double pad, uint32_t *cnt, double4 *slot,
    int32_t *sub) {
  __shared__ double4 se[256 / GP_WAVE][GP_WAVE];
  const int wave = (int)(threadIdx.x / GP_WAVE);
  const uint32_t w = (uint32_t)uniform((int32_t)(blockIdx.x * (blockDim.x / GP_WAVE)) + wave);
  if (w >= ngroups) return;
  const int2 gr = group[w];
  const int32_t c = uniform(gr.x);
  const LocCell ce = cell[c];
  const GroupLane g = group_lane(ce.m, uniform(gr.y));
  const double a = cs / (double)(1u << ce.m);  // exact: a power of two
  const double ox = x0 + (double)(c % nx) * cs, oy = y0 + (double)(c / nx) * cs;
  const double gx = ox + (double)g.gx * a, gy = oy + (double)g.gy * a, gs = (double)g.gw * a;
  const Box gb{gx - pad, gy - pad, gx + gs + pad, gy + gs + pad};
  const double sx = ox + (double)g.sx * a, sy = oy + (double)g.sy * a;
  const Box b{sx - pad, sy - pad, sx + a + pad, sy + a + pad};
  const uint32_t at = ce.base + ((uint32_t)g.sy << ce.m) + (uint32_t)g.sx;
  const uint32_t first = EMIT && g.act ? cnt[at] : 0u;
  uint32_t n = 0;     // slots so far
  uint32_t hpos = 0;  // open header (EMIT)
  LocHead hd{-1, 0, 0, -1, {0, 0, 0, 0}};
  bool open = false, done = !g.act;
  int32_t last = -1;
  const int32_t k1 = cand_off[c + 1];
  for (int32_t k = cand_off[c]; k < k1; ++k) {
    if (ballot(!done) == 0) break;
    const uint32_t e0 = (uint32_t)uniform((int32_t)eoffs[k]);
    const uint32_t e1 = (uint32_t)uniform((int32_t)eoffs[k + 1]);
    uint32_t p = par[k];
    uint32_t m = 0;  // this polygon's elements here
    double ra = 0.0, rb = 0.0;
    const uint32_t hslot = n;
    auto put = [&](const double4 e) {
      if (EMIT && !done) slot[first + hslot + 1 + m] = e;
      ++m;
    };
    auto flush = [&]() {
      if (ra != rb) {
        const double lo = fmin(ra, rb), hi = fmax(ra, rb);
        if (lo == -INFINITY) {
          p ^= 1u;
          if (hi != INFINITY) put(make_double4(kFarX, hi, kFarX, INFINITY));
        } else {
          put(make_double4(kFarX, lo, kFarX, hi));
        }
      }
      ra = rb = 0.0;
    };
    for (uint32_t j0 = e0; j0 < e1; j0 += GP_WAVE) {
      const uint32_t j = j0 + lane_id();
      double4 mine;
      bool use = false;
      if (j < e1) {
        mine = elem[j];
        use = loc_class(mine, gb) != LOC_NEVER;
      }
      const uint64_t mk = ballot(use);
      wave_lds_sync();
      if (use) se[wave][__popcll(mk & lanemask_lt())] = mine;
      wave_lds_sync();
      const int nu = (int)__popcll(mk);
      for (int q = 0; q < nu; ++q) {
        const double4 e = se[wave][q];
        const int cl = loc_class(e, b);
        if (cl == LOC_GUARD) {
          put(e);
        } else if (cl == LOC_RIGHT) {
          const double l = e.y <= b.y0 ? -INFINITY : e.y;
          const double h = e.w > b.y1 ? INFINITY : e.w;
          if (ra == rb) { ra = l; rb = h; }
          else if (l == rb) rb = h;
          else if (h == rb) rb = l;
          else if (l == ra) ra = h;
          else if (h == ra) ra = l;
          else { flush(); ra = l; rb = h; }
        }
      }
    }
    flush();
    if (done) continue;
    const int32_t f = cand_id[k];
    if (m == 0) {
      if (p) {
        last = f;
        done = true;
      }
      continue;
    }
    if (EMIT) {
      if (open) {
        hd.more = 1;
        *(LocHead *)&slot[first + hpos] = hd;
      }
      hd.f = f;
      hd.npar = (int32_t)(m << 1 | p);
      hpos = hslot;
    }
    open = true;
    n += 1 + m;
  }
  if (!g.act) return;
  if (EMIT) {
    if (open) {
      hd.more = 0;
      hd.last = last;
      *(LocHead *)&slot[first + hpos] = hd;
    }
    sub[at] = open ? -(int32_t)(first + 2u) : last;
  } else {
    cnt[at] = n;
  }
}

// ------------------------------------------------------------------------- P2P build

// Squared distance from c to the segment a + t d, t in [0, 1]; inv = 1 / |d|^2 (0 for a
// zero-length segment).  For the build's bounds only.
__device__ __forceinline__ double seg_dist2(double cx, double cy, double ax, double ay,
                                            double dx, double dy, double inv) {
  const double wx = cx - ax, wy = cy - ay;
  const double t = fmin(fmax(fma(wx, dx, wy * dy) * inv, 0.0), 1.0);
  const double ex = fma(-t, dx, wx), ey = fma(-t, dy, wy);
  return fma(ex, ex, ey * ey);
}

// A segment g can only be the nearest within D of a point p of a box with centre c and
// half diagonal r when d(c, g) <= min(d(c, u) + 2 r, D + r) for every other segment u:
// otherwise d(p, g) >= d(c, g) - r > d(c, u) + r >= d(p, u), or > D.  slack is over 100
// times the rounding of the FP64 distances, here and in the definition.
__device__ __forceinline__ double keep_limit2(double dmin2, double r, double D, double slack) {
  const double t = fmin(sqrt(dmin2) + 2.0 * r, D + r) + slack;
  return t * t;
}

// Segments of every cell, one wave per cell: the candidates' near-segment ranges laid end
// to end, 64 segments per step.  EMIT = false: counts and the squared distance of the
// nearest segment to the cell's centre; EMIT: cnt holds the first entries, writes the
// segments, ascending.
template <bool EMIT>
__global__ __launch_bounds__(256) void k_loc_cell_segs(
    const int32_t *cand_off, const int2 *near, const double4 *edge64, int32_t ncells, double x0,
    double y0, double cs, int32_t nx, double r, double D,
    double slack, uint32_t *cnt, double *cmin, int32_t *list) {
  __shared__ int32_t win[256 / GP_WAVE][2 * GP_WAVE];
  int32_t *wseg = win[threadIdx.x / GP_WAVE], *wstart = wseg + GP_WAVE;
  const uint32_t lane = lane_id();
  const int32_t nw = (int32_t)(gridDim.x * (blockDim.x / GP_WAVE));
  for (int32_t c = uniform((int32_t)(blockIdx.x * (blockDim.x / GP_WAVE) + threadIdx.x / GP_WAVE));
       c < ncells; c += nw) {
    const int32_t k0 = cand_off[c], k1 = cand_off[c + 1];
    const double cx = x0 + ((double)(c % nx) + 0.5) * cs, cy = y0 + ((double)(c / nx) + 0.5) * cs;
    double dmin = EMIT ? cmin[c] : INFINITY;
    uint32_t n = EMIT ? cnt[c] : 0u;
    for (int sweep = EMIT ? 1 : 0; sweep < 2; ++sweep) {
      const double lim2 = keep_limit2(dmin, r, D, slack);
      for (int32_t kw = k0; kw < k1; kw += GP_WAVE) {
        const int32_t kk = kw + (int32_t)lane;
        const int nk = k1 - kw < GP_WAVE ? k1 - kw : GP_WAVE;
        int32_t s0 = 0, len = 0;
        if (kk < k1) {
          const int2 nr = near[kk];
          s0 = nr.x;
          len = nr.y - nr.x;
        }
        uint32_t inc = (uint32_t)len;
#pragma unroll
        for (int off = 1; off < GP_WAVE; off <<= 1) {
          const uint32_t u = __shfl_up(inc, off, GP_WAVE);
          if (lane >= (uint32_t)off) inc += u;
        }
        const int32_t total = __builtin_amdgcn_readlane((int32_t)inc, GP_WAVE - 1);
        wave_lds_sync();
        wseg[lane] = s0;
        wstart[lane] = (int32_t)inc - len;
        wave_lds_sync();
        int w = 0;  // this lane's candidate in the window (its flat indices only grow)
        for (int32_t F0 = 0; F0 < total; F0 += GP_WAVE) {
          const int32_t F = F0 + (int32_t)lane;
          double d2 = INFINITY;
          int32_t sg = 0;
          if (F < total) {
            while (w + 1 < nk && wstart[w + 1] <= F) ++w;
            sg = wseg[w] + (F - wstart[w]);
            const double4 e = edge64[sg];
            const double dx = e.z - e.x, dy = e.w - e.y, L2 = dx * dx + dy * dy;
            d2 = seg_dist2(cx, cy, e.x, e.y, dx, dy, L2 > 0.0 ? 1.0 / L2 : 0.0);
          }
          if (sweep == 0) {
            dmin = fmin(dmin, d2);
          } else {
            const bool keep = F < total && !(d2 > lim2);
            const uint64_t m = ballot(keep);
            if (EMIT && keep) list[n + (uint32_t)__popcll(m & lanemask_lt())] = sg;
            n += (uint32_t)__popcll(m);
          }
        }
      }
      if (sweep == 0)
        for (int off = 32; off > 0; off >>= 1) dmin = fmin(dmin, __shfl_xor(dmin, off, GP_WAVE));
    }
    if (!EMIT && lane == 0) {
      cnt[c] = n;
      cmin[c] = dmin;
    }
  }
}

// Subdivision of a cell of n segments: k such that n / k is about `target` (segments per
// subcell fall like 1 / k where D does not bound them).
__device__ __forceinline__ uint32_t p2p_shape(uint32_t n, uint32_t target, uint32_t cap) {
  uint32_t m = 0;
  while (m < cap && (n >> m) > target) ++m;
  return m;
}

// reach of a cell: no point of it has its nearest segment within D farther away.
// cost[0] += subcells, cost[1] += subcells * segments, cost[2] += expected entries,
// cost[3] += groups of the list builder, cost[4] = max(segments).
__global__ __launch_bounds__(256) void k_loc_p2p_cells(const uint32_t *first, const double *cmin,
                                                       int32_t nx, int32_t ny, double r,
                                                       double D, double slack, uint32_t target,
                                                       uint32_t cap, uint32_t *nsub,
                                                       LocSegCell *cell,
                                                       unsigned long long *cost) {
  const int32_t ncells = nx * ny;
  unsigned long long s0 = 0, s1 = 0, s2 = 0, s3 = 0, most = 0;
  for (int32_t c = blockIdx.x * blockDim.x + threadIdx.x; c <= ncells;
       c += gridDim.x * blockDim.x) {
    if (c < ncells) {
      const uint32_t n = first[c + 1] - first[c];
      const uint32_t m = p2p_shape(n, target, cap);
      const uint32_t q = n ? 1u << (2 * m) : 0u;
      nsub[tiled_rank(c, nx, ny)] = q;
      cell[c].m = n ? m : LOC_CONST;
      cell[c].reach = fmin(sqrt(cmin[c]) + r, D) + slack;
      s0 += q;
      s1 += (unsigned long long)q * n;
      s2 += (unsigned long long)n << m;
      s3 += n ? group_count(m) : 0u;
      most = most > n ? most : n;
    } else {
      nsub[c] = 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off, GP_WAVE);
    s1 += __shfl_xor(s1, off, GP_WAVE);
    s2 += __shfl_xor(s2, off, GP_WAVE);
    s3 += __shfl_xor(s3, off, GP_WAVE);
    const unsigned long long o = __shfl_xor(most, off, GP_WAVE);
    most = most > o ? most : o;
  }
  if (lane_id() == 0 && s0) {
    atomicAdd(cost, s0);
    atomicAdd(cost + 1, s1);
    atomicAdd(cost + 2, s2);
    atomicAdd(cost + 3, s3);
    raise_to(cost + 4, most);
  }
}

// Segments by value with their polyline, 64 bytes each, in the order of the index's cells (by
// the cell of the midpoint), so that segments near each other share lines and pages.
// *flag becomes 1 where a segment that is not a point has |d|^2 below min_L2.
__global__ void k_loc_seg_keys(const double4 *edge64, int32_t n, double x0, double y0, double cs,
                               int32_t nx, int32_t ny, double min_L2, uint32_t *key,
                               uint32_t *flag) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const double4 e = edge64[i];
    const double dx = e.z - e.x, dy = e.w - e.y;
    if ((dx != 0.0 || dy != 0.0) && dx * dx + dy * dy < min_L2) atomicOr(flag, 1u);
    const double fx = floor((0.5 * (e.x + e.z) - x0) / cs), fy = floor((0.5 * (e.y + e.w) - y0) / cs);
    const int32_t x = (int32_t)fmin(fmax(fx, 0.0), (double)(nx - 1));
    const int32_t y = (int32_t)fmin(fmax(fy, 0.0), (double)(ny - 1));
    key[i] = (uint32_t)tiled_rank(y * nx + x, nx, ny);
  }
}

__global__ __launch_bounds__(256) void k_loc_polylines(const int32_t *eoff, int32_t nf, int32_t *f) {
  const int32_t nw = (int32_t)(gridDim.x * (blockDim.x / GP_WAVE));
  for (int32_t q = (int32_t)(blockIdx.x * (blockDim.x / GP_WAVE) + threadIdx.x / GP_WAVE); q < nf;
       q += nw)
    for (int32_t e = eoff[q] + (int32_t)lane_id(); e < eoff[q + 1]; e += GP_WAVE) f[e] = q;
}

// place[old] = new, from the sorted order.
__global__ void k_loc_segments(const uint32_t *order, const int32_t *f, const double4 *edge64,
                               int32_t n, LocSeg *seg, int32_t *place) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int32_t o = (int32_t)order[i];
    seg[i].e = edge64[o];
    seg[i].f = f[o];
    place[o] = i;
  }
}

__global__ void k_loc_add(uint32_t *v, size_t n, uint32_t d) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    v[i] += d;
}

// Frame of a cell's entries: the cell widened by its reach on every side, in LOC_UNITS
// steps.  An entry is the part of its segment inside the frame, endpoints rounded to whole
// steps: for a point of the cell that distance is within 0.71 steps of the segment's
// wherever the segment's nearest point is inside the frame, and at least the reach
// otherwise, when the segment cannot be the answer.
constexpr double LOC_UNITS = 65535.0;

__device__ __forceinline__ uint2 quantised(const double4 e, double ox, double oy, double side) {
  const double dx = e.z - e.x, dy = e.w - e.y;
  double t0 = 0.0, t1 = 1.0;
  bool in = true;
  auto clip = [&](double q, double d) {  // keeps q + t d >= 0
    if (d == 0.0) {
      in &= q >= 0.0;
    } else {
      const double t = -q / d;
      if (d > 0.0) t0 = fmax(t0, t);
      else t1 = fmin(t1, t);
    }
  };
  clip(e.x - ox, dx);
  clip(ox + side - e.x, -dx);
  clip(e.y - oy, dy);
  clip(oy + side - e.y, -dy);
  if (!in || !(t0 <= t1)) return make_uint2(0u, 0u);  // outside: the frame's corner
  const double f = LOC_UNITS / side;
  auto q = [&](double v) { return (uint32_t)fmin(fmax(v * f + 0.5, 0.0), LOC_UNITS); };
  // an endpoint inside is taken as it is
  const double ax = t0 > 0.0 ? e.x + t0 * dx : e.x, ay = t0 > 0.0 ? e.y + t0 * dy : e.y;
  const double bx = t1 < 1.0 ? e.x + t1 * dx : e.z, by = t1 < 1.0 ? e.y + t1 * dy : e.w;
  return make_uint2(q(ax - ox) | q(ay - oy) << 16, q(bx - ox) | q(by - oy) << 16);
}

// Lists of the subcells, one wave per group, lanes over its subcells.  The cell's segments
// pass 64 at a time, a lane each, and those that cannot be the nearest anywhere in the
// group (by the same rule, with the group's box) are dropped; the rest are broadcast
// through LDS.  A list is ordered by rings around the subcell's centre, LOC_RINGS of equal
// width from its nearest segment to its limit, so that a query can stop at the first block
// whose rings are too far.  The first blocks of subcell s are 2 s and 2 s + 1, one 128-byte
// line; the second gives up an entry for the index of the block that goes on.
// EMIT = false: blocks beyond the line per subcell in cnt, the distance of the nearest
// segment and the squared limit in lim; EMIT: cnt holds the first of those blocks.
constexpr int LOC_RINGS = 8;

template <bool EMIT>
__global__ __launch_bounds__(256) void k_loc_sub_segs(
    const uint32_t *first, const int32_t *list, const double4 *edge64, const int2 *group,
    uint32_t ngroups, const LocSegCell *cell, double x0, double y0, double cs, int32_t nx,
    double pad, double D, double slack, const int32_t *place, double *glim, uint32_t *cnt,
    double2 *lim, LocBlock *block) {
  __shared__ double4 sa[256 / GP_WAVE][GP_WAVE];  // a.x, a.y, d.x, d.y
  __shared__ double si[256 / GP_WAVE][GP_WAVE];   // 1 / |d|^2
  __shared__ uint2 sl[256 / GP_WAVE][GP_WAVE];    // the entry
  __shared__ int32_t sg[256 / GP_WAVE][GP_WAVE];  // the segment
  __shared__ uint32_t ring[LOC_RINGS + 1][256];   // EMIT: entries before each ring, per lane
  const int wave = (int)(threadIdx.x / GP_WAVE);
  const uint32_t lane = lane_id();
  const uint32_t w = (uint32_t)uniform((int32_t)(blockIdx.x * (blockDim.x / GP_WAVE)) + wave);
  if (w >= ngroups) return;
  const int2 gr = group[w];
  const int32_t c = uniform(gr.x);
  const LocSegCell ce = cell[c];
  const GroupLane g = group_lane(ce.m, uniform(gr.y));
  const double a = cs / (double)(1u << ce.m), gs = (double)g.gw * a;
  constexpr double kHalfDiag = 0.70710678118654757 * (1.0 + 0x1p-40);
  const double r = kHalfDiag * (a + 2.0 * pad), rg = kHalfDiag * (gs + 2.0 * pad);
  const double ox = x0 + (double)(c % nx) * cs, oy = y0 + (double)(c / nx) * cs;
  const double gx = ox + (double)g.gx * a + 0.5 * gs, gy = oy + (double)g.gy * a + 0.5 * gs;
  const double px = ox + ((double)g.sx + 0.5) * a, py = oy + ((double)g.sy + 0.5) * a;
  const uint32_t at = ce.base + ((uint32_t)g.sy << ce.m) + (uint32_t)g.sx;
  const uint32_t l0 = first[c], l1 = first[c + 1];
  double glim2;  // the group's limit
  if constexpr (!EMIT) {
    double gmin = INFINITY;
    for (uint32_t l = l0 + lane; l < l1; l += GP_WAVE) {
      const double4 e = edge64[list[l]];
      const double dx = e.z - e.x, dy = e.w - e.y, L2 = dx * dx + dy * dy;
      gmin = fmin(gmin, seg_dist2(gx, gy, e.x, e.y, dx, dy, L2 > 0.0 ? 1.0 / L2 : 0.0));
    }
    for (int off = 32; off > 0; off >>= 1) gmin = fmin(gmin, __shfl_xor(gmin, off, GP_WAVE));
    glim2 = keep_limit2(gmin, rg, D, slack);
    if (lane == 0) glim[w] = glim2;
  } else {
    glim2 = glim[w];
  }
  // the group's segments, broadcast one by one
  auto sweep = [&](auto &&meet) {
    for (uint32_t l = l0; l < l1; l += GP_WAVE) {
      bool use = false;
      int32_t seg = 0;
      double4 e;
      double dx = 0.0, dy = 0.0, inv = 0.0;
      if (l + lane < l1) {
        seg = list[l + lane];
        e = edge64[seg];
        dx = e.z - e.x;
        dy = e.w - e.y;
        const double L2 = dx * dx + dy * dy;
        inv = L2 > 0.0 ? 1.0 / L2 : 0.0;
        use = !(seg_dist2(gx, gy, e.x, e.y, dx, dy, inv) > glim2);
      }
      const uint64_t mk = ballot(use);
      wave_lds_sync();
      if (use) {
        const int q = (int)__popcll(mk & lanemask_lt());
        sa[wave][q] = make_double4(e.x, e.y, dx, dy);
        si[wave][q] = inv;
        if (EMIT) {
          sl[wave][q] = quantised(e, ox - ce.reach, oy - ce.reach, cs + 2.0 * ce.reach);
          sg[wave][q] = place[seg];
        }
      }
      wave_lds_sync();
      const int nu = (int)__popcll(mk);
      for (int q = 0; q < nu; ++q) {
        const double4 v = sa[wave][q];
        meet(q, seg_dist2(px, py, v.x, v.y, v.z, v.w, si[wave][q]));
      }
    }
  };
  if constexpr (!EMIT) {
    double dmin = INFINITY;
    sweep([&](int, double d2) { dmin = fmin(dmin, d2); });
    const double lim2 = keep_limit2(dmin, r, D, slack);
    uint32_t n = 0;
    sweep([&](int, double d2) { n += !(d2 > lim2); });
    if (g.act) {
      cnt[at] = n > LOC_LINE ? (n - LOC_LINE + LOC_ENTRIES - 1) / LOC_ENTRIES : 0u;
      lim[at] = make_double2(sqrt(dmin), lim2);
    }
  } else {
    const double2 dl = g.act ? lim[at] : make_double2(0.0, 0.0);
    const double lim2 = dl.y, step = (sqrt(lim2) - dl.x) * (1.0 / LOC_RINGS);
    // FP32, in units of the limit: within 2^-21 of the true place, which from ring 1 on is
    // under 2^-18 of the distance (against 7 FP64 compares an entry: 6.3 -> 5.6 ms for a map of
    // 5.3M segments in 200 x 200 cells)
    const double unit = lim2 > 1e-290 ? 1.0 / lim2 : 0.0;
    const float inner = (float)(dl.x * sqrt(unit)), rings = (float)LOC_RINGS / (1.0f - inner);
    auto ring_of = [&](double d2) {
      const float t = (__builtin_amdgcn_sqrtf((float)(d2 * unit)) - inner) * rings;
      return (int)fminf(fmaxf(t, 0.0f), (float)(LOC_RINGS - 1));
    };
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i <= LOC_RINGS; ++i) ring[i][tid] = 0;
    sweep([&](int, double d2) {
      if (!(d2 > lim2)) ++ring[ring_of(d2) + 1][tid];
    });
#pragma unroll
    for (int i = 1; i <= LOC_RINGS; ++i) ring[i][tid] += ring[i - 1][tid];
    const uint32_t n = ring[LOC_RINGS][tid];
    const uint32_t more = g.act ? cnt[at] : 0u;
    // block and slot of entry e
    auto block_of = [&](uint32_t e) {
      return e < LOC_LINE ? 2 * at + e / LOC_ENTRIES : more + (e - LOC_LINE) / LOC_ENTRIES;
    };
    auto slot_of = [](uint32_t e) { return (e < LOC_LINE ? e : e - LOC_LINE) % LOC_ENTRIES; };
    if (g.act) {
      // a block's `rest` is at most the distance to the centre of any later entry, in steps
      // of the frame; the last block's ends the list
      const double f = LOC_UNITS / (cs + 2.0 * ce.reach) * (1.0 - 0x1p-15);
      auto rest = [&](uint32_t e) {  // of the block before the one entry e begins
        int i = 0;
        while (i + 1 < LOC_RINGS && ring[i + 1][tid] <= e) ++i;
        return e < n ? (float)((dl.x + (double)i * step) * f) : INFINITY;
      };
      block[2 * at].rest = rest(LOC_ENTRIES);
      LocBlock &l = block[2 * at + 1];
      l.rest = rest(LOC_LINE);
      l.e[LOC_ENTRIES - 1] = LocEntry{more, 0u, -1};
      uint32_t e = LOC_LINE;
      for (; e < n; e += LOC_ENTRIES) block[block_of(e)].rest = rest(e + LOC_ENTRIES);
      for (uint32_t k = n; k < e; ++k)  // places without an entry
        block[block_of(k)].e[slot_of(k)] = LocEntry{0u, 0u, -1};
    }
    sweep([&](int q, double d2) {
      if (g.act && !(d2 > lim2)) {
        const uint32_t e = ring[ring_of(d2)][tid]++;
        block[block_of(e)].e[slot_of(e)] = LocEntry{sl[wave][q].x, sl[wave][q].y, sg[wave][q]};
      }
    });
  }
}

// ------------------------------------------------------------------------- queries

// The point's cell, as the pairing computes it (-1 when unpaired), and its place in the
// cell in units of a cell: fx - floor(fx) and its product with a power of two are exact.
__device__ __forceinline__ int32_t locate_cell(const LocArgs &a, double x, double y, double &ux,
                                               double &uy) {
  const double fx = (x - a.x0) / a.cs, fy = (y - a.y0) / a.cs;
  const double cx = floor(fx), cy = floor(fy);
  const bool ok = cx >= 0.0 && cx < (double)a.nx && cy >= 0.0 && cy < (double)a.ny;
  ux = fx - cx;
  uy = fy - cy;
  return ok ? (int32_t)cy * a.nx + (int32_t)cx : -1;
}

__device__ __forceinline__ uint32_t subcell(uint32_t base, uint32_t m, double ux, double uy) {
  const double k = (double)(1u << m);
  return base + ((uint32_t)(uy * k) << m) + (uint32_t)(ux * k);
}

// Zeroes the counters that k_locate_count adds to next on the same stream.
__device__ __forceinline__ void reset_counts(unsigned long long *counts) {
  if (counts && blockIdx.x == 0 && threadIdx.x < 3) counts[threadIdx.x] = 0;
}

// Adds a workgroup's candidate tests to one of the request's partial sums (a single counter
// would queue the atomics of all workgroups).
__device__ __forceinline__ void add_tests(LocServed *sv, unsigned long long t) {
  __shared__ unsigned long long sum[256 / GP_WAVE];
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, GP_WAVE);
  if (lane_id() == 0) sum[threadIdx.x / GP_WAVE] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / GP_WAVE; ++w) t += sum[w];
    if (t) atomicAdd(&sv->part[blockIdx.x % LOC_PARTS], t);
  }
}

// Hands a request to the kernels that follow on the stream, and its test count to the host
// after them (`tests` is pinned host memory).
__global__ void k_serve_begin(LocServed *sv, LocRequest r) {
  if (threadIdx.x == 0) sv->r = r;
  for (uint32_t i = threadIdx.x; i < LOC_PARTS; i += blockDim.x) sv->part[i] = 0;
}

__global__ void k_serve_end(const LocServed *sv) {
  unsigned long long t = threadIdx.x < LOC_PARTS ? sv->part[threadIdx.x] : 0;
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, GP_WAVE);
  if (threadIdx.x == 0) *sv->r.tests = t;
}

// The answer of a list: per polygon its header and elements, by the definition's predicate.
// A header's first element is read with it and every other one ahead of its turn, so that a
// lane does not wait out each slot's latency (50M points 0.98 -> 0.92 ms, 1M 0.030 -> 0.028).
__device__ __forceinline__ int32_t list_answer(const double4 *s, double x, double y) {
  for (;;) {
    const int4 hd = *(const int4 *)s;  // id, elements << 1 | parity, more, last
    double4 e = s[1];                  // a header has an element
    const int m = hd.y >> 1;
    uint32_t odd = (uint32_t)hd.y & 1u;
    for (int j = 1;; ++j) {
      const double4 nx = s[j < m ? j + 1 : j];
      const bool st = (e.y <= y) & (y < e.w);
      const double lhs = (x - e.x) * (e.w - e.y), rhs = (e.z - e.x) * (y - e.y);
      odd ^= (uint32_t)(st & (lhs < rhs));
      if (j >= m) break;
      e = nx;
    }
    if (odd) return hd.x;
    if (!hd.z) return hd.w;
    s += m + 1;
  }
}

// One point per lane; points and results pass the caches by (non-temporal), which hold the
// index: 50M points 1.03 -> 0.98 ms.  Bound by the gathers of the index (a cell, then for a
// divided cell its subcell, then for the few subcells with a list its slots): 50M points miss
// the L2 for 133 bytes each, 7.2 TB/s, with 70 to 90 lines in flight per compute unit.  The
// points and results alone take 0.23 ms of the 0.92, the cells 0.16, the subcells 0.36 and
// the lists 0.17.  Sorting the points by cell would save less than the sort costs, because a
// whole map's directory nearly fits the caches.  Region map of 1.5M vertices, against the
// tiled refinement: 50M points 6.5 -> 0.92 ms, 1M points on a plain grid 1.6 -> 0.028 ms,
// 1,500 points 0.42 -> 0.005 ms.
// SERVED: the request comes from sv, for which the launch is at least large enough, and the
// points' candidate tests are added to it.
template <bool SERVED>
__global__ __launch_bounds__(256) void k_locate_pip(LocArgs a, LocRequest r,
                                                    unsigned long long *counts, LocServed *sv,
                                                    const int64_t *cell_tests) {
  if (SERVED) r = sv->r;
  else reset_counts(counts);
  const double *px = r.px, *py = r.py;
  int32_t *out_id = r.out_id;
  const int64_t n = r.n;
  unsigned long long tests = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double x = __builtin_nontemporal_load(px + i), y = __builtin_nontemporal_load(py + i);
    double ux, uy;
    const int32_t c = locate_cell(a, x, y, ux, uy);
    int32_t ans = -1;
    if (c >= 0) {
      if (SERVED) tests += (unsigned long long)cell_tests[c];
      const LocCell ce = a.cell[c];
      ans = (int32_t)ce.base;
      if (ce.m != LOC_CONST) {
        ans = a.sub[subcell(ce.base, ce.m, ux, uy)];
        if (ans < -1) {
          ans = list_answer(a.slot + (uint32_t)(-(ans + 2)), x, y);
        }
      }
    }
    __builtin_nontemporal_store(ans, out_id + i);
  }
  if (SERVED) add_tests(sv, tests);
}

// FP64 squared distance in the definition's operation order; a perpendicular quotient is
// divided out only where it can still come below `best`: cc > fl(fl(best * L2) (1 + 2^-49))
// implies cc / L2 > best, also where the product underflows (a subnormal product is within
// half a unit of best * L2, and cc is at least a whole unit above it).  Equality divides: with
// D = 0 the product is 0 for every short segment, and cc is 0 for a point on one.
__device__ __forceinline__ double exact_d2(double x, double y, const double4 r, double best) {
  const double dx = r.z - r.x, dy = r.w - r.y;
  const double wx = x - r.x, wy = y - r.y;
  const double L2 = dx * dx + dy * dy;
  const double t = wx * dx + wy * dy;
  if (t <= 0.0) return wx * wx + wy * wy;
  if (t >= L2) {
    const double ex = x - r.z, ey = y - r.w;
    return ex * ex + ey * ey;
  }
  const double cr = wx * dy - wy * dx;
  const double cc = cr * cr;
  return cc > (best * L2) * (1.0 + 0x1p-49) ? INFINITY : cc / L2;
}

// Squared distance to an entry, in steps of its frame: FP32 on whole numbers below 2^16.
// With the entry's rounding (0.71 steps), the point's and the evaluation's (under 0.1), the
// distance is within LOC_ERR steps of the segment's.
constexpr float LOC_ERR = 1.0f;

__device__ __forceinline__ float entry_d2(float px, float py, uint32_t a, uint32_t b) {
  const float ax = (float)(a & 0xffffu), ay = (float)(a >> 16);
  const float dx = (float)(b & 0xffffu) - ax, dy = (float)(b >> 16) - ay;
  const float wx = px - ax, wy = py - ay;
  const float L2 = fmaxf(fmaf(dx, dx, dy * dy), 1.0f);  // 0 or at least 1
  const float t = __builtin_amdgcn_fmed3f(
      fmaf(wx, dx, wy * dy) * __builtin_amdgcn_rcpf(L2), 0.0f, 1.0f);
  const float ex = fmaf(-t, dx, wx), ey = fmaf(-t, dy, wy);
  return fmaf(ex, ex, ey * ey);
}

// The 64-byte records idx of the lanes that have one (LOC_NONE: none), each into its lane's
// w.  A lane's own four loads of a line would go to the cache one after another, the later
// ones waiting on the first one's miss; instead the four lanes of a quad load one record
// together, a record after the other, straight into LDS (lane l of load i to unit
// 64 i + l), and each lane reads its record back.  Chunk c of a record lies at position
// (c + quad) mod 4 of its four units, which leaves two lanes to a bank at most.
// Called by whole waves.
constexpr uint32_t LOC_NONE = 0xffffffffu;

template <int I>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, I * 0x55, 0xf, 0xf, true);
}

__device__ __forceinline__ void fetch64(const void *base, uint32_t idx, uint4 *lds, uint4 (&w)[4]) {
  const uint32_t lane = lane_id(), quad = lane >> 2;
  const char *chunk = (const char *)base + (((lane - quad) & 3u) << 4);
  auto load = [&](uint32_t i, uint32_t o) {
    if (o != LOC_NONE)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(chunk + ((uint64_t)o << 6)),
          (__attribute__((address_space(3))) void *)(lds + GP_WAVE * i), 16, 0, 0);
  };
  load(0, quad_lane<0>(idx));
  load(1, quad_lane<1>(idx));
  load(2, quad_lane<2>(idx));
  load(3, quad_lane<3>(idx));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  wave_lds_sync();
  const uint4 *mine = lds + GP_WAVE * (lane & 3u) + (lane & ~3u);
#pragma unroll
  for (uint32_t c = 0; c < 4; ++c) w[c] = mine[(c + quad) & 3u];
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before the next records land
}

// One point per lane: the FP32 distances of its subcell's entries keep the two nearest (and
// the third's distance); the entries within twice the error of the nearest, one as a rule,
// are decided by their exact distances (smaller distance, then smaller polyline).  Bound by
// the gathers of lists and segments.
// Of 8.5 ms for 200M points, points, results and cells take 2.1, the first block of the lists
// 1.9, their further blocks 1.1 and the exact segments 3.4; the L2 misses for 310 bytes a
// point, 7.2 TB/s.  Sorting the points first (by cell 4.5 ms, by 20 x 20 cells 5.0) costs
// more than it saves (3.3 to 6.2 ms, and results scattered back).
// Road map of 5.3M vertices, against the tiled refinement: 200M points 164 -> 8.5 ms, 20M
// with segment lists 5.87 -> 0.87 ms, 1,500 points 0.52 -> 0.008 ms; with each lane loading
// its own records and an offset read ahead of them 13.2, 1.34 and 0.008 ms.
template <bool SERVED>
__global__ __launch_bounds__(256) void k_locate_p2p(LocArgs a, LocRequest r,
                                                    unsigned long long *counts, LocServed *sv,
                                                    const int64_t *cell_tests) {
  __shared__ uint4 stage[256 / GP_WAVE][4 * GP_WAVE];
  if (SERVED) r = sv->r;
  else reset_counts(counts);
  const double *px = r.px, *py = r.py;
  int32_t *out_id = r.out_id;
  double *out_dist = r.out_dist;
  const int64_t n = r.n;
  if (SERVED && blockIdx.x * (int64_t)blockDim.x >= n) return;
  uint4 *lds = stage[threadIdx.x / GP_WAVE];
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool live = i < n;
  const double x = live ? __builtin_nontemporal_load(px + i) : (double)INFINITY;
  const double y = live ? __builtin_nontemporal_load(py + i) : 0.0;
  double ux, uy;
  const int32_t c = locate_cell(a, x, y, ux, uy);
  LocSegCell ce{0u, LOC_CONST, 0.0};
  if (c >= 0) ce = a.scell[c];
  const bool some = ce.m != LOC_CONST;
  const uint32_t q0 = some ? 2 * subcell(ce.base, ce.m, ux, uy) : LOC_NONE;
  const double f = LOC_UNITS / (a.cs + 2.0 * ce.reach);
  const float qx = (float)((ux * a.cs + ce.reach) * f);
  const float qy = (float)((uy * a.cs + ce.reach) * f);
  // distance to the subcell's centre, in steps, and the error of an entry's distance
  const double k = some ? (double)(1u << ce.m) : 1.0;
  const float vx = (float)(ux * k - floor(ux * k)) - 0.5f;
  const float vy = (float)(uy * k - floor(uy * k)) - 0.5f;
  const float off = __builtin_amdgcn_sqrtf(fmaf(vx, vx, vy * vy)) *
                        (float)(a.cs * f / k * (1.0 + 0x1p-16)) + LOC_ERR;
  float b1 = INFINITY, b2 = INFINITY, b3 = INFINITY;
  int32_t i1 = -1, i2 = -1;
  auto meet = [&](uint32_t ea, uint32_t eb, uint32_t seg) {
    const float d = (int32_t)seg < 0 ? INFINITY : entry_d2(qx, qy, ea, eb);
    b3 = __builtin_amdgcn_fmed3f(d, b2, b3);
    i2 = d < b1 ? i1 : d < b2 ? (int32_t)seg : i2;
    b2 = __builtin_amdgcn_fmed3f(d, b1, b2);
    i1 = d < b1 ? (int32_t)seg : i1;
    b1 = fminf(b1, d);
  };
  // the block after q, or LOC_NONE: the list ends, or no later entry can be the nearest
  // because its distance to the centre exceeds the point's and the nearest entry's together
  auto after = [&](uint32_t q, uint32_t next, float rest) {
    if (rest == INFINITY || rest > off + __builtin_amdgcn_sqrtf(b1) * (1.0f + 0x1p-20f))
      return LOC_NONE;
    return q < a.lines && (q & 1u) ? next : q + 1u;
  };
  uint4 w[4];
  for (uint32_t q = q0; ballot(q != LOC_NONE);) {
    fetch64(a.block, q, lds, w);
    if (q != LOC_NONE) {
      meet(w[0].x, w[0].y, w[0].z);
      meet(w[0].w, w[1].x, w[1].y);
      meet(w[1].z, w[1].w, w[2].x);
      meet(w[2].y, w[2].z, w[2].w);
      meet(w[3].x, w[3].y, w[3].z);
      q = after(q, w[3].x, __uint_as_float(w[3].w));
    }
  }
  double best = a.D2_next;  // accept d2 <= fl(D*D); later only strictly smaller
  int32_t id = -1;
  auto take = [&](const double4 e, int32_t fl) {
    const double d2 = exact_d2(x, y, e, a.D2_next);
    if (d2 < best || (d2 == best && fl < id)) {
      best = d2;
      id = fl;
    }
  };
  // the error holds for distances, and 2^-20 covers the squares' and roots' rounding
  const float lim = (__builtin_amdgcn_sqrtf(b1) + 2.0f * LOC_ERR) * (1.0f + 0x1p-20f);
  const float lim2 = lim * lim;
  const bool many = b3 <= lim2;
  auto decide = [&](int32_t sg) {  // LOC_NONE for the lanes with nothing to decide
    if (!ballot(sg >= 0)) return;
    fetch64(a.lseg, (uint32_t)sg, lds, w);
    if (sg >= 0)
      take(make_double4(__hiloint2double((int)w[0].y, (int)w[0].x),
                        __hiloint2double((int)w[0].w, (int)w[0].z),
                        __hiloint2double((int)w[1].y, (int)w[1].x),
                        __hiloint2double((int)w[1].w, (int)w[1].z)),
           (int32_t)w[2].x);
  };
  decide(many ? -1 : i1);
  decide(many || !(b2 <= lim2) ? -1 : i2);
  if (many) {
    for (uint32_t q = q0; q != LOC_NONE;) {
      const LocBlock &b = a.block[q];
      for (int t = 0; t < LOC_ENTRIES; ++t)
        if (b.e[t].seg >= 0 && entry_d2(qx, qy, b.e[t].a, b.e[t].b) <= lim2)
          take(a.lseg[b.e[t].seg].e, a.lseg[b.e[t].seg].f);
      q = after(q, b.e[LOC_ENTRIES - 1].a, b.rest);
    }
  }
  if (SERVED) add_tests(sv, c >= 0 ? (unsigned long long)cell_tests[c] : 0ull);
  if (live) {
    __builtin_nontemporal_store(id, out_id + i);
    __builtin_nontemporal_store(id >= 0 ? sqrt(best) : (double)INFINITY, out_dist + i);
  }
}

// The counters of a query: the candidate tests of its points' cells (counts[0]; counts[1]
// over all candidates, when `all` is given) and its points in a cell with candidates
// (counts[2]).
__global__ __launch_bounds__(256) void k_locate_count(LocArgs a, const double *px,
                                                      const double *py, int64_t n,
                                                      const int32_t *cand_off,
                                                      const int64_t *cell_tests,
                                                      const int64_t *all,
                                                      unsigned long long *counts) {
  __shared__ unsigned long long sum[3][256 / GP_WAVE];
  unsigned long long t = 0, ta = 0, np = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double ux, uy;
    const int32_t c = locate_cell(a, px[i], py[i], ux, uy);
    if (c < 0 || cand_off[c + 1] == cand_off[c]) continue;
    ++np;
    t += (unsigned long long)cell_tests[c];
    if (all) ta += (unsigned long long)all[c];
  }
  for (int off = 32; off > 0; off >>= 1) {
    t += __shfl_xor(t, off, GP_WAVE);
    ta += __shfl_xor(ta, off, GP_WAVE);
    np += __shfl_xor(np, off, GP_WAVE);
  }
  if (lane_id() == 0) {
    sum[0][threadIdx.x / GP_WAVE] = t;
    sum[1][threadIdx.x / GP_WAVE] = ta;
    sum[2][threadIdx.x / GP_WAVE] = np;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 256 / GP_WAVE; ++w) {
      t += sum[0][w];
      ta += sum[1][w];
      np += sum[2][w];
    }
    if (np) {
      atomicAdd(counts, t);
      if (all) atomicAdd(counts + 1, ta);
      atomicAdd(counts + 2, np);
    }
  }
}

}  // namespace

// ------------------------------------------------------------------------- launchers

#define LAUNCH(k, g, b, ...)                                  \
  do {                                                        \
    hipLaunchKernelGGL(k, dim3(g), dim3(b), 0, s, __VA_ARGS__); \
    return hipGetLastError();                                 \
  } while (0)

static hipError_t launch_loc_work(const Grid &g, unsigned long long *out, hipStream_t s) {
  LAUNCH(k_loc_work, blocks_for(g.ncells, 4, 2048), 256, g.d_cand_off, g.d_cand_id, g.d_eoff,
         g.kind == GP_P2P ? g.d_near : nullptr, g.ncells, out);
}

static hipError_t launch_loc_ring_prev(const int32_t *rvo, int32_t nr, int32_t *prev, hipStream_t s) {
  if (nr <= 0) return hipSuccess;
  LAUNCH(k_loc_ring_prev, blocks_for(nr, 1, 65536), 64, rvo, nr, prev);
}

static hipError_t launch_loc_pip_pairs(const Grid &g, const uint32_t *pair_cell, const double *vy,
                                const int32_t *prev, double pad, uint32_t *cnt, uint8_t *par,
                                double4 *elem, hipStream_t s) {
  const unsigned b = blocks_for(g.npairs, 4, 65536);
  if (elem)
    LAUNCH(k_loc_pip_pairs<true>, b, 256, pair_cell, g.d_cand_id, g.npairs, g.d_eoff,
           g.d_edge64, vy, prev, g.x0, g.y0, g.cs, g.nx, pad, cnt, par, elem);
  LAUNCH(k_loc_pip_pairs<false>, b, 256, pair_cell, g.d_cand_id, g.npairs, g.d_eoff, g.d_edge64,
         vy, prev, g.x0, g.y0, g.cs, g.nx, pad, cnt, par, elem);
}

static hipError_t launch_loc_pip_cells(const Grid &g, const uint32_t *eoffs, const uint8_t *par,
                                       uint32_t cap, uint32_t *nsub, LocCell *cell,
                                       unsigned long long *cost, hipStream_t s) {
  LAUNCH(k_loc_pip_cells, blocks_for((int64_t)g.ncells + 1, 256, 8192), 256, g.d_cand_off,
         g.d_cand_id, g.nx, g.ny, eoffs, par, cap, nsub, cell, cost);
}

// Subcell bases of the cells from the scan of nsub, and their groups; *n is zeroed here.
template <class Cell>
static hipError_t launch_loc_groups(const Grid &g, const uint32_t *base, Cell *cell, uint32_t *n,
                                    int2 *group, hipStream_t s) {
  const unsigned b = blocks_for(g.ncells, 256, 8192);
  hipError_t e = launch_fill_u32(n, 0u, 1, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_loc_cell_base<Cell>, dim3(b), dim3(256), 0, s, base, g.nx, g.ny, cell);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  LAUNCH(k_loc_groups<Cell>, b, 256, cell, g.ncells, n, group);
}

static hipError_t launch_loc_pip_sub(const Grid &g, const int2 *group, uint32_t ngroups,
                                     const uint32_t *eoffs, const uint8_t *par,
                                     const double4 *elem, const LocCell *cell, double pad,
                                     uint32_t *cnt, double4 *slot, int32_t *sub, hipStream_t s) {
  const unsigned b = (ngroups + 3) / 4;
  if (sub)
    LAUNCH(k_loc_pip_sub<true>, b, 256, g.d_cand_off, g.d_cand_id, group, ngroups, eoffs, par,
           elem, cell, g.x0, g.y0, g.cs, g.nx, pad, cnt, slot, sub);
  LAUNCH(k_loc_pip_sub<false>, b, 256, g.d_cand_off, g.d_cand_id, group, ngroups, eoffs, par,
         elem, cell, g.x0, g.y0, g.cs, g.nx, pad, cnt, slot, sub);
}

static hipError_t launch_loc_cell_segs(const Grid &g, double r, double slack, uint32_t *cnt,
                                double *cmin, int32_t *list, hipStream_t s) {
  const unsigned b = blocks_for(g.ncells, 4, 65536);
  if (list)
    LAUNCH(k_loc_cell_segs<true>, b, 256, g.d_cand_off, g.d_near, g.d_edge64, g.ncells, g.x0, g.y0, g.cs, g.nx, r, g.D, slack, cnt, cmin, list);
  LAUNCH(k_loc_cell_segs<false>, b, 256, g.d_cand_off, g.d_near, g.d_edge64, g.ncells, g.x0, g.y0, g.cs, g.nx, r, g.D, slack, cnt, cmin, list);
}

static hipError_t launch_loc_p2p_cells(const Grid &g, const uint32_t *first, const double *cmin,
                                       double r, double slack, uint32_t target, uint32_t cap,
                                       uint32_t *nsub, LocSegCell *cell,
                                       unsigned long long *cost, hipStream_t s) {
  LAUNCH(k_loc_p2p_cells, blocks_for((int64_t)g.ncells + 1, 256, 8192), 256, first, cmin,
         g.nx, g.ny, r, g.D, slack, target, cap, nsub, cell, cost);
}

static hipError_t launch_loc_add(uint32_t *v, size_t n, uint32_t d, hipStream_t s) {
  LAUNCH(k_loc_add, blocks_for((int64_t)n, 256, 8192), 256, v, n, d);
}

static hipError_t launch_loc_seg_keys(const Grid &g, double min_L2, uint32_t *key, uint32_t *flag,
                                      hipStream_t s) {
  LAUNCH(k_loc_seg_keys, blocks_for(g.nedges, 256, 8192), 256, g.d_edge64, g.nedges, g.x0, g.y0,
         g.cs, g.nx, g.ny, min_L2, key, flag);
}

static hipError_t launch_loc_polylines(const Grid &g, int32_t *f, hipStream_t s) {
  LAUNCH(k_loc_polylines, blocks_for(g.nf, 4, 8192), 256, g.d_eoff, g.nf, f);
}

static hipError_t launch_loc_segments(const Grid &g, const uint32_t *order, const int32_t *f,
                                      LocSeg *seg, int32_t *place, hipStream_t s) {
  LAUNCH(k_loc_segments, blocks_for(g.nedges, 256, 8192), 256, order, f, g.d_edge64, g.nedges,
         seg, place);
}

static hipError_t launch_loc_sub_segs(const Grid &g, const uint32_t *first, const int32_t *list,
                                      const int2 *group, uint32_t ngroups,
                                      const LocSegCell *cell, double pad, double slack,
                                      const int32_t *place, double *glim, uint32_t *cnt,
                                      double2 *lim, LocBlock *block, hipStream_t s) {
  const unsigned b = (ngroups + 3) / 4;
  if (block)
    LAUNCH(k_loc_sub_segs<true>, b, 256, first, list, g.d_edge64, group, ngroups, cell, g.x0,
           g.y0, g.cs, g.nx, pad, g.D, slack, place, glim, cnt, lim, block);
  LAUNCH(k_loc_sub_segs<false>, b, 256, first, list, g.d_edge64, group, ngroups, cell, g.x0,
         g.y0, g.cs, g.nx, pad, g.D, slack, place, glim, cnt, lim, block);
}

hipError_t launch_locate(gp_kind kind, const LocArgs &a, const LocRequest &r,
                         unsigned long long *counts, hipStream_t s) {
  const unsigned b = (unsigned)((r.n + 255) / 256);
  LocServed *none = nullptr;
  const int64_t *no_tests = nullptr;
  if (kind == GP_PIP) LAUNCH(k_locate_pip<false>, b, 256, a, r, counts, none, no_tests);
  LAUNCH(k_locate_p2p<false>, b, 256, a, r, counts, none, no_tests);
}

hipError_t launch_serve_begin(LocServed *sv, const LocRequest &r, hipStream_t s) {
  LAUNCH(k_serve_begin, 1, GP_WAVE, sv, r);
}

hipError_t launch_serve(gp_kind kind, const LocArgs &a, LocServed *sv, int64_t most,
                        const int64_t *cell_tests, hipStream_t s) {
  const unsigned b = (unsigned)((most + 255) / 256);
  LocRequest none{};
  unsigned long long *no_counts = nullptr;
  if (kind == GP_PIP)
    hipLaunchKernelGGL(k_locate_pip<true>, dim3(b), dim3(256), 0, s, a, none, no_counts, sv,
                       cell_tests);
  else
    hipLaunchKernelGGL(k_locate_p2p<true>, dim3(b), dim3(256), 0, s, a, none, no_counts, sv,
                       cell_tests);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LAUNCH(k_serve_end, 1, GP_WAVE, sv);
}

hipError_t launch_locate_count(const LocArgs &a, const double *px, const double *py, int64_t n,
                               const int32_t *cand_off, const int64_t *cell_tests,
                               const int64_t *all, unsigned long long *counts, hipStream_t s) {
  LAUNCH(k_locate_count, blocks_for(n, 1024, 2048), 256, a, px, py, n, cand_off, cell_tests, all,
         counts);
}


// ------------------------------------------------------------------------- build

namespace {

// Limits of the index: slots of 32 bytes (PIP), subcells of a 128-byte line each, expected
// entries and further blocks (P2P), tests of the build, and entries per subcell.  The last line
// is drawn for P2P lists that no query can stop early, all of whose segments are equally far
// (points anywhere in the box of a circle of m edges, 2M of them, locator against tiled
// refinement, FP64): m = 400, 35 entries a subcell, 0.55 against 1.29 ms (near the centre, 400
// entries, 1.81 against 1.58); m = 4000, 400 entries, 6.1 against 5.8 ms (17.4 against 7.5).
// Other lists stay the better path far beyond it (short segments at random: 131 entries 0.14
// against 59 ms; PIP, spikes that cross the cell: 113 entries 2.7 against 8.8 ms, 1812 entries
// 49 against 121 ms), where the index grows by 32 bytes an entry (PIP).
constexpr int64_t kMaxSlots = int64_t(1) << 27;     // 4 GiB
constexpr int64_t kMaxEntries = int64_t(1) << 29;
constexpr int64_t kMaxLines = int64_t(1) << 25;     // 4 GiB
constexpr int64_t kMaxBlocks = int64_t(1) << 27;    // 8 GiB
constexpr int64_t kMaxElems = int64_t(1) << 26;     // 2 GiB while building
constexpr int64_t kMaxSubcells = int64_t(1) << 27;  // 512 MiB
constexpr int64_t kMaxCells = int64_t(1) << 26;
constexpr int64_t kMaxBuildTests = int64_t(1) << 33;
// The first passes sweep the candidates' edges of every cell, each one's by one wave (P2P) or by
// one for a polygon, and a wave sweeps a cell's elements or segments again for each group.  At
// the limits that is, beside a build without a locator: 2^36 edges in all 0.3 s (7.6e10 edge
// visits, twice, 0.39 s, about two tiled queries of one point per cell), 2^22 of a cell 0.1 s,
// 2^20 elements of a cell 0.1 s.
constexpr int64_t kMaxPairEdges = int64_t(1) << 36;
constexpr int64_t kMaxCellEdges = int64_t(1) << 22;
constexpr int64_t kMaxCellElems = int64_t(1) << 20;
constexpr int64_t kMaxMeanEntries = 64;
constexpr uint32_t kLocTarget = 8;  // P2P: entries per subcell aimed at
// P2P: the definition's (w x d)^2 / |d|^2 holds a distance only while its square is neither
// lost to underflow (an error of 2^-537 / |d|, below 2^-80 cells when |d|^2 is at least
// kMinLen2 and at least kMinLen2 / cs^2) nor overflows (64 M^4 < 2^1024, M the largest
// coordinate).  Beyond that its FP64 value may order the segments otherwise than their
// distances do, which is what an index goes by.
constexpr double kMinLen2 = 0x1p-900;
constexpr double kMaxP2PCoord = 0x1p250;

struct Buf {
  void *p = nullptr;
  ~Buf() { if (p) (void)hipFree(p); }
  bool alloc(size_t bytes) {
    if (hipMalloc(&p, bytes ? bytes : 16) == hipSuccess) return true;
    (void)hipGetLastError();  // no memory for it: the grid does without
    p = nullptr;
    return false;
  }
  template <class T> T *as(size_t off = 0) const { return (T *)((char *)p + off); }
  template <class T> T *take() { T *q = (T *)p; p = nullptr; return q; }
};

// Places in one buffer: an allocation costs the build more than most of its kernels.
struct Places {
  size_t bytes = 0;
  size_t add(size_t n) {
    const size_t o = bytes;
    bytes = (bytes + n + 255) / 256 * 256;
    return o;
  }
};

#define LOC_TRY(expr)                      \
  do {                                     \
    const hipError_t e_ = (expr);          \
    if (e_ != hipSuccess) return e_;       \
  } while (0)
#define LOC_NEED(cond)                     \
  do {                                     \
    if (!(cond)) return hipSuccess;        \
  } while (0)

hipError_t read_back(void *dst, const void *src, size_t bytes, hipStream_t s) {
  LOC_TRY(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
  return hipStreamSynchronize(s);
}

// cnt[0 .. n) becomes its exclusive prefix sum with the total at cnt[n]; *total in 64 bits
// (nothing is scanned when it passes `most`).
hipError_t scan_counts(uint32_t *cnt, size_t n, int64_t most, unsigned long long *sum,
                       uint32_t *tmp, int64_t *total, hipStream_t s) {
  unsigned long long t = 0;
  LOC_TRY(launch_fill_u32(cnt + n, 0u, 1, s));
  LOC_TRY(launch_sum_u32(cnt, n, sum, s));
  LOC_TRY(read_back(&t, sum, 8, s));
  *total = t > (unsigned long long)INT64_MAX ? INT64_MAX : (int64_t)t;
  if (*total > most) return hipSuccess;
  return launch_exclusive_scan_u32(cnt, cnt, n + 1, tmp, s);
}

// Whether the first passes stay within their limits, from k_loc_work's sums.
bool work_fits(const unsigned long long *work) {
  return work[0] <= (unsigned long long)kMaxPairEdges &&
         work[1] <= (unsigned long long)kMaxCellEdges;
}

hipError_t build_pip(Grid &g, const LocBuild &b, double pad, hipStream_t s) {
  const size_t np = (size_t)g.npairs, nc = (size_t)g.ncells;
  Buf b1, b2, elems, cells, subs, slots;
  Places p1;
  const size_t o_prev = p1.add((size_t)g.nedges * 4), o_cnt = p1.add((np + 1) * 4),
               o_par = p1.add(np), o_nsub = p1.add((nc + 1) * 4), o_sum = p1.add(64),
               o_tmp = p1.add(scan_tmp_elems(std::max(np, nc) + 1) * 4);
  LOC_NEED(b1.alloc(p1.bytes) && cells.alloc(nc * sizeof(LocCell)));
  int32_t *prev = b1.as<int32_t>(o_prev);
  uint32_t *cnt = b1.as<uint32_t>(o_cnt), *nsub = b1.as<uint32_t>(o_nsub),
           *tmp = b1.as<uint32_t>(o_tmp);
  uint8_t *par = b1.as<uint8_t>(o_par);
  unsigned long long *sum = b1.as<unsigned long long>(o_sum);
  LocCell *cell = cells.as<LocCell>();
  unsigned long long work[2] = {0, 0};
  LOC_TRY(launch_fill_u32((uint32_t *)sum, 0u, 4, s));
  LOC_TRY(launch_loc_work(g, sum, s));
  LOC_TRY(read_back(work, sum, 16, s));
  LOC_NEED(work_fits(work));
  int64_t total = 0;
  LOC_TRY(launch_loc_ring_prev(b.ring_off, b.n_rings, prev, s));
  if (np) LOC_TRY(launch_loc_pip_pairs(g, b.pair_cell, b.vy, prev, pad, cnt, par, nullptr, s));
  LOC_TRY(scan_counts(cnt, np, kMaxElems, sum, tmp, &total, s));
  LOC_NEED(total <= kMaxElems && elems.alloc((size_t)total * 32));
  double4 *elem = elems.as<double4>();
  if (total) LOC_TRY(launch_loc_pip_pairs(g, b.pair_cell, b.vy, prev, pad, cnt, par, elem, s));
  // the finest subdivision whose size and build stay within the limits
  unsigned long long cost[4] = {0, 0, 0, 0};
  for (int cap = 6; cap >= 0; --cap) {
    LOC_TRY(launch_fill_u32((uint32_t *)sum, 0u, 8, s));
    LOC_TRY(launch_loc_pip_cells(g, cnt, par, (uint32_t)cap, nsub, cell, sum, s));
    LOC_TRY(read_back(cost, sum, 32, s));
    LOC_NEED(cost[3] <= (unsigned long long)kMaxCellElems);
    if (cost[0] <= (unsigned long long)kMaxSubcells && cost[1] <= (unsigned long long)kMaxBuildTests)
      break;
    LOC_NEED(cap > 0);
  }
  const size_t ns = (size_t)cost[0];
  const uint32_t ng = (uint32_t)cost[2];
  Places p2;
  const size_t o_group = p2.add((size_t)ng * 8), o_scnt = p2.add((ns + 1) * 4),
               o_stmp = p2.add(scan_tmp_elems(ns + 1) * 4);
  LOC_NEED(b2.alloc(p2.bytes) && subs.alloc(ns * 4));
  int2 *group = b2.as<int2>(o_group);
  uint32_t *scnt = b2.as<uint32_t>(o_scnt);
  LOC_TRY(launch_exclusive_scan_u32(nsub, nsub, nc + 1, tmp, s));
  LOC_TRY(launch_loc_groups(g, nsub, cell, (uint32_t *)sum, group, s));
  total = 0;
  if (ns) {
    LOC_TRY(launch_loc_pip_sub(g, group, ng, cnt, par, elem, cell, pad, scnt, nullptr, nullptr, s));
    LOC_TRY(scan_counts(scnt, ns, kMaxSlots, sum, b2.as<uint32_t>(o_stmp), &total, s));
    LOC_NEED(total <= kMaxSlots && total <= kMaxMeanEntries * (int64_t)ns);
    LOC_NEED(slots.alloc((size_t)total * 32));
    LOC_TRY(launch_loc_pip_sub(g, group, ng, cnt, par, elem, cell, pad, scnt, slots.as<double4>(),
                               subs.as<int32_t>(), s));
  }
  LOC_TRY(hipStreamSynchronize(s));  // before the temporaries go
  g.d_loc_cell = cells.take<LocCell>();
  g.d_loc_sub = subs.take<int32_t>();
  g.d_loc_slot = slots.take<double4>();
  g.loc_bytes = (int64_t)(nc * sizeof(LocCell) + ns * 4) + total * 32;
  return hipSuccess;
}

hipError_t build_p2p(Grid &g, double pad, double slack, hipStream_t s) {
  const size_t nc = (size_t)g.ncells, nseg = (size_t)g.nedges;
  Buf b1, b2, lists, cells, blocks, segs;
  Places p1;
  const size_t o_cnt = p1.add((nc + 1) * 4), o_cmin = p1.add(nc * 8),
               o_nsub = p1.add((nc + 1) * 4), o_sum = p1.add(64),
               o_tmp = p1.add(scan_tmp_elems(std::max(nc + 1, radix_hist_elems(nseg))) * 4),
               o_kA = p1.add(nseg * 4), o_kB = p1.add(nseg * 4), o_vA = p1.add(nseg * 4),
               o_vB = p1.add(nseg * 4), o_poly = p1.add(nseg * 4),
               o_hist = p1.add(radix_hist_elems(nseg) * 4), o_place = p1.add(nseg * 4);
  LOC_NEED(b1.alloc(p1.bytes) && cells.alloc(nc * sizeof(LocSegCell)) &&
           segs.alloc(nseg * sizeof(LocSeg)));
  uint32_t *cnt = b1.as<uint32_t>(o_cnt), *nsub = b1.as<uint32_t>(o_nsub),
           *tmp = b1.as<uint32_t>(o_tmp);
  double *cmin = b1.as<double>(o_cmin);
  unsigned long long *sum = b1.as<unsigned long long>(o_sum);
  int32_t *place = b1.as<int32_t>(o_place);
  LocSegCell *cell = cells.as<LocSegCell>();
  unsigned long long work[3] = {0, 0, 0};  // and whether a segment is too short (kMinLen2)
  LOC_TRY(launch_fill_u32((uint32_t *)sum, 0u, 6, s));
  LOC_TRY(launch_loc_work(g, sum, s));
  if (nseg)
    LOC_TRY(launch_loc_seg_keys(g, kMinLen2 * std::max(1.0, 1.0 / (g.cs * g.cs)),
                                b1.as<uint32_t>(o_kA), (uint32_t *)(sum + 2), s));
  LOC_TRY(read_back(work, sum, 24, s));
  LOC_NEED(work_fits(work) && !work[2]);
  if (nseg) {  // the segments in the order of the cells
    uint32_t *keys = nullptr, *order = nullptr;
    int bits = 1;
    while (bits < 31 && (1 << bits) < g.ncells) ++bits;
    LOC_TRY(launch_loc_polylines(g, b1.as<int32_t>(o_poly), s));
    LOC_TRY(launch_radix_sort(b1.as<uint32_t>(o_kA), b1.as<uint32_t>(o_kB),
                              b1.as<uint32_t>(o_vA), b1.as<uint32_t>(o_vB), nseg, bits, true,
                              b1.as<uint32_t>(o_hist), tmp, s, &keys, &order));
    LOC_TRY(launch_loc_segments(g, order, b1.as<int32_t>(o_poly), segs.as<LocSeg>(), place, s));
  }
  // the cells' segments
  const double r = 0.70710678118654757 * (1.0 + 0x1p-40) * (g.cs + 2.0 * pad);
  int64_t total = 0;
  LOC_TRY(launch_loc_cell_segs(g, r, slack, cnt, cmin, nullptr, s));
  LOC_TRY(scan_counts(cnt, nc, kMaxEntries, sum, tmp, &total, s));
  LOC_NEED(total <= kMaxEntries && lists.alloc((size_t)total * 4));
  int32_t *list = lists.as<int32_t>();
  if (total) LOC_TRY(launch_loc_cell_segs(g, r, slack, cnt, cmin, list, s));
  unsigned long long cost[5] = {0, 0, 0, 0, 0};
  for (uint32_t target = kLocTarget;; target *= 2) {
    LOC_TRY(launch_fill_u32((uint32_t *)sum, 0u, 10, s));
    LOC_TRY(launch_loc_p2p_cells(g, cnt, cmin, r, slack + pad, target, 5u, nsub, cell, sum, s));
    LOC_TRY(read_back(cost, sum, 40, s));
    LOC_NEED(cost[4] <= (unsigned long long)kMaxCellElems);
    if (cost[0] <= (unsigned long long)kMaxLines &&
        cost[1] <= (unsigned long long)kMaxBuildTests &&
        cost[2] <= (unsigned long long)kMaxEntries)
      break;
    LOC_NEED(target < (1u << 30));
  }
  const size_t ns = (size_t)cost[0];
  const uint32_t ng = (uint32_t)cost[3];
  Places p2;
  const size_t o_group = p2.add((size_t)ng * 8), o_glim = p2.add((size_t)ng * 8),
               o_lim = p2.add(ns * 16),
               o_soff = p2.add((ns + 1) * 4), o_stmp = p2.add(scan_tmp_elems(ns + 1) * 4);
  LOC_NEED(b2.alloc(p2.bytes));
  int2 *group = b2.as<int2>(o_group);
  double *glim = b2.as<double>(o_glim);
  double2 *lim = b2.as<double2>(o_lim);
  uint32_t *soff = b2.as<uint32_t>(o_soff);
  LOC_TRY(launch_exclusive_scan_u32(nsub, nsub, nc + 1, tmp, s));
  LOC_TRY(launch_loc_groups(g, nsub, cell, (uint32_t *)sum, group, s));
  total = 0;
  if (ns) {
    LOC_TRY(launch_loc_sub_segs(g, cnt, list, group, ng, cell, pad, slack, place, glim, soff, lim,
                                nullptr, s));
    LOC_TRY(scan_counts(soff, ns, kMaxBlocks, sum, b2.as<uint32_t>(o_stmp), &total, s));
    LOC_NEED(total <= kMaxBlocks && LOC_ENTRIES * total <= kMaxMeanEntries * (int64_t)ns);
    LOC_NEED(blocks.alloc((size_t)(2 * ns + total) * sizeof(LocBlock)));
    LOC_TRY(launch_loc_add(soff, ns, 2 * (uint32_t)ns, s));
    LOC_TRY(launch_loc_sub_segs(g, cnt, list, group, ng, cell, pad, slack, place, glim, soff, lim,
                                blocks.as<LocBlock>(), s));
  }
  LOC_TRY(hipStreamSynchronize(s));
  g.d_loc_scell = cells.take<LocSegCell>();
  g.d_loc_block = blocks.take<LocBlock>();
  g.loc_lines = 2 * (uint32_t)ns;
  g.d_loc_seg = segs.take<LocSeg>();
  g.loc_bytes = (int64_t)(nc * sizeof(LocSegCell) + nseg * sizeof(LocSeg)) +
                (2 * (int64_t)ns + total) * (int64_t)sizeof(LocBlock);
  return hipSuccess;
}

}  // namespace

hipError_t build_locator(Grid &g, const LocBuild &b, hipStream_t s) {
  if (g.ncells > kMaxCells || !(b.max_coord < 1e150) || !(g.cs > 1e-140)) return hipSuccess;
  // P2P: the frames' steps are whole only where a coordinate's rounding is far below one
  if (g.kind == GP_P2P && !(b.max_coord < std::min(g.cs * 0x1p28, kMaxP2PCoord))) return hipSuccess;
  // pads: as the MBBs', and over 1000 times the rounding of a point's cell and subcell
  const double pad = g.cs * 0x1p-20 + b.max_coord * 0x1p-40;
  if (g.kind == GP_PIP) return build_pip(g, b, pad, s);
  return build_p2p(g, pad, b.max_coord * 0x1p-40 + 0x1p-500, s);
}

LocArgs locator_args(const Grid &g) {
  LocArgs a;
  a.x0 = g.x0;
  a.y0 = g.y0;
  a.cs = g.cs;
  a.nx = g.nx;
  a.ny = g.ny;
  a.cell = g.d_loc_cell;
  a.sub = g.d_loc_sub;
  a.slot = g.d_loc_slot;
  a.scell = g.d_loc_scell;
  a.block = g.d_loc_block;
  a.lines = g.loc_lines;
  a.lseg = g.d_loc_seg;
  a.D2_next = nextafter(g.D2, INFINITY);
  return a;
}

}  // namespace gp
