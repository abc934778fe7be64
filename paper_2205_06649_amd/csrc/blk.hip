// Sweeps over several levels per launch (FP64 state): the step kernels'
// arithmetic, cell by cell and bit for bit, on blocks of a box that keep
// their levels on chip.
//
// A block is a run of whole 256-cell tiles of one box.  One workgroup takes
// it through several levels in one launch: the current level (state,
// perturbation, or lambda^{n+1}) sits in an LDS frame over the block's rows,
// one column wider on either side and one row above and below, which carries
// the frozen ring of the level (zeros for the perturbation and the adjoint)
// or, for a box spanning the circle, copies of the box's own cells across the
// seam or the pole.  The level before it (the leapfrog base, lambda^{n+2})
// sits in a second frame where two fit (TWO, at most three passes): a cell's
// new value replaces its base there, and the frames change roles at the one
// barrier of a level.  Larger blocks hold it in registers, one value per thread
// and pass, and swap the two after each level, between two barriers.  A block
// that is a whole box runs all its levels in one launch.
// A box too large for one frame, or worth spreading over idle compute units,
// is cut into blocks that compute, besides their own cells, e rows above and
// below them at the level e levels before the launch's last one, so that no
// block waits for another: neighbours compute those cells too, from the same
// inputs by the same expressions.
//
// Cells map to threads in box order, 64 consecutive cells (an aligned chunk
// of a tile) to a wave, so that a tile's share of J is the sum the step
// kernel takes: a shuffle tree per chunk, then the chunks in order, level by
// level.
//
// What bounds it: the step kernels launch once per level and move 72 B
// (forward) and 111 B (adjoint) per cell and level; here a level is written
// once (forward) or read once (adjoint), plus the launch's two levels in and
// out.  Small blocks are bound by their passes' instructions and latencies (an
// adjoint pass of 64 cells is about 200 vector instructions, 75 of them FP64;
// of the adjoint's 190 us on 64 boxes of 40 x 72 cells, 50 are the launches'
// starts, 38 waiting for the state's loads), large ones by memory.  Step
// kernels -> one frame -> two, per evaluation: 8 boxes of 18 x 36 cells, 13
// levels 113 -> 57 -> 52 us; 64 boxes of 40 x 72, 34 levels 518 -> 283 -> 273
// us; 1024 boxes of 72 x 136, 34 levels, one frame 16.6 -> 8.0 ms (forward 4.9
// -> 2.4 ms, 3.3 TB/s of its 7.9 GB; adjoint 11.7 -> 5.6 ms).  In a small
// block an adjoint level takes about 6800 clocks on its compute unit, 2500 to
// 3400 of them until the state, target and observation bin are there: 31 KB
// from beyond the L2, a unit's own rate, and no latency to hide: all loads of a
// launch's start issued before the first is used, a pass's or a whole level's
// loads issued ahead, the state in a third frame (12 of 15 loads fewer), 10 %
// fewer instructions by scalar bases gained nothing or lost.  512 threads of
// twice the passes, with registers to spare, were 25 % slower than 1024, which
// leave 128 registers: hence the values pinned to their pass below.
#include <algorithm>
#include <array>
#include <map>
#include <type_traits>
#include <vector>

#include "kernels.h"
#include "launch.h"
#include "stencil.h"

namespace dd4dvar {

using namespace stencil;

namespace {
constexpr int kRowTab = 8;                 // doubles per row of the row table
constexpr int kBorderMax = 1024;           // border items of a block
constexpr int border_items(int threads) { return (kBorderMax + threads - 1) / threads; }

// cells of the block [out0, out1) grown by e rows within the box
struct Range {
  int lo, hi;
};
__device__ __forceinline__ Range grown(const BlkWork& w, int e, int nx, int ncell) {
  return {max(0, w.out0 - e * nx), min(ncell, w.out1 + e * nx)};
}

// Observation entries of the calling lane's cell at one level, one wave per
// 64-cell chunk of a tile (bin: the tile's entry of Dom::obs_bin; bin and
// chunk uniform over the wave).  z is the state (or, dz true, the perturbation, whose
// misfit is itself); adds nothing where the lane's cell is not observed.
// Forcing q r into f, the terms of J into jloc, field by field.  By masks and
// not through LDS as in the step kernels: a wave takes its chunks by itself, with
// no barrier per tile.
__device__ __forceinline__ void obs_terms(const Dom<double>& D, int bin, int chunk, const V3<double>& z,
                                          bool dz, double* f, double& jloc) {
  const ObsTile& o = D.obs_tile[__builtin_amdgcn_readfirstlane(bin)];
  const uint64_t m[3] = {o.mask[chunk][0], o.mask[chunk][1], o.mask[chunk][2]};   // scalar registers
  const int lane = int(threadIdx.x & 63);
  int k = o.base[chunk];
#pragma unroll
  for (int i = 0; i < 3; ++i)               // entries of the lanes below
    k = __builtin_amdgcn_mbcnt_hi(uint32_t(m[i] >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m[i]), k));
  const double zz[3] = {z.h, z.u, z.v};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (!(m[i] >> lane & 1)) continue;
    const double qo = D.obs_q[k];
    const double rr = dz ? zz[i] : zz[i] - D.obs_val[k];
    f[i] = qo * rr;
    if (!dz) jloc += 0.5 * qo * rr * rr;
    ++k;
  }
}

// a block's frame: rows rb - 1 .. re + 1 of the box, columns -1 .. nx
struct Frame {
  int rb, re, fw;
  __device__ __forceinline__ int pos(int r, int c) const { return ((r - rb + 1) * fw + c + 1) * 3; }
  __device__ __forceinline__ int size() const { return (re - rb + 3) * fw * 3; }
  __device__ __forceinline__ int rows() const { return re - rb + 1; }
};

// the state of level n of a box (every level is stored: level n at slot n)
__device__ __forceinline__ double* state(const Dom<double>& D, const SubDev& S, int n) {
  return D.traj + S.zoff + int64_t(n) * 3 * S.ncell;
}
__device__ __forceinline__ V3<double> get(const double* f, int p) { return {f[p], f[p + 1], f[p + 2]}; }
__device__ __forceinline__ void put(double* f, int p, const V3<double>& v) {
  f[p] = v.h;
  f[p + 1] = v.u;
  f[p + 2] = v.v;
}

// a cell's value into the frame; in a box spanning the circle also into the
// frame positions that wrap onto it (across a pole with u, v times sg)
__device__ __forceinline__ void put_cell(double* f, const Frame& F, const SubDev& S, int half, int r,
                                         int c, const V3<double>& v, double sg) {
  put(f, F.pos(r, c), v);
  if (S.span) {
    if (c == 0) put(f, F.pos(r, S.nx), v);
    if (c == S.nx - 1) put(f, F.pos(r, -1), v);
    const int cc = c >= half ? c - half : c + half;
    const V3<double> w = {v.h, sg * v.u, sg * v.v};
    if (r == 0 && S.pole_s) put(f, F.pos(-1, cc), w);
    if (r == S.ny - 1 && S.pole_n) put(f, F.pos(S.ny, cc), w);
  }
}

// rows of the frame: forward table {a1, a2, a3, cf, ct, cN, cS}, adjoint
// table {a1, a2, a3n, a3s, cf, ct, c} (a3 of the rows whose increments read
// the row from the north and the south; a row at the box's edge takes its
// own, where the reader's adjoint is zero or lies across a pole)
template <int NT, bool ADJ>
__device__ __forceinline__ void fill_rows(double* tab, const Dom<double>& D, const SubDev& S,
                                          const Frame& F) {
  for (int i = threadIdx.x; i < F.rows(); i += NT) {
    const int r = F.rb + i, j = S.row0 + r;
    const RowCoef<double> rc = D.rows[j];
    double* q = tab + kRowTab * i;
    q[0] = rc.a1;
    q[1] = rc.a2;
    if (ADJ) {
      q[2] = D.rows[r + 1 < S.ny ? j + 1 : j].a3;
      q[3] = D.rows[r > 0 ? j - 1 : j].a3;
      q[4] = rc.cf;
      q[5] = rc.ct;
      q[6] = rc.c;
    } else {
      q[2] = rc.a3;
      q[3] = D.cosx[j + 2];
      q[4] = rc.cf;
      q[5] = rc.ct;
      q[6] = D.cosx[j];
    }
  }
}

// border items of a block: the west and the east column of its rows, then
// the rows beyond the box's own first and last (positions that wrap inside
// the box are not items)
struct Border {
  int cols, south, north;                  // items of each kind; cols per side
  __device__ __forceinline__ Border(const SubDev& S, const Frame& F)
      : cols(S.span ? 0 : F.rows()),
        south(F.rb == 0 && !S.pole_s ? S.nx : 0),
        north(F.re == S.ny - 1 && !S.pole_n ? S.nx : 0) {}
  __device__ __forceinline__ int count() const { return 2 * cols + south + north; }
  // first item of each kind
  __device__ __forceinline__ int east0() const { return cols; }
  __device__ __forceinline__ int south0() const { return 2 * cols; }
  __device__ __forceinline__ int north0() const { return 2 * cols + south; }
  // frame position and ring index of item i < count()
  __device__ __forceinline__ void item(int i, const SubDev& S, const Frame& F, int* pos, int* k) const {
    if (i < 2 * cols) {
      const bool east = i >= cols;
      const int r = F.rb + (east ? i - cols : i);
      *pos = F.pos(r, east ? S.nx : -1);
      *k = 2 * S.nx + (east ? S.ny : 0) + r;
    } else if (i < north0()) {
      *pos = F.pos(-1, i - south0());
      *k = i - south0();
    } else {
      *pos = F.pos(S.ny, i - north0());
      *k = S.nx + i - north0();
    }
  }
};

// A thread's cell in one word: frame row (11 bits), column (11), coverage (8).
__device__ __forceinline__ int cell_word(int row, int c, int cover) { return row << 19 | c << 8 | cover; }
__device__ __forceinline__ int cell_row(int w) { return w >> 19; }
__device__ __forceinline__ int cell_col(int w) { return (w >> 8) & 0x7ff; }
__device__ __forceinline__ int cell_cover(int w) { return w & 0xff; }

// keeps what is computed from v inside the pass (left alone, the compiler
// computes every pass's addresses ahead of the level loop and spills them)
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The stored state of level n at a cell and its neighbours, from the box's
// level Z (uniform) by 32-bit offsets.  A neighbour on the frozen ring reads
// the cell itself here (any address in the box) and takes its ring value from
// the staged items in `fix`, once the loads are back.
template <bool SPAN>
struct State5 {
  V3<double> C, E, W, N, S;
  double sn, ss;
  bool ringE, ringW, ringN, ringS;
  static __device__ __forceinline__ V3<double> at(const double* Z, int64_t plane, uint32_t off) {
    const char* z = reinterpret_cast<const char*>(Z);
    const int64_t f = plane * int64_t(sizeof(double));
    return {*reinterpret_cast<const double*>(z + off), *reinterpret_cast<const double*>(z + f + off),
            *reinterpret_cast<const double*>(z + 2 * f + off)};
  }
  __device__ __forceinline__ void load(const double* Z, int64_t plane, const SubDev& B, int half,
                                       int m, int r, int c) {
    const bool e_in = c + 1 < B.nx, w_in = c > 0, n_in = r + 1 < B.ny, s_in = r > 0;
    int de = e_in ? 1 : 0, dw = w_in ? -1 : 0, dn = n_in ? B.nx : 0, ds = s_in ? -B.nx : 0;
    ringE = !e_in;
    ringW = !w_in;
    ringN = !n_in;
    ringS = !s_in;
    sn = ss = 1.0;
    if (SPAN && B.span) {                    // uniform
      const int across = c + half >= B.nx ? half - B.nx : half;
      de = e_in ? 1 : 1 - B.nx;
      dw = w_in ? -1 : B.nx - 1;
      ringE = ringW = false;
      if (B.pole_n) {
        dn = n_in ? B.nx : across;
        sn = n_in ? 1.0 : -1.0;
        ringN = false;
      }
      if (B.pole_s) {
        ds = s_in ? -B.nx : across;
        ss = s_in ? 1.0 : -1.0;
        ringS = false;
      }
    }
    C = at(Z, plane, uint32_t(m) * 8u);
    E = at(Z, plane, uint32_t(m + de) * 8u);
    W = at(Z, plane, uint32_t(m + dw) * 8u);
    N = at(Z, plane, uint32_t(m + dn) * 8u);
    S = at(Z, plane, uint32_t(m + ds) * 8u);
  }
  // ring: the staged items of the level; row: the cell's row in the frame.
  // At most one of the east and west neighbours is on the ring (a box has two
  // columns at least), so one read without a branch serves both; the rows
  // above and below the box concern few waves.
  __device__ __forceinline__ void fix(const double* ring, const Border& b, int row, int c) {
    if (b.cols > 0) {                        // uniform
      const V3<double> r = get(ring, 3 * (ringE ? b.cols + row : row));
      E = {ringE ? r.h : E.h, ringE ? r.u : E.u, ringE ? r.v : E.v};
      W = {ringW ? r.h : W.h, ringW ? r.u : W.u, ringW ? r.v : W.v};
    }
    if (__any(ringN)) {
      if (ringN) N = get(ring, 3 * (b.north0() + c));
    }
    if (__any(ringS)) {
      if (ringS) S = get(ring, 3 * (b.south0() + c));
    }
    if (SPAN) {
      N.u *= sn;
      N.v *= sn;
      S.u *= ss;
      S.v *= ss;
    }
  }
};
}  // namespace

// Levels n0 + 1 .. n0 + steps of the forward sweep from levels n0 and n0 - 1
// (n0 = 0: from the packed FP64 controls x, level 0 written as well).
// traj_out (nullable): the packed FP64 trajectory, written beside each level.
template <int NT, int K, bool TWO>
__device__ __forceinline__ void fwd_blk(const Dom<double>& D, const BlkWork& w, int n0, int steps,
                                        const double* __restrict__ x, double* __restrict__ traj_out) {
  constexpr int NI = border_items(NT);
  extern __shared__ double lds[];
  if (D.active && !D.active[w.box]) return;
  const SubDev S = D.subs[w.box];
  const int L = S.nlev - 1;
  if (n0 > L || (n0 == L && n0 > 0)) return;
  steps = min(steps, L - n0);
  const int t = threadIdx.x, nx = S.nx, ncell = S.ncell;
  const int64_t plane = ncell;
  const Range in = grown(w, steps, nx, ncell);
  const Range first = grown(w, max(steps - 1, 0), nx, ncell);
  const Frame F = {in.lo / nx, (in.hi - 1) / nx, nx + 2};
  double* fr = lds;
  double* fo = lds + F.size();              // TWO: the frame of the level before
  double* tab = lds + (TWO ? 2 : 1) * F.size();
  fill_rows<NT, false>(tab, D, S, F);
  const double h0 = D.h0, st = D.st, stg = D.stg;

  // level n0 into the frame
  for (int m = in.lo + t; m < in.hi; m += NT) {
    const int r = m / nx, c = m - r * nx;
    V3<double> z;
    if (n0 == 0) {
      const double* xs = x + S.ctrl_off + m;
      z = {xs[0] - h0, xs[plane], xs[2 * plane]};
      if (m >= w.out0 && m < w.out1) {
        double* o = state(D, S, 0) + m;
        o[0] = z.h;
        o[plane] = z.u;
        o[2 * plane] = z.v;
        if (traj_out) {
          double* q = traj_out + S.traj_off + m;
          q[0] = z.h + h0;
          q[plane] = z.u;
          q[2 * plane] = z.v;
        }
      }
    } else {
      z = ld_box(state(D, S, n0), plane, m, 1.0);
    }
    put_cell(fr, F, S, D.half, r, c, z, -1.0);
  }
  if (steps <= 0) return;                   // a one-level box: level 0 only
  const Border B(S, F);
  int bpos[NI], bk[NI];
  bool bon[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    bon[i] = t + i * NT < B.count();
    B.item(t + i * NT, S, F, &bpos[i], &bk[i]);
  }
  // (a level's ring values are loaded one level ahead)
  auto ring_at = [&](int n, int b) {
    return ld_ring(D.ring + S.ring_off + int64_t(n) * 3 * S.nring, S.nring, bk[b]);
  };
#pragma unroll
  for (int b = 0; b < NI; ++b)
    if (bon[b]) put(fr, bpos[b], ring_at(n0, b));
  __syncthreads();

  // the cells of this thread: chunk by chunk from the first computed one
  const int cb = (first.lo & ~63) + t;
  V3<double> prev[K];
  int rc[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int m = cb + p * NT;
    const int r = m / nx, c = m - r * nx;
    rc[p] = cell_word(r - F.rb, c, 0);
    prev[p] = {0.0, 0.0, 0.0};
    if (m >= first.lo && m < first.hi) {
      prev[p] = n0 > 0 ? ld_box(state(D, S, n0 - 1), plane, m, 1.0) : get(fr, F.pos(r, c));
      if (TWO) put(fo, F.pos(r, c), prev[p]);
    }
  }

  for (int i = 0; i < steps; ++i) {
    const int n = n0 + i;
    const Range g = grown(w, steps - 1 - i, nx, ncell);
    const bool more = i + 1 < steps;
    V3<double> ring[NI];
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (more && bon[b]) ring[b] = ring_at(n + 1, b);
    double* out = state(D, S, n + 1);
    const double wgt = n == 0 ? 0.5 : 1.0;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int m = here(cb) + p * NT;
      if (m < g.lo || m >= g.hi) continue;
      const int cell = here(rc[p]), row = cell_row(cell);
      const int q = ((row + 1) * F.fw + cell_col(cell) + 1) * 3, up = F.fw * 3;
      const double* k = tab + kRowTab * row;
      const V3<double> C = get(fr, q), E = get(fr, q + 3), W = get(fr, q - 3);
      const V3<double> N = get(fr, q + up), Sv = get(fr, q - up);
      const V3<double> f = swe_increment(C, E, W, N, Sv, k[0], k[1], k[2], k[4], k[5], k[3], k[6], st, stg, h0);
      const V3<double> b = TWO ? get(fo, q) : prev[p];
      const V3<double> z = {b.h + wgt * f.h, b.u + wgt * f.u, b.v + wgt * f.v};
      if (!TWO) prev[p] = z;
      else if (more) put_cell(fo, F, S, D.half, F.rb + row, cell_col(cell), z, -1.0);
      if (m >= w.out0 && m < w.out1) {
        out[m] = z.h;
        out[plane + m] = z.u;
        out[2 * plane + m] = z.v;
        if (traj_out) {
          double* o = traj_out + S.traj_off + int64_t(n + 1) * 3 * plane + m;
          o[0] = z.h + h0;
          o[plane] = z.u;
          o[2 * plane] = z.v;
        }
      }
    }
    if (!more) break;
    if (!TWO) {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < K; ++p) {
        const int m = here(cb) + p * NT;
        if (m < g.lo || m >= g.hi) continue;
        const int cell = here(rc[p]), r = F.rb + cell_row(cell), c = cell_col(cell);
        const V3<double> old = get(fr, F.pos(r, c));
        put_cell(fr, F, S, D.half, r, c, prev[p], -1.0);
        prev[p] = old;
      }
    }
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (bon[b]) put(TWO ? fo : fr, bpos[b], ring[b]);
    __syncthreads();
    if (TWO) {
      double* f = fr;
      fr = fo;
      fo = f;
    }
  }
}

template <int NT, int K, bool TWO>
__global__ __launch_bounds__(NT) void k_fwd_blk(Dom<double> D, const BlkWork* __restrict__ work,
                                                int n0, int steps, const double* __restrict__ x,
                                                double* __restrict__ traj_out) {
  const BlkWork w = work[blockIdx.x];
  fwd_blk<NT, K, TWO>(D, w, n0, steps, x, traj_out);
}

// Levels n0 + 1 .. n0 + steps of the tangent-linear sweep about the stored
// trajectory (n0 = 0: from the packed FP64 perturbation dx).  dtraj_out
// (nullable): the packed FP64 perturbation trajectory.
template <int NT, int K, bool SPAN, bool TWO>
__global__ __launch_bounds__(NT) void k_tlm_blk(Dom<double> D, const BlkWork* __restrict__ work,
                                                int n0, int steps, const double* __restrict__ dx,
                                                double* __restrict__ dtraj_out) {
  constexpr int NI = border_items(NT);
  extern __shared__ double lds[];
  const BlkWork w = work[blockIdx.x];
  if (D.active && !D.active[w.box]) return;
  const SubDev S = D.subs[w.box];
  const int L = S.nlev - 1;
  if (n0 > L || (n0 == L && n0 > 0)) return;
  steps = min(steps, L - n0);
  const int t = threadIdx.x, nx = S.nx, ncell = S.ncell;
  const int64_t plane = ncell;
  const Range in = grown(w, steps, nx, ncell);
  const Range first = grown(w, max(steps - 1, 0), nx, ncell);
  const Frame F = {in.lo / nx, (in.hi - 1) / nx, nx + 2};
  double* fr = lds;
  double* fo = lds + F.size();              // TWO: the frame of the level before
  double* tab = lds + (TWO ? 2 : 1) * F.size();
  fill_rows<NT, false>(tab, D, S, F);
  const double h0 = D.h0, st = D.st, stg = D.stg;
  double* dz = D.dz + S.zoff;
  auto store = [&](int n, int m, const V3<double>& v) {
    double* o = dz + int64_t(n) * 3 * plane + m;
    o[0] = v.h;
    o[plane] = v.u;
    o[2 * plane] = v.v;
    if (dtraj_out) {
      double* q = dtraj_out + S.traj_off + int64_t(n) * 3 * plane + m;
      q[0] = v.h;
      q[plane] = v.u;
      q[2 * plane] = v.v;
    }
  };
  for (int m = in.lo + t; m < in.hi; m += NT) {
    const int r = m / nx, c = m - r * nx;
    const V3<double> z = ld_box(n0 == 0 ? dx + S.ctrl_off : dz + int64_t(n0) * 3 * plane, plane, m, 1.0);
    if (n0 == 0 && m >= w.out0 && m < w.out1) store(0, m, z);
    put_cell(fr, F, S, D.half, r, c, z, -1.0);
  }
  if (steps <= 0) return;
  // the frozen ring is not perturbed: zeros on the frame's border; the state's
  // ring of a level is staged behind the row table
  const Border B(S, F);
  double* ring = tab + kRowTab * F.rows();
  double* ringo = ring + 3 * B.count();     // TWO: the next level's
  int bk[NI];
  auto ring_at = [&](int n, int b) {
    return ld_ring(D.ring + S.ring_off + int64_t(n) * 3 * S.nring, S.nring, bk[b]);
  };
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    int pos;
    B.item(t + i * NT, S, F, &pos, &bk[i]);
    if (t + i * NT < B.count()) {
      put(fr, pos, {0.0, 0.0, 0.0});
      if (TWO) put(fo, pos, {0.0, 0.0, 0.0});
      put(ring, 3 * (t + i * NT), ring_at(n0, i));
    }
  }
  __syncthreads();
  // the cells of this thread, chunk by chunk from the first computed one; a
  // lane past the computed range takes its nearest cell and keeps no result
  const int cb = (first.lo & ~63) + t;
  V3<double> prev[K];
  int rc[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int m = min(max(cb + p * NT, first.lo), first.hi - 1);
    const int r = m / nx, c = m - r * nx;
    rc[p] = cell_word(r - F.rb, c, 0);
    prev[p] = n0 > 0 ? ld_box(dz + int64_t(n0 - 1) * 3 * plane, plane, m, 1.0) : get(fr, F.pos(r, c));
    if (TWO && m == cb + p * NT) put(fo, F.pos(r, c), prev[p]);
  }
  // the state's loads of a pass, issued together at its start
  auto issue = [&](State5<SPAN>& q, int p, int n, const Range& g) {
    const int m = here(cb) + p * NT;
    const int chunk = __builtin_amdgcn_readfirstlane(m & ~63);
    if (chunk >= g.hi || chunk + 64 <= g.lo) return;          // uniform over the wave
    const int cell = here(rc[p]);
    q.load(state(D, S, n), plane, S, D.half, min(max(m, first.lo), first.hi - 1),
           F.rb + cell_row(cell), cell_col(cell));
  };
  for (int i = 0; i < steps; ++i) {
    const int n = n0 + i;
    const Range g = grown(w, steps - 1 - i, nx, ncell);
    const bool more = i + 1 < steps;
    const double wgt = n == 0 ? 0.5 : 1.0;
    V3<double> rv[NI];
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (more && t + b * NT < B.count()) rv[b] = ring_at(n + 1, b);
#pragma unroll
    for (int p = 0; p < K; ++p) {
      State5<SPAN> q;
      issue(q, p, n, g);
      const int m = here(cb) + p * NT;
      const int chunk = __builtin_amdgcn_readfirstlane(m & ~63);
      if (chunk >= g.hi || chunk + 64 <= g.lo) continue;
      const int cell = here(rc[p]), row = cell_row(cell), c = cell_col(cell);
      q.fix(ring, B, row, c);
      const int a = ((row + 1) * F.fw + c + 1) * 3, up = F.fw * 3;
      const double* k = tab + kRowTab * row;
      const V3<double> f = swe_tangent(q.C, q.E, q.W, q.N, q.S, get(fr, a), get(fr, a + 3),
                                       get(fr, a - 3), get(fr, a + up), get(fr, a - up), k[0], k[1],
                                       k[2], k[4], k[5], k[3], k[6], st, stg, h0);
      if (m >= g.lo && m < g.hi) {
        const V3<double> b = TWO ? get(fo, a) : prev[p];
        const V3<double> z = {b.h + wgt * f.h, b.u + wgt * f.u, b.v + wgt * f.v};
        if (!TWO) prev[p] = z;
        else if (more) put_cell(fo, F, S, D.half, F.rb + row, c, z, -1.0);
        if (m >= w.out0 && m < w.out1) store(n + 1, m, z);
      }
    }
    if (!more) break;
    if (!TWO) {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < K; ++p) {
        const int m = here(cb) + p * NT;
        if (m < g.lo || m >= g.hi) continue;
        const int cell = here(rc[p]), r = F.rb + cell_row(cell), c = cell_col(cell);
        const V3<double> old = get(fr, F.pos(r, c));
        put_cell(fr, F, S, D.half, r, c, prev[p], -1.0);
        prev[p] = old;
      }
    }
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (t + b * NT < B.count()) put(TWO ? ringo : ring, 3 * (t + b * NT), rv[b]);
    __syncthreads();
    if (TWO) {
      double* f = fr;
      fr = fo;
      fo = f;
      f = ring;
      ring = ringo;
      ringo = f;
    }
  }
}

// Levels nhi .. nlo of the adjoint sweep (modes as k_adj).  lam: the adjoint
// arena, four slots per box; the launch reads lambda^{nhi+1}, lambda^{nhi+2}
// from slots 2 pin, 2 pin + 1 and leaves lambda^{nlo}, lambda^{nlo+1} in
// slots 2 (1 - pin), 2 (1 - pin) + 1 (other blocks of the box still read the
// first two).
template <int NT, int K, int MODE, bool SPAN, bool TWO>
__device__ __forceinline__ void adj_blk(const Dom<double>& D, const BlkWork& w, int nhi, int nlo, int pin,
                                        const double* __restrict__ x, const double* __restrict__ xb,
                                        const double* __restrict__ forcing, double* __restrict__ out) {
  constexpr int NI = border_items(NT);
  extern __shared__ double lds[];
  if (D.active && !D.active[w.box]) return;
  const SubDev S = D.subs[w.box];
  const int L = S.nlev - 1;
  if (nlo > L) return;
  const int top = min(nhi, L), steps = top - nlo + 1;
  const bool begin = top == L;
  const int t = threadIdx.x, nx = S.nx, ncell = S.ncell;
  const int64_t plane = ncell;
  const Range in = grown(w, steps, nx, ncell), first = grown(w, steps - 1, nx, ncell);
  const Frame F = {in.lo / nx, (in.hi - 1) / nx, nx + 2};
  double* fr = lds;
  double* fo = lds + F.size();              // TWO: the frame of the level before
  double* tab = lds + (TWO ? 2 : 1) * F.size();
  // the state's ring of a level, staged; J of each 64-cell chunk of the block
  const Border B(S, F);
  double* ring = tab + kRowTab * F.rows();
  double* ringo = ring + 3 * B.count();     // TWO: the next level's
  double* pj = ring + (TWO ? 6 : 3) * B.count();
  const int nchunk = (w.out1 - w.out0 + 63) / 64, npj = (nchunk + 3) & ~3;
  double* pjo = pj + npj;                   // TWO: the next level's
  int* tcnt = reinterpret_cast<int*>(pj + (TWO ? 2 : 1) * npj);   // intervals covering a level
  if (MODE != 1)
    for (int i = t; i < steps; i += NT) tcnt[i] = D.tcount[S.lev0 + nlo + i];
  fill_rows<NT, true>(tab, D, S, F);
  const double h0 = D.h0, st = D.st, stg = D.stg;
  const double mis[3] = {D.mu * D.isb2[0], D.mu * D.isb2[1], D.mu * D.isb2[2]};
  double* A = D.adj + (S.adj_off / 9) * 12;
  const double* l1 = A + int64_t(2 * pin) * 3 * plane;
  const double* l2 = A + int64_t(2 * pin + 1) * 3 * plane;

  // lambda^{top+1}, zero past the box's last level and on the border
  for (int i = t; i < (TWO ? 2 : 1) * F.size(); i += NT) fr[i] = 0.0;
  for (int i = t; i < (TWO ? 2 : 1) * npj; i += NT) pj[i] = 0.0;
  int bk[NI];
  auto ring_at = [&](int n, int b) {
    return ld_ring(D.ring + S.ring_off + int64_t(n) * 3 * S.nring, S.nring, bk[b]);
  };
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    int pos;
    B.item(t + i * NT, S, F, &pos, &bk[i]);
    if (t + i * NT < B.count()) {
      put(ring, 3 * (t + i * NT), ring_at(top, i));
    }
  }
  __syncthreads();
  if (!begin)
    for (int m = in.lo + t; m < in.hi; m += NT) {
      const int r = m / nx;
      put_cell(fr, F, S, D.half, r, m - r * nx, ld_box(l1, plane, m, 1.0), 1.0);
    }
  // the cells of this thread, chunk by chunk from the first computed one; a
  // lane past the computed range takes its nearest cell and keeps no result
  const int cb = (first.lo & ~63) + t;
  V3<double> prev[K];
  int rc[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const int m = min(max(cb + p * NT, first.lo), first.hi - 1);
    const int r = m / nx;
    rc[p] = cell_word(r - F.rb, m - r * nx, MODE != 1 ? int(D.cover[S.cell_off + m]) : 0);
    prev[p] = {0.0, 0.0, 0.0};
    if (!begin) {
      prev[p] = ld_box(l2, plane, m, 1.0);
      if (TWO && m == cb + p * NT) put(fo, F.pos(r, m - r * nx), prev[p]);
    }
  }
  // thread q: J of the block's q-th tile
  const int ntile = (w.out1 - w.out0 + kTile - 1) / kTile;
  double jt = 0.0;
  double* jp = D.jpart + S.tile0 + w.out0 / kTile + t;
  if ((MODE == 0 || MODE == 2) && !begin && t < ntile) jt = *jp;
  __syncthreads();

  // a pass's loads, issued together at its start: the state around the cell, the
  // overlap target (mode 3: the perturbation; mode 1: the caller's forcing), the
  // tile's observations
  struct Pass {
    State5<SPAN> q;
    V3<double> f;
    int bin;
  };
  auto issue = [&](Pass& b, int p, int n, const Range& g) {
    const int m = here(cb) + p * NT;
    const int chunk = __builtin_amdgcn_readfirstlane(m & ~63);
    if (chunk >= g.hi || chunk + 64 <= g.lo) return;          // uniform over the wave
    const int cell = here(rc[p]), mm = min(max(m, first.lo), first.hi - 1);
    b.q.load(state(D, S, n), plane, S, D.half, mm, F.rb + cell_row(cell), cell_col(cell));
    const int64_t lev = S.traj_off + int64_t(n) * 3 * plane;
    if (MODE == 1) {
      b.f = State5<SPAN>::at(forcing + lev, plane, uint32_t(mm) * 8u);
    } else if (MODE == 3) {
      b.f = State5<SPAN>::at(D.dz + S.zoff + int64_t(n) * 3 * plane, plane, uint32_t(mm) * 8u);
    } else {
      // cells no other box covers read element 0 (weight zero)
      const bool covered = cell_cover(cell) * tcnt[n - nlo] > 1;
      b.f = State5<SPAN>::at(D.targ + lev, plane, covered ? uint32_t(mm) * 8u : 0u);
    }
    // (a vector load: a scalar one would be waited for with the LDS reads)
    if (MODE != 1)
      b.bin = D.obs_bin[obs_key(S.tile0, S.ntile, D.maxlev, max(chunk, first.lo) / kTile, n) + here(0)];
  };
  for (int n = top; n >= nlo; --n) {
    const Range g = grown(w, n - nlo, nx, ncell);
    V3<double> rv[NI];
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (n > nlo && t + b * NT < B.count()) rv[b] = ring_at(n - 1, b);
    const int tc = MODE != 1 ? tcnt[n - nlo] : 0;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      Pass buf;
      issue(buf, p, n, g);
      const int m = here(cb) + p * NT;
      const int chunk = __builtin_amdgcn_readfirstlane(m & ~63);
      if (chunk >= g.hi || chunk + 64 <= g.lo) continue;      // uniform over the wave
      State5<SPAN>& q = buf.q;
      const V3<double>& tg = buf.f;
      const int bin = buf.bin;
      double jloc = 0.0;
      {
        const int cell = here(rc[p]), row = cell_row(cell), c = cell_col(cell);
        const int kc = cell_cover(cell) * tc - 1;
        double f[3] = {0.0, 0.0, 0.0};
        if (MODE == 1) {
          f[0] = tg.h;
          f[1] = tg.u;
          f[2] = tg.v;
        }
        q.fix(ring, B, row, c);
        __builtin_amdgcn_sched_barrier(0);
        const V3<double>& C = q.C;
        const int a = ((row + 1) * F.fw + c + 1) * 3, up = F.fw * 3;
        const double* k = tab + kRowTab * row;
        const V3<double> l0 = get(fr, a);
        const V3<double> ew = swe_adjoint_ew(C, q.E, q.W, q.N, q.S, l0, get(fr, a + 3), get(fr, a - 3),
                                             k[0], k[1], k[4], k[5], st, h0);
        __builtin_amdgcn_sched_barrier(0);
        const V3<double> v = swe_adjoint_ns(ew, C, q.N, q.S, get(fr, a + up), get(fr, a - up), k[6],
                                            k[2], k[3], q.sn, q.ss, st, stg, h0);
        double ah = v.h, au = v.u, av = v.v;
        asm volatile("" : "+v"(ah), "+v"(au), "+v"(av));   // computed here
        if (n == 0) {                        // (a branch, not selects at every level)
          asm volatile("");
          au = l0.u + 0.5 * au;
          av = l0.v + 0.5 * av;
          ah = l0.h + 0.5 * ah;
        }
        if (MODE != 1) {
          if (__builtin_amdgcn_readfirstlane(bin) >= 0)
            obs_terms(D, bin, (chunk / 64) & 3, MODE == 3 ? tg : C, MODE == 3, f, jloc);
          const V3<double> e = MODE == 3 ? tg : V3<double>{C.h - tg.h, C.u - tg.u, C.v - tg.v};
          overlap_terms(e, kc, mis, MODE != 3, f, jloc);
        }
        const V3<double> b = TWO ? get(fo, a) : prev[p];
        const double bh = f[0] + ah + b.h;
        const double bu = f[1] + au + b.u;
        const double bv = f[2] + av + b.v;
        if (m >= g.lo && m < g.hi) {
          if (!TWO) prev[p] = {bh, bu, bv};
          else if (n > nlo) put_cell(fo, F, S, D.half, F.rb + row, c, {bh, bu, bv}, 1.0);
        }
        const bool own = m >= w.out0 && m < w.out1;
        if (n == nlo && n > 0 && own) {
          double* b0 = A + int64_t(2 - 2 * pin) * 3 * plane + m;
          double* b1 = A + int64_t(3 - 2 * pin) * 3 * plane + m;
          b0[0] = bh;
          b0[plane] = bu;
          b0[2 * plane] = bv;
          b1[0] = l0.h;
          b1[plane] = l0.u;
          b1[2 * plane] = l0.v;
        } else if (n == 0 && own) {
          const int64_t o = S.ctrl_off + m;
          double gh = bh, gu = bu, gv = bv;
          if (MODE == 0) {
            const double wb = D.weight_mode ? 1.0 : 1.0 / double(cell_cover(cell));
            const double dh = x[o] - xb[o];
            const double du = x[o + plane] - xb[o + plane];
            const double dv = x[o + 2 * plane] - xb[o + 2 * plane];
            gh = wb * dh * D.isb2[0] + bh;
            gu = wb * du * D.isb2[1] + bu;
            gv = wb * dv * D.isb2[2] + bv;
            jloc += 0.5 * wb * (dh * dh * D.isb2[0] + du * du * D.isb2[1] + dv * dv * D.isb2[2]);
          }
          out[o] = gh;
          out[o + plane] = gu;
          out[o + 2 * plane] = gv;
          flag_nonfinite(D.nonfinite, !(isfinite(gh) && isfinite(gu) && isfinite(gv)));
        }
        if (!own) jloc = 0.0;
      }
      if ((MODE == 0 || MODE == 2) && chunk >= w.out0 && chunk < w.out1) {
        jloc = wave_sum(jloc);
        if ((t & 63) == 0) pj[(chunk - w.out0) / 64] = jloc;
      }
    }
    if (TWO && n > nlo) {
#pragma unroll
      for (int b = 0; b < NI; ++b)
        if (t + b * NT < B.count()) put(ringo, 3 * (t + b * NT), rv[b]);
    }
    __syncthreads();
    if ((MODE == 0 || MODE == 2) && t < ntile) {
      const double* s = pj + 4 * t;
      const double tot = 0.0 + s[0] + s[1] + s[2] + s[3];
      jt = n == L ? tot : jt + tot;
    }
    if (n == nlo) break;
    if (TWO) {
      double* f = fr;
      fr = fo;
      fo = f;
      f = ring;
      ring = ringo;
      ringo = f;
      f = pj;
      pj = pjo;
      pjo = f;
      continue;
    }
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int m = here(cb) + p * NT;
      if (m < g.lo || m >= g.hi) continue;
      const int cell = here(rc[p]), r = F.rb + cell_row(cell), c = cell_col(cell);
      const V3<double> old = get(fr, F.pos(r, c));
      put_cell(fr, F, S, D.half, r, c, prev[p], 1.0);
      prev[p] = old;
    }
#pragma unroll
    for (int b = 0; b < NI; ++b)
      if (t + b * NT < B.count()) put(ring, 3 * (t + b * NT), rv[b]);
    __syncthreads();
  }
  if ((MODE == 0 || MODE == 2) && t < ntile) *jp = jt;
}

template <int NT, int K, int MODE, bool SPAN, bool TWO>
__global__ __launch_bounds__(NT) void k_adj_blk(Dom<double> D, const BlkWork* __restrict__ work,
                                                int nhi, int nlo, int pin,
                                                const double* __restrict__ x,
                                                const double* __restrict__ xb,
                                                const double* __restrict__ forcing,
                                                double* __restrict__ out) {
  const BlkWork w = work[blockIdx.x];
  adj_blk<NT, K, MODE, SPAN, TWO>(D, w, nhi, nlo, pin, x, xb, forcing, out);
}

// Both sweeps of the cost and its gradient, where every block is a whole box:
// the adjoint reads the levels that its own workgroup has just written, from
// its XCD's L2 (a launch of its own starts with that cache's lines dropped),
// and one launch is saved: 8 boxes of 18 x 36, 13 levels 52.4 -> 49.5 us.
template <int NT, int K, bool SPAN, bool TWO>
__global__ __launch_bounds__(NT) void k_eval_blk(Dom<double> D, const BlkWork* __restrict__ work,
                                                 int levels, const double* __restrict__ x,
                                                 const double* __restrict__ xb,
                                                 double* __restrict__ out) {
  const BlkWork w = work[blockIdx.x];
  fwd_blk<NT, K, TWO>(D, w, 0, levels - 1, x, nullptr);
  __syncthreads();
  adj_blk<NT, K, 0, SPAN, TWO>(D, w, levels - 1, 0, 0, x, xb, nullptr, out);
}

// ---- plan and launchers -------------------------------------------------------
namespace {
constexpr int kBlkThreads = 1024;
constexpr int kBlkPassMax = 6;             // 128 registers hold six passes
constexpr int kBlkPassTwo = 3;             // and the LDS two frames of three

// what a block of `steps` levels a launch takes of a workgroup
struct BlkFit {
  bool ok;                    // it has that
  int passes;                 // cells computed at a launch's first level, in passes
  size_t lds, lds2;           // with one frame, with two
};
// first cell, and the one past the last, of the block grown by e rows
int blk_lo(const SubDev& S, const BlkWork& w, int e) { return std::max(0, w.out0 - e * S.nx); }
int blk_hi(const SubDev& S, const BlkWork& w, int e) { return std::min(S.ncell, w.out1 + e * S.nx); }
BlkFit blk_fit(const SubDev& S, const BlkWork& w, int steps) {
  const int rows = (blk_hi(S, w, steps) - 1) / S.nx - blk_lo(S, w, steps) / S.nx + 1;
  BlkFit f{};
  f.lds = size_t(rows + 2) * (S.nx + 2) * 3 * sizeof(double) + size_t(rows) * kRowTab * sizeof(double) +
          size_t(2 * rows + 2 * S.nx) * 3 * sizeof(double) +
          size_t((w.out1 - w.out0 + 255) / 64) * sizeof(double) + size_t(std::max(steps, S.nlev) + 2) * sizeof(int);
  f.lds2 = f.lds + size_t(rows + 2) * (S.nx + 2) * 3 * sizeof(double) + size_t(2 * rows + 2 * S.nx) * 3 * sizeof(double) +
           size_t((w.out1 - w.out0 + 255) / 64) * sizeof(double);
  f.passes = (blk_hi(S, w, steps - 1) - (blk_lo(S, w, steps - 1) & ~63) + kBlkThreads - 1) / kBlkThreads;
  f.ok = f.lds <= kBlkLdsMax && f.passes <= kBlkPassMax && 2 * (rows + S.nx) <= kBorderMax &&
         S.nx >= 2 && S.ny >= 2;
  return f;
}
// what a block's level costs, both sweeps
struct BlkCost {
  double cells;               // computed, on the mean of a launch's levels
  double us;                  // time on a compute unit of its own
  double bytes;               // memory traffic
};
BlkCost blk_cost(const SubDev& S, const BlkWork& w, int steps) {
  double cells = 0.0;
  for (int e = 0; e < steps; ++e) cells += double(blk_hi(S, w, e) - blk_lo(S, w, e)) / steps;
  const double own = w.out1 - w.out0, in = blk_hi(S, w, steps) - blk_lo(S, w, steps);
  return {cells, 2.0 + 0.0031 * cells, 24.0 * (own + 1.65 * cells + (4.0 * in + 2.0 * own) / steps)};
}
// block b of a box cut into nb blocks of whole tiles: its first tile
int cut_at(const SubDev& S, int nb, int b) { return int(int64_t(S.ntile) * b / nb); }
BlkWork tiles_of(const SubDev& S, int t0, int t1) { return {0, t0 * kTile, std::min(S.ncell, t1 * kTile)}; }

// The boxes of one shape and their cuts into blocks of one number of levels a
// launch.  What a block takes grows with it: reach holds, for each first tile,
// the tiles of the longest block that fits, so that a cut is tested by
// comparisons, and boxes too wide for any block are known at once.
struct BlkShape {
  SubDev S;
  std::vector<int> reach;
  int most, least;            // most tiles of any block that fits; of as many every block fits
  struct Cut {
    std::vector<std::pair<double, BlkWork>> blocks;       // a launch's time, block
    double us = 0.0, longest = 0.0, bytes = 0.0, cells = 0.0;   // cells: of the largest block
    size_t lds = 0, lds2 = 0;
    int passes = 0;
  };
  std::map<int, Cut> cuts;    // by the number of blocks
  std::map<int, int> found;   // fewest blocks that fit, by the number asked for

  // whether every tile fits as a block of its own
  bool prepare(int steps) {
    cuts.clear();
    found.clear();
    reach.assign(S.ntile, 0);
    most = 0;
    least = S.ntile;
    for (int t = 0, end = 0; t < S.ntile; ++t) {
      end = std::max(end, t);
      while (end < S.ntile && blk_fit(S, tiles_of(S, t, end + 1), steps).ok) ++end;
      if (end == t) return false;
      reach[t] = end - t;
      most = std::max(most, reach[t]);
      if (end < S.ntile) least = std::min(least, reach[t]);
    }
    return true;
  }
  // the fewest blocks, at least nb0, of a cut whose blocks all fit
  int blocks(int nb0) {
    auto [it, fresh] = found.try_emplace(nb0, 0);
    if (!fresh) return it->second;
    int nb = std::max(nb0, (S.ntile + most - 1) / most);
    for (; (S.ntile + nb - 1) / nb > least; ++nb) {       // (one block per tile fits)
      int b = 0;
      while (b < nb && cut_at(S, nb, b + 1) - cut_at(S, nb, b) <= reach[cut_at(S, nb, b)]) ++b;
      if (b == nb) break;
    }
    return it->second = nb;
  }
  const Cut& cut(int nb, int steps) {
    auto [it, fresh] = cuts.try_emplace(nb);
    Cut& c = it->second;
    for (int b = 0; fresh && b < nb; ++b) {
      const BlkWork w = tiles_of(S, cut_at(S, nb, b), cut_at(S, nb, b + 1));
      const BlkFit f = blk_fit(S, w, steps);
      const BlkCost q = blk_cost(S, w, steps);
      c.lds = std::max(c.lds, f.lds);
      c.lds2 = std::max(c.lds2, f.lds2);
      c.passes = std::max(c.passes, f.passes);
      c.us += q.us;
      c.longest = std::max(c.longest, q.us);
      c.cells = std::max(c.cells, q.cells);
      c.bytes += q.bytes;
      c.blocks.emplace_back(q.us * std::min(steps, S.nlev), w);
    }
    return c;
  }
};
}  // namespace

// The sweeps that are faster in blocks, where every block has a compute unit of
// its own: `most` cells computed per level in the largest block, `steps` levels
// per launch, `whole` where no box is cut, `cells` of all boxes.  (With more blocks
// than units the step kernels are bound by memory: every sweep was faster in
// blocks, by a fifth at least.)  Lines through measured times of a level, us:
// a block's grow with its cells and, cut, with the levels that a launch loads; a
// step kernel's are a launch, and more with more cells, until memory binds it.
// Step kernel against block:
//                          forward     cost adj.  forced adj.  tangent   product
//   2 spheres 20 x 50     3.6 -> 1.5  5.4 -> 3.2  4.0 -> 2.5  3.8 -> 2.7   8.4 -> 5.7
//   2 spheres 24 x 70     3.5 -> 2.3  5.3 -> 4.6  3.9 -> 3.7  3.8 -> 4.0   8.4 -> 8.5
//   2 spheres 25 x 84     3.5 -> 2.6  5.2 -> 5.7  3.9 -> 4.9  3.8 -> 5.0   8.4 -> 10.9
//   2 spheres 33 x 86     3.6 -> 3.7  5.2 -> 7.6  4.0 -> 6.1  3.8 -> 6.5   8.6 -> 14.0
//   64 boxes 26 x 64      4.3 -> 2.3  6.6 -> 5.1  5.2 -> 3.8  5.1 -> 4.2  11.4 -> 9.1
//   4 boxes 40 x 358,
//    128 blocks, 3 levels 3.5 -> 3.1  5.6 -> 6.4  4.4 -> 5.3  4.0 -> 4.8  11.9 -> 14.3
//   24 boxes 34 x 266,
//    192 blocks, 5 levels 5.1 -> 3.7  7.9 -> 7.9  6.6 -> 6.7  6.3 -> 6.3  16.3 -> 16.7
//   32 boxes 38 x 246,
//    192 blocks, 5 levels 6.6 -> 4.0 11.0 -> 8.7  9.2 -> 7.5  8.3 -> 7.0  21.9 -> 19.3
int blk_faster(double most, int steps, bool whole, double cells) {
  struct Line {
    double block, per_cell, launch, launch_cut, step, step_per_cell, step_memory;
    double gain(double most, int steps, bool whole, double cells) const {
      return std::max(step + step_per_cell * cells, step_memory * cells) -
             (block + per_cell * most + (whole ? launch : launch_cut) / steps);
    }
  };
  constexpr Line fwd = {0.5, 0.00107, 2.0, 4.0, 3.5, 0.75e-5, 1.6e-5};
  constexpr Line adj = {1.1, 0.00215, 3.0, 8.5, 5.2, 1.25e-5, 3.2e-5};
  constexpr Line forced = {0.8, 0.0017, 4.0, 7.0, 4.0, 1.25e-5, 2.8e-5};
  constexpr Line gn = {0.9, 0.00215, 4.0, 8.0, 4.6, 1.25e-5, 2.9e-5};
  constexpr Line tlm = {0.85, 0.0020, 1.0, 4.5, 3.8, 1.25e-5, 2.5e-5};
  auto gain = [&](const Line& l) { return l.gain(most, steps, whole, cells); };
  return (gain(fwd) > 0 ? kBlkFwd : 0) | (gain(adj) > 0 ? kBlkAdj : 0) | (gain(forced) > 0 ? kBlkForced : 0) |
         (gain(tlm) > 0 ? kBlkTlm : 0) | (gain(tlm) + gain(gn) > 0 ? kBlkProduct : 0);
}

// The decomposition into blocks that the model below finds fastest for an
// evaluation, and the sweeps that it serves; not ok where no box decomposition
// fits or the step kernels are faster.  Measured (both sweeps, one block to a
// compute unit): a level takes 3.9 us for 570 cells and 9.4 us for 2350, 10 us
// per launch besides; memory moves 4 TB/s under these kernels; the step kernels
// are taken at 4.5 and 6.5 us per level (3.5 and 5.2 on the smallest problems:
// blk_faster has the last word), or 72 + 111 B per cell at 4.4 TB/s.  More blocks
// than boxes spread few boxes over the chip (64 boxes of 40 x 72 cells: 64 whole
// ones 430 us per evaluation, 256 blocks of 7 levels 301 us, 480 of 5 454 us), at the
// price of the rows that two blocks compute both.
BlkPlan plan_blocks(const std::vector<SubDev>& subs, int maxlev, int cus) {
  double cells = 0.0;
  for (const SubDev& S : subs) cells += S.ncell;
  const int levels = std::max(1, maxlev - 1);
  // boxes of one shape are cut alike
  std::vector<BlkShape> shapes;
  std::vector<int> shape(subs.size());
  {
    std::map<std::array<int, 4>, int> index;
    for (size_t s = 0; s < subs.size(); ++s) {
      const SubDev& S = subs[s];
      const auto [it, fresh] = index.try_emplace({S.ny, S.nx, S.nlev, S.span}, int(shapes.size()));
      if (fresh) shapes.emplace_back().S = S;
      shape[s] = it->second;
    }
  }
  BlkPlan best{};
  double best_us = levels * (std::max(4.5, cells * 72 / 4.4e6) + std::max(6.5, cells * 111 / 4.4e6));
  for (int k : {levels, 24, 16, 12, 10, 8, 7, 6, 5, 4, 3}) {
    if (k > levels) continue;
    auto whole = [&](const SubDev& S) { return S.span || k == levels; };       // not to be cut
    bool fits = true;
    for (BlkShape& q : shapes) {
      if (whole(q.S)) {
        q.cuts.clear();
        fits = blk_fit(q.S, tiles_of(q.S, 0, q.S.ntile), k).ok;
      } else {
        fits = q.prepare(k);
      }
      if (!fits) break;
    }
    if (!fits) continue;
    std::vector<const BlkShape::Cut*> cut(shapes.size());
    for (int want : {1, cus / 2, cus * 3 / 4, cus * 7 / 8, cus, 2 * cus}) {     // blocks wanted on the whole
      BlkPlan p{};
      p.ok = true;
      p.levels = k;
      double sum = 0.0, longest = 0.0, bytes = 0.0, most = 0.0;
      size_t lds2 = 0, nwork = 0;
      for (size_t i = 0; i < shapes.size(); ++i) {
        BlkShape& q = shapes[i];
        const int nb0 = std::min(q.S.ntile, std::max(1, int(want * (q.S.ncell / cells) + 0.5)));
        cut[i] = &q.cut(whole(q.S) ? 1 : q.blocks(nb0), k);
        p.lds = std::max(p.lds, cut[i]->lds);
        lds2 = std::max(lds2, cut[i]->lds2);
        p.passes = std::max(p.passes, cut[i]->passes);
        longest = std::max(longest, cut[i]->longest);
        most = std::max(most, cut[i]->cells);
      }
      for (int i : shape) {
        sum += cut[i]->us;
        bytes += cut[i]->bytes;
        nwork += cut[i]->blocks.size();
      }
      const double pack = int(nwork) <= cus ? longest : sum / cus + 0.5 * longest;
      const double us = (levels + k - 1) / k * 10.0 + levels * std::max(pack, bytes / 4.0e6);
      if (us >= best_us) continue;
      p.sweeps = int(nwork) <= cus ? blk_faster(most, k, nwork == subs.size(), cells) : kBlkAll;
      p.two = p.passes <= kBlkPassTwo && lds2 <= kBlkLdsMax;
      if (p.two) p.lds = lds2;
      best = p;
      best_us = us;
      best.us = us;
      if (k == levels) best.levels = maxlev;          // no box is cut: one launch per sweep
      std::vector<std::pair<double, BlkWork>> work;
      for (size_t s = 0; s < subs.size(); ++s)
        for (auto w : cut[shape[s]]->blocks) {
          w.second.box = int(s);
          work.push_back(w);
        }
      // launch order: the longest first where blocks differ, else box by box
      // (one XCD holding neighbouring blocks, as the step kernels do: 8.0 ->
      // 8.5 ms on 1024 boxes of 72 x 136 cells)
      if (longest > 1.25 * sum / double(nwork))
        std::stable_sort(work.begin(), work.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
      best.work.clear();
      for (const auto& w : work) best.work.push_back(w.second);
    }
  }
  best.ok = best.ok && best.sweeps;
  return best;
}

namespace {
template <typename F>
hipError_t blk_allow(F* k) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(kBlkLdsMax));
}
template <int K, bool SPAN, bool TWO>
hipError_t blk_prepare_k() {
  hipError_t e = blk_allow(&k_fwd_blk<kBlkThreads, K, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_eval_blk<kBlkThreads, K, SPAN, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_tlm_blk<kBlkThreads, K, SPAN, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_adj_blk<kBlkThreads, K, 0, SPAN, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_adj_blk<kBlkThreads, K, 1, SPAN, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_adj_blk<kBlkThreads, K, 2, SPAN, TWO>);
  if (e == hipSuccess) e = blk_allow(&k_adj_blk<kBlkThreads, K, 3, SPAN, TWO>);
  return e;
}
// f(passes, span, two frames) with the smallest compiled pass count that holds p
template <typename F>
void with_plan(int p, bool span, bool two, F f) {
  auto go = [&](auto k) {
    constexpr int K = decltype(k)::value;
    auto frames = [&](auto sp) {
      if constexpr (K <= kBlkPassTwo) {
        if (two) return f(k, sp, std::true_type{});
      }
      f(k, sp, std::false_type{});
    };
    if (span) frames(std::true_type{});
    else frames(std::false_type{});
  };
  if (p <= 1) go(std::integral_constant<int, 1>{});
  else if (p <= 2) go(std::integral_constant<int, 2>{});
  else if (p <= 3) go(std::integral_constant<int, 3>{});
  else if (p <= 4) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, kBlkPassMax>{});
}
}  // namespace

hipError_t blk_prepare(int passes, bool span, bool two) {
  hipError_t e = hipSuccess;
  with_plan(passes, span, two, [&](auto k, auto s, auto w) {
    e = blk_prepare_k<decltype(k)::value, decltype(s)::value, decltype(w)::value>();
  });
  return e;
}

void launch_fwd_blk(const Dom<double>& D, const BlkLaunch& b, int n0, int levels, const double* x, double* traj_out,
                    hipStream_t st) {
  with_plan(b.passes, false, b.two, [&](auto k, auto, auto w) {
    auto* kern = &k_fwd_blk<kBlkThreads, decltype(k)::value, decltype(w)::value>;
    hipLaunchKernelGGL(kern, dim3(b.nwork), dim3(kBlkThreads), b.lds, st, D, b.work, n0, levels, x, traj_out);
  });
}
void launch_tlm_blk(const Dom<double>& D, const BlkLaunch& b, int n0, int levels, const double* dx, double* dtraj_out,
                    hipStream_t st) {
  with_plan(b.passes, b.span, b.two, [&](auto k, auto s, auto w) {
    auto* kern = &k_tlm_blk<kBlkThreads, decltype(k)::value, decltype(s)::value, decltype(w)::value>;
    hipLaunchKernelGGL(kern, dim3(b.nwork), dim3(kBlkThreads), b.lds, st, D, b.work, n0, levels, dx, dtraj_out);
  });
}
void launch_adj_blk(const Dom<double>& D, const BlkLaunch& b, int mode, int nhi, int nlo, int pin,
                    const double* x, const double* xb, const double* forcing, double* out,
                    hipStream_t st) {
  with_plan(b.passes, b.span, b.two, [&](auto k, auto s, auto w) {
    constexpr int K = decltype(k)::value;
    constexpr bool SPAN = decltype(s)::value, TWO = decltype(w)::value;
    auto* kern = mode == 0 ? &k_adj_blk<kBlkThreads, K, 0, SPAN, TWO>
                 : mode == 1 ? &k_adj_blk<kBlkThreads, K, 1, SPAN, TWO>
                 : mode == 2 ? &k_adj_blk<kBlkThreads, K, 2, SPAN, TWO> : &k_adj_blk<kBlkThreads, K, 3, SPAN, TWO>;
    hipLaunchKernelGGL(kern, dim3(b.nwork), dim3(kBlkThreads), b.lds, st, D, b.work, nhi, nlo, pin, x, xb,
                       forcing, out);
  });
}

void launch_eval_blk(const Dom<double>& D, const BlkLaunch& b, int levels, const double* x, const double* xb,
                     double* out, hipStream_t st) {
  with_plan(b.passes, b.span, b.two, [&](auto k, auto s, auto w) {
    auto* kern = &k_eval_blk<kBlkThreads, decltype(k)::value, decltype(s)::value, decltype(w)::value>;
    hipLaunchKernelGGL(kern, dim3(b.nwork), dim3(kBlkThreads), b.lds, st, D, b.work, levels, x, xb, out);
  });
}

}  // namespace dd4dvar
