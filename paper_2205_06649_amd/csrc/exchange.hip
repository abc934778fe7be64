// Exchange between subdomains in device memory ("Exchange u_ji between
// adjacent subdomains", Alg. 1) and the partition-of-unity gather (eq. rest).
//
// * Halo rings: every frozen ring position of subdomain s reads, at each of
//   its levels, the core owner of the (pole-mapped) cell in the same time
//   interval, with u and v negated across a pole.
// * Overlap targets: for every (level, cell) of s covered by K other extended
//   space-time boxes, the mean of their trajectories there and, once per
//   subdomain, the constant sum_{s'} (T_{s'} - mean)^2 / sigma_b^2, so that
//   sum_{s'} (Z - T_{s'})^2 = K (Z - mean)^2 + constant.
// * Before any local solve both come from the global background run.
#include <algorithm>

#include "kernels.h"
#include "launch.h"
#include "stencil.h"

namespace dd4dvar {

namespace {
// neighbour entries of a level whose loads are issued together (FP64 values
// take twice the registers)
template <typename T>
constexpr int kGather = sizeof(T) == 4 ? 8 : 4;

// blocks that share a box's levels in the ring kernels (a position's levels
// one after another in one thread left the chip waiting: FP64, 128 x 256 in 32
// boxes of half of 50 steps 33.6 -> 8.4 us; FP32, 512 x 1024 in 256 boxes of 33
// levels 130 us either way: a memory line per value of an east or west ring)
constexpr int kRingSplit = 8;

constexpr int kWaves = kTile / 64;         // partial sums per tile
constexpr int kRedMax = 1024;              // threads that add up a box's partial sums, at most
}  // namespace

// targets (and backgrounds at level 0) from the global FP64 trajectory, whose
// h is stored as h - h_ref
template <typename T>
__global__ __launch_bounds__(kTile) void k_from_global(Dom<T> D, const double* __restrict__ bg,
                                                       int64_t gplane, double* __restrict__ xb,
                                                       int n0) {
  const int n = n0 + blockIdx.y;
  const int2 wt = D.tiles[xcd_tile(blockIdx.x, gridDim.x)];
  const SubDev S = D.subs[wt.x];
  if (n >= S.nlev) return;
  const int m = wt.y * kTile + threadIdx.x;
  if (m >= S.ncell) return;
  const int r = m / S.nx, c = m - r * S.nx;
  int gcol = S.col0 + c;
  if (gcol >= D.nlon) gcol -= D.nlon;
  const int64_t g = int64_t(S.row0 + r) * D.nlon + gcol;
  const double* B = bg + int64_t(S.lev0 + n) * 3 * gplane;
  const int64_t plane = S.ncell;
  T* Tg = D.targ + S.traj_off + int64_t(n) * 3 * plane;
  Tg[m] = T(B[g]);
  Tg[plane + m] = T(B[gplane + g]);
  Tg[2 * plane + m] = T(B[2 * gplane + g]);
  if (n == 0) {
    double* xo = xb + S.ctrl_off;
    xo[m] = B[g] + double(D.h0);
    xo[plane + m] = B[gplane + g];
    xo[2 * plane + m] = B[2 * gplane + g];
  }
}

template <typename T>
__global__ void k_ring_from_global(Dom<T> D, const double* __restrict__ bg, int64_t gplane) {
  const SubDev S = D.subs[blockIdx.x];
  const int k = blockIdx.y * blockDim.x + threadIdx.x;
  if (k >= S.nring) return;
  const int src = D.hsrc[S.hmap_off + k];
  if (src < 0) return;
  const int64_t g = D.hgcell[S.hmap_off + k];
  const T sg = T(D.hsign[S.hmap_off + k]);
  for (int n = blockIdx.z; n < S.nlev; n += gridDim.z) {
    const double* B = bg + int64_t(S.lev0 + n) * 3 * gplane;
    T* R = D.ring + S.ring_off + int64_t(n) * 3 * S.nring;
    R[k] = T(B[g]);
    R[S.nring + k] = sg * T(B[gplane + g]);
    R[2 * S.nring + k] = sg * T(B[2 * gplane + g]);
  }
}

// every level (level < 0) or one local level of the boxes box_base, ...
template <typename T>
__global__ void k_ring_from_local(Dom<T> D, int box_base, int level) {
  const SubDev S = D.subs[box_base + blockIdx.x];
  const int k = blockIdx.y * blockDim.x + threadIdx.x;
  if (k >= S.nring) return;
  const int src = D.hsrc[S.hmap_off + k];
  if (src < 0) return;
  const SubDev P = D.subs[src];
  const int64_t off = D.hoff[S.hmap_off + k];
  const T sg = T(D.hsign[S.hmap_off + k]);
  const int n0 = level < 0 ? int(blockIdx.z) : level;
  const int n1 = level < 0 ? S.nlev : (level < S.nlev ? level + 1 : level);
  for (int n = n0; n < n1; n += gridDim.z) {   // same interval: same levels
    const T* Z = zlevel(D, P, n);
    T* R = D.ring + S.ring_off + int64_t(n) * 3 * S.nring;
    R[k] = Z[off];
    R[S.nring + k] = sg * Z[P.ncell + off];
    R[2 * S.nring + k] = sg * Z[2 * P.ncell + off];
  }
}

// Overlap targets of one local level (level >= 0) or of every level (level
// < 0) of the boxes of a tile range.  Lane i of every wave holds entry i of
// its box's neighbour list (at most 64).  Each cell first marks, once, the
// entries whose extended boxes contain it in space (one bit per entry), then
// at each level visits the entries marked by some lane of its wave and takes
// the mean and the spread of the marked neighbours that hold the level, in
// one pass with sums shifted by the first value (the values of one cell
// differ little between boxes, so the shifted sums lose nothing to
// cancellation).
//
// The cells of wide pieces come in the order of Dom::perm: in rows, almost every
// wave of a box touches its east and west overlaps and visits their boxes with
// a fraction of its lanes; in that order a wave's cells share their boxes and
// the waves without a covered cell have nothing to do.  (Narrow pieces stay in
// rows, and so do those that share no cell; the rule is where the order is made.)  The waves need
// nothing of each other: each adds up its own spreads, over the levels in
// order (or every split-th of them, see dd4dvar_ctx::jc_split).  FP32, 64
// pieces of 512 x 1024 in 4 intervals of 33 levels: 712 us in rows with a
// barrier per level (the vector units 80 % busy, 199 instructions per wave and
// level), 536 us now, held by the memory: 2 GB move, three times the values,
// since an overlap is 8 of the 32 cells of a line wide.
template <typename T>
__global__ __launch_bounds__(kTile) void k_targets_from_local(Dom<T> D, int level, int tile_base,
                                                              int split, double* __restrict__ jc) {
  const int w = tile_base + xcd_tile(blockIdx.x, gridDim.x);
  const int2 wt = D.tiles[w];
  const SubDev S = D.subs[wt.x];
  // levels n0, n0 + split, ...: one of the sums z = 0 .. split - 1 of the wave
  const int n0 = level < 0 ? int(blockIdx.y) : level, n1 = level < 0 ? S.nlev : level + 1;
  if (n0 >= S.nlev) return;                 // uniform over the block
  const int lane = threadIdx.x & 63;
  // the wave's cells in the exchange's order
  const int e = wt.y * kTile + threadIdx.x;
  const bool valid = e < S.ncell;
  int m = valid ? e : 0;
  if (S.perm0 >= 0) m = D.perm[S.perm0 + m];   // (uniform; else in rows)
  const int cov = valid ? int(D.cover[S.cell_off + m]) : 0;
  // where the wave's sum of these levels goes
  double* J = jc + (int64_t(w) * kWaves + (threadIdx.x >> 6)) * split + n0 % split;
  if (level >= 0 && D.tcount[S.lev0 + level] == 1 && !__any(cov > 1)) {
    // one level, none of the cells covered: done without the boxes' data
    // (FP32, 1024 x 2048 in 256 boxes and 4 intervals, two of three waves:
    // exchange over shared level slots 5.76 -> 5.46 ms)
    if (lane == 0 && n0 < split) *J = 0.0;
    return;
  }
  const int nq = S.nbr1 - S.nbr0;           // <= 64 (checked at set-up)
  // the lane's entry: first level, levels, first row and column, width,
  // height, cells, state offset
  int my_lev0 = 0, my_nlev = 0, my_row0 = 0, my_col0 = 0, my_nx = 0, my_ny = 0, my_ncell = 0;
  int64_t my_zoff = 0;
  if (lane < nq) {
    const SubDev& P = D.subs[D.nbr_idx[S.nbr0 + lane]];
    my_lev0 = P.lev0;
    my_nlev = P.nlev;
    my_row0 = P.row0;
    my_col0 = P.col0;
    my_nx = P.nx;
    my_ny = P.ny;
    my_ncell = P.ncell;
    my_zoff = P.zoff;
  }
  const int r = m / S.nx, c = m - r * S.nx;
  const int grow = S.row0 + r;
  int gcol = S.col0 + c;
  if (gcol >= D.nlon) gcol -= D.nlon;
  // at each level: boxes of the level's intervals, and the slot that the
  // lane's entry holds the level in (both loaded a turn ahead)
  auto slot = [&](int n) {
    const int pl = S.lev0 + n - my_lev0;
    return pl >= 0 && pl < my_nlev ? D.zslot[pl] : -1;
  };
  int tc_next = D.tcount[S.lev0 + n0], slot_next = slot(n0);
  // per lane: the entries whose boxes contain the cell (one level: of those that
  // hold it, for a launch per level marks anew: 140 boxes of 70 x 20 cells in 4
  // intervals, exchange over shared level slots 1.97 -> 1.78 ms); per wave: their
  // union
  uint64_t hits = 0, wave_hits = 0;
  for (uint64_t todo = __ballot(level < 0 ? lane < nq : slot_next >= 0); todo; todo &= todo - 1) {
    const int i = __builtin_ctzll(todo);
    const int rr = grow - __builtin_amdgcn_readlane(my_row0, i);
    int cc = gcol - __builtin_amdgcn_readlane(my_col0, i);
    if (cc < 0) cc += D.nlon;
    const bool hit = valid && rr >= 0 && rr < __builtin_amdgcn_readlane(my_ny, i) &&
                     cc < __builtin_amdgcn_readlane(my_nx, i);
    hits |= uint64_t(hit) << i;
    wave_hits |= uint64_t(__ballot(hit) != 0) << i;
  }
  const bool band = __any(cov > 1);         // a cell that other boxes of the interval cover
  const int64_t plane = S.ncell;
  double acc = 0.0;                         // the wave's sum over levels
  for (int n = n0; n < n1; n += split) {
    const int tc = tc_next, my_slot = slot_next;
    if (n + split < n1) {
      tc_next = D.tcount[S.lev0 + n + split];
      slot_next = slot(n + split);
    }
    if (tc == 1 && !band) continue;          // none of the cells is covered (uniform)
    const int K = cov * tc - 1;
    // entries that some lane of the wave hits and that hold the level, in
    // list order; the first kGather<T> of them are loaded together, before any
    // is used, then summed in list order
    const int64_t my_base = my_zoff + int64_t(my_slot) * 3 * my_ncell;
    const int my_lo = int(uint32_t(my_base)), my_hi = int(my_base >> 32);
    uint64_t rem = wave_hits & uint64_t(__ballot(my_slot >= 0));
    auto cell_of = [&](int i, int& pc) -> const T* {           // i: uniform
      const int rr = grow - __builtin_amdgcn_readlane(my_row0, i);
      int cc = gcol - __builtin_amdgcn_readlane(my_col0, i);
      if (cc < 0) cc += D.nlon;
      pc = __builtin_amdgcn_readlane(my_ncell, i);
      const int64_t base = int64_t(uint32_t(__builtin_amdgcn_readlane(my_lo, i))) |
                           (int64_t(__builtin_amdgcn_readlane(my_hi, i)) << 32);
      return D.traj + base + (rr * __builtin_amdgcn_readlane(my_nx, i) + cc);
    };
    T zh[kGather<T>], zu[kGather<T>], zv[kGather<T>];
    bool hk[kGather<T>];
#pragma unroll
    for (int k = 0; k < kGather<T>; ++k) {
      hk[k] = false;
      zh[k] = zu[k] = zv[k] = T(0);
      if (rem) {                                               // uniform
        const int i = __builtin_ctzll(rem);
        rem &= rem - 1;
        int pc;
        const T* Z = cell_of(i, pc);
        hk[k] = (hits >> i) & 1;
        if (hk[k]) {
          zh[k] = Z[0];
          zu[k] = Z[pc];
          zv[k] = Z[2 * int64_t(pc)];
        }
      }
    }
    double ch = 0, cu = 0, cv = 0;                 // shift: the first value
    double ah = 0, au = 0, av = 0, bh = 0, bu = 0, bv = 0;
    int cnt = 0;
    auto add = [&](double z0, double z1, double z2) {
      if (cnt == 0) {
        ch = z0;
        cu = z1;
        cv = z2;
      }
      const double dh = z0 - ch, du = z1 - cu, dv = z2 - cv;
      ah += dh;
      au += du;
      av += dv;
      bh += dh * dh;
      bu += du * du;
      bv += dv * dv;
      ++cnt;
    };
#pragma unroll
    for (int k = 0; k < kGather<T>; ++k)
      if (hk[k]) add(double(zh[k]), double(zu[k]), double(zv[k]));
    for (; rem; rem &= rem - 1) {                              // beyond kGather<T> entries
      const int i = __builtin_ctzll(rem);
      int pc;
      const T* Z = cell_of(i, pc);
      if (!((hits >> i) & 1)) continue;
      add(double(Z[0]), double(Z[pc]), double(Z[2 * int64_t(pc)]));
    }
    double jloc = 0.0;
    if (valid && K > 0 && cnt > 0) {
      const double inv = 1.0 / double(cnt);
      T* Tg = D.targ + S.traj_off + int64_t(n) * 3 * plane;
      Tg[m] = T(ch + ah * inv);
      Tg[plane + m] = T(cu + au * inv);
      Tg[2 * plane + m] = T(cv + av * inv);
      // sum over the neighbours of (value - mean)^2
      const double sh = bh - ah * ah * inv, su = bu - au * au * inv, sv = bv - av * av * inv;
      jloc = sh * D.isb2[0] + su * D.isb2[1] + sv * D.isb2[2];
    }
    // the level's sum, added in level order (as one launch per level adds
    // them), so both ways give the same bits; where one other box covers
    // every cell of the wave there is no spread to sum
    if (__any(jloc != 0.0)) acc += stencil::wave_sum(jloc);
  }
  if (lane == 0) *J = (n0 < split) ? acc : *J + acc;
}

// One workgroup per box: thread t adds its partial sums t, t + blockDim.x, ... in order
// (their loads are independent of one another), then the wave's tree, then
// the waves in order.  Sums that hold no level of their box are zero since
// the context's creation.  (One wave per box with an index division per sum:
// exchange of two FP64 boxes of 256 x 512 cells, 8192 sums each, 208 us, now 171;
// of four FP32 boxes of 1024 x 2048, 32768 sums each, 1.82 ms, now 1.57.)
__global__ __launch_bounds__(kRedMax) void k_reduce_jconst(const SubDev* __restrict__ subs,
                                                         const double* __restrict__ jc, int split,
                                                         double half_mu, double* __restrict__ jconst) {
  __shared__ double red[kRedMax / 64];
  const SubDev& S = subs[blockIdx.x];
  const double* p = jc + int64_t(S.tile0) * kWaves * split;
  const int n = S.ntile * kWaves * split;
  double acc = 0.0;
#pragma unroll 8
  for (int t = int(threadIdx.x); t < n; t += int(blockDim.x)) acc += p[t];
  acc = stencil::wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < int(blockDim.x >> 6); ++i) acc += red[i];
  jconst[blockIdx.x] = half_mu * acc;
}

template <typename T>
__global__ void k_gather(Dom<T> D, int nspace, int ntime, int level, int64_t ncell,
                         const int32_t* __restrict__ cptr, const int32_t* __restrict__ cpiece,
                         double* __restrict__ out) {
  const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= ncell) return;
  const int row = int(g / D.nlon), col = int(g - int64_t(row) * D.nlon);
  double ah = 0, au = 0, av = 0;
  int cnt = 0;
  for (int q = cptr[g]; q < cptr[g + 1]; ++q) {
    const int p = cpiece[q];
    for (int j = 0; j < ntime; ++j) {
      const SubDev S = D.subs[j * nspace + p];
      if (level < S.lev0 || level >= S.lev0 + S.nlev) continue;
      int cc = col - S.col0;
      if (cc < 0) cc += D.nlon;
      const T* Z = zlevel(D, S, level - S.lev0) + int64_t(row - S.row0) * S.nx + cc;
      ah += double(Z[0]);
      au += double(Z[S.ncell]);
      av += double(Z[2 * S.ncell]);
      ++cnt;
    }
  }
  const double inv = 1.0 / double(cnt);
  out[g] = ah * inv + double(D.h0);
  out[ncell + g] = au * inv;
  out[2 * ncell + g] = av * inv;
}

__global__ void k_add_href(double* traj, int64_t nlev, int64_t plane, double h0) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nlev * plane) return;
  const int64_t n = i / plane, g = i - n * plane;
  traj[n * 3 * plane + g] += h0;
}

__global__ void k_fill(double* p, int64_t n, double v) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---- launchers --------------------------------------------------------------
template <typename T>
void launch_from_global(const Dom<T>& D, const double* bg, int64_t gplane, double* xb, int nlev,
                        int ntiles, hipStream_t st) {
  constexpr int kGrid = 32768;             // levels per launch: within the grid's limit of 65535
  for (int n = 0; n < nlev; n += kGrid)
    hipLaunchKernelGGL(k_from_global<T>, dim3(ntiles, std::min(nlev - n, kGrid)), dim3(kTile), 0, st, D, bg,
                       gplane, xb, n);
}
// grid.y covers the largest ring; positions beyond a box's own ring exit
template <typename T>
void launch_ring_from_global(const Dom<T>& D, int nsub, int ring_blocks, const double* bg,
                             int64_t gplane, hipStream_t st) {
  hipLaunchKernelGGL(k_ring_from_global<T>, dim3(nsub, ring_blocks, kRingSplit), dim3(256), 0, st, D, bg,
                     gplane);
}
template <typename T>
void launch_ring_from_local(const Dom<T>& D, int box_base, int nbox, int ring_blocks, int level,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_ring_from_local<T>, dim3(nbox, ring_blocks, level < 0 ? kRingSplit : 1), dim3(256), 0,
                     st, D, box_base, level);
}
template <typename T>
void launch_targets_from_local(const Dom<T>& D, int level, int tile_base, int ntiles, int split,
                               double* jc, hipStream_t st) {
  hipLaunchKernelGGL(k_targets_from_local<T>, dim3(ntiles, level < 0 ? split : 1), dim3(kTile), 0, st, D,
                     level, tile_base, split, jc);
}
void launch_reduce_jconst(const SubDev* subs, int nsub, int ntiles, const double* jc, int split,
                          double half_mu, double* jconst, hipStream_t st) {
  // many sums in few boxes: a thread's own take longer than 16 waves' meeting
  const int threads = int64_t(ntiles) * kWaves * split > int64_t(2048) * nsub ? kRedMax : 256;
  hipLaunchKernelGGL(k_reduce_jconst, dim3(nsub), dim3(threads), 0, st, subs, jc, split, half_mu, jconst);
}
template <typename T>
void launch_gather(const Dom<T>& D, int nspace, int ntime, int level, int64_t ncell,
                   const int32_t* cptr, const int32_t* cpiece, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_gather<T>, dim3(unsigned((ncell + 255) / 256)), dim3(256), 0, st, D, nspace,
                     ntime, level, ncell, cptr, cpiece, out);
}
void launch_add_href(double* traj, int64_t nlev, int64_t plane, double h0, hipStream_t st) {
  const int64_t n = nlev * plane;
  hipLaunchKernelGGL(k_add_href, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, traj, nlev,
                     plane, h0);
}
void launch_fill(double* p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p, n, v);
}

#define DD4DVAR_INST(T)                                                                          \
  template void launch_from_global<T>(const Dom<T>&, const double*, int64_t, double*, int, int,  \
                                      hipStream_t);                                              \
  template void launch_ring_from_global<T>(const Dom<T>&, int, int, const double*, int64_t,      \
                                           hipStream_t);                                         \
  template void launch_ring_from_local<T>(const Dom<T>&, int, int, int, int, hipStream_t);       \
  template void launch_targets_from_local<T>(const Dom<T>&, int, int, int, int, double*,           \
                                             hipStream_t);                                 \
  template void launch_gather<T>(const Dom<T>&, int, int, int, int64_t, const int32_t*,          \
                                 const int32_t*, double*, hipStream_t);
DD4DVAR_INST(float)
DD4DVAR_INST(double)
#undef DD4DVAR_INST

}  // namespace dd4dvar
