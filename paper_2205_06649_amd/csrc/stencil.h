// Stencil helpers shared by the step kernels (sweep.hip, tlm.hip), the block
// sweeps (blk.hip) and the per-box kernels (box.hip): neighbour indexing of a
// box cell (inside, wrapped, or a frozen ring position), branch-free loads,
// the FP64 arithmetic that step kernels and block sweeps have in common, and
// sums over a wave and a workgroup.
#pragma once

#include "kernels.h"

namespace dd4dvar {
namespace stencil {


template <typename T>
struct V3 {
  T h, u, v;
};

template <typename T>
__device__ __forceinline__ V3<T> ld_box(const T* Z, int64_t plane, int64_t idx, T sgn) {
  return {Z[idx], sgn * Z[plane + idx], sgn * Z[2 * plane + idx]};
}

template <typename T>
__device__ __forceinline__ V3<T> ld_ring(const T* R, int nring, int k) {
  return {R[k], R[nring + k], R[2 * nring + k]};
}

// Neighbour positions of box cell (r, c): index into the box (>= 0) or ring
// position (encoded as -1 - k), plus the sign applied to u, v.  Computed
// with selects only, so that every neighbour load is issued unconditionally
// (branches around loads make the compiler wait for each one in turn).
struct NbrIdx {
  int e, w, n, s;
  int sn, ss;       // -1 across a pole
};

__device__ __forceinline__ NbrIdx nbr_index(const SubDev& S, int r, int c, int half) {
  NbrIdx q;
  const int m = r * S.nx + c;
  int ch = c + half;                       // column across the pole (span boxes)
  ch = ch >= S.nx ? ch - S.nx : ch;
  const bool e_in = c + 1 < S.nx, w_in = c > 0, n_in = r + 1 < S.ny, s_in = r > 0;
  q.e = e_in ? m + 1 : (S.span ? m + 1 - S.nx : -1 - (2 * S.nx + S.ny + r));
  q.w = w_in ? m - 1 : (S.span ? m - 1 + S.nx : -1 - (2 * S.nx + r));
  q.n = n_in ? m + S.nx : (S.pole_n ? r * S.nx + ch : -1 - (S.nx + c));
  q.s = s_in ? m - S.nx : (S.pole_s ? ch : -1 - c);
  q.sn = (!n_in && S.pole_n) ? -1 : 1;
  q.ss = (!s_in && S.pole_s) ? -1 : 1;
  return q;
}

template <typename T>
__device__ __forceinline__ V3<T> ld_nbr(const T* Z, const T* R, int64_t plane, int nring,
                                        int idx, int sgn) {
  const bool in = idx >= 0;
  const T* p = in ? Z + idx : R + (-1 - idx);
  const int64_t st = in ? plane : int64_t(nring);
  const T sg = T(in ? sgn : 1);
  return {p[0], sg * p[st], sg * p[2 * st]};
}

// Adjoint of level n+1 at a neighbour, zero when the neighbour is a frozen
// ring position (its increment is not part of the local model).  The load
// is unconditional (from the cell itself when the neighbour is frozen).
template <typename T>
__device__ __forceinline__ V3<T> ld_lam(const T* L1, int64_t plane, int idx, int m) {
  const bool in = idx >= 0;
  const int i = in ? idx : m;
  const T h = L1[i], u = L1[plane + i], v = L1[2 * plane + i];
  return {in ? h : T(0), in ? u : T(0), in ? v : T(0)};
}

// ---- FP64 arithmetic shared by the step kernels and the block sweeps, whose
// results are equal bit for bit: contracted by hand (the FP64 sources are
// compiled without contraction), with factors that several terms share taken
// out.  Products that cancel in a steady state (h u of the east and the west)
// are rounded alike.

// The increment F(Z^n) of a cell (discrete U, V, H of Sec. 7 with p = q = 1,
// alpha = 0) from its five-point neighbourhood; cN, cS the cosines of the
// rows to the north and south.
__device__ __forceinline__ V3<double> swe_increment(const V3<double>& C, const V3<double>& E,
                                                    const V3<double>& W, const V3<double>& N,
                                                    const V3<double>& Sv, double a1, double a2,
                                                    double a3, double cf, double ct, double cN,
                                                    double cS, double st, double stg, double h0) {
  const double cor = fma(ct, C.u, cf), ua = a1 * C.u, va = st * C.v;
  const double due = E.u - W.u, vn = N.v * cN, vs = Sv.v * cS;
  const double U = fma(cor, C.v, -fma(a2, E.h - W.h, fma(va, N.u - Sv.u, ua * due)));
  const double V = -fma(cor, C.u, fma(stg, N.h - Sv.h, fma(va, N.v - Sv.v, ua * (E.v - W.v))));
  const double x = fma(h0, due, E.h * E.u - W.h * W.u);
  const double y = fma(h0, vn - vs, N.h * vn - Sv.h * vs);
  return {-fma(a3, y, a1 * x), U, V};
}

// Its tangent linear at the same neighbourhood applied to dC .. dS.
__device__ __forceinline__ V3<double> swe_tangent(
    const V3<double>& C, const V3<double>& E, const V3<double>& W, const V3<double>& N,
    const V3<double>& Sv, const V3<double>& dC, const V3<double>& dE, const V3<double>& dW,
    const V3<double>& dN, const V3<double>& dS, double a1, double a2, double a3, double cf,
    double ct, double cN, double cS, double st, double stg, double h0) {
  const double cor = fma(ct, C.u, cf), dcor = ct * dC.u;
  const double ue = fma(dC.u, E.u - W.u, C.u * (dE.u - dW.u));
  const double un = fma(dC.v, N.u - Sv.u, C.v * (dN.u - dS.u));
  const double ve = fma(dC.u, E.v - W.v, C.u * (dE.v - dW.v));
  const double vn = fma(dC.v, N.v - Sv.v, C.v * (dN.v - dS.v));
  const double dU = fma(dcor, C.v, cor * dC.v) - fma(a2, dE.h - dW.h, fma(st, un, a1 * ue));
  const double dV = -(fma(dcor, C.u, cor * dC.u) + fma(stg, dN.h - dS.h, fma(st, vn, a1 * ve)));
  const double x = fma(h0 + E.h, dE.u, dE.h * E.u) - fma(h0 + W.h, dW.u, dW.h * W.u);
  const double y = fma(h0 + N.h, dN.v, dN.h * N.v) * cN - fma(h0 + Sv.h, dS.v, dS.h * Sv.v) * cS;
  return {-fma(a3, y, a1 * x), dU, dV};
}

// J_F(Z^n)^T lambda^{n+1} at a cell, in two steps that share few values: its
// own terms and those of the east and west neighbours, then those of the
// north and south ones, whose increments read it (east k sees it as west,
// north k as south, across a pole the north k sees it as north with u, v
// negated).  l0 .. kS: lambda^{n+1} at the cell and its neighbours (zero at
// frozen ring positions); a3n, a3s, the a3 of the rows of the north and south
// readers; sn, ss the across-pole signs.
__device__ __forceinline__ V3<double> swe_adjoint_ew(const V3<double>& C, const V3<double>& E,
                                                     const V3<double>& W, const V3<double>& N,
                                                     const V3<double>& Sv, const V3<double>& l0,
                                                     const V3<double>& kE, const V3<double>& kW,
                                                     double a1, double a2, double cf, double ct,
                                                     double st, double h0) {
  const double cor = fma(ct, C.u, cf), dkh = kE.h - kW.h;
  double au = fma(l0.u, fma(-a1, E.u - W.u, ct * C.v), -(l0.v * fma(a1, E.v - W.v, fma(ct, C.u, cor))));
  double av = fma(l0.u, fma(-st, N.u - Sv.u, cor), -(l0.v * (st * (N.v - Sv.v))));
  au = fma(a1, fma(h0 + C.h, dkh, fma(kE.u, E.u, -(kW.u * W.u))), au);
  av = fma(a1, fma(kE.v, E.u, -(kW.v * W.u)), av);
  return {fma(a2, kE.u - kW.u, (a1 * C.u) * dkh), au, av};
}
__device__ __forceinline__ V3<double> swe_adjoint_ns(const V3<double>& a, const V3<double>& C,
                                                     const V3<double>& N, const V3<double>& Sv,
                                                     const V3<double>& kN, const V3<double>& kS,
                                                     double c, double a3n, double a3s, double sn,
                                                     double ss, double st, double stg, double h0) {
  const double vkn = sn * N.v, vks = ss * Sv.v;          // raw v at the neighbours
  const double q = fma(kN.h, a3n, -(kS.h * a3s)) * c;
  const double au = fma(st, fma(kN.u, vkn, -(kS.u * vks)), a.u);
  const double av = fma(h0 + C.h, q, fma(st, fma(kN.v, vkn, -(kS.v * vks)), a.v));
  const double ah = fma(C.v, q, fma(stg, fma(sn, kN.v, -(ss * kS.v)), a.h));
  return {ah, au, av};
}

// Overlap misfit of a cell that K other boxes cover: forcing K mu e / sigma_b^2
// added to f, its term of J to jloc (cost false: the forcing alone).  mis: mu
// / sigma_b^2.
__device__ __forceinline__ void overlap_terms(const V3<double>& e, int K, const double* mis, bool cost,
                                              double* f, double& jloc) {
  const double k = double(K);
  const double gh = (mis[0] * k) * e.h, gu = (mis[1] * k) * e.u, gv = (mis[2] * k) * e.v;
  f[0] += gh;
  f[1] += gu;
  f[2] += gv;
  if (cost) jloc = fma(0.5, fma(gv, e.v, fma(gu, e.u, gh * e.h)), jloc);
}

// Sum of a wave's 64 values in every lane, in the order of block_sum's
// shuffle tree (lanes 32, 16, 8, 4, 2, 1 apart; a sum of two does not depend on
// their order, so that exchanging partners gives both lanes the tree's
// value).  By lane permutations of the vector unit: the shuffles go through
// the LDS crossbar, six dependent round trips of it.
template <int CTRL>
__device__ __forceinline__ double lane_exchange(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(b)), CTRL, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(b >> 32)), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, uint64_t(hi) << 32 | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  auto half = [](double x, auto swap) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const auto lo = swap(uint32_t(b)), hi = swap(uint32_t(b >> 32));
    return __builtin_bit_cast(double, uint64_t(hi[0]) << 32 | lo[0]) +
           __builtin_bit_cast(double, uint64_t(hi[1]) << 32 | lo[1]);
  };
  v = half(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
  v = half(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
  v += lane_exchange<0x128>(v);            // 8 apart: rotation within 16 lanes
  v += lane_exchange<0x124>(v);            // 4
  v += lane_exchange<0x4e>(v);             // 2: quad_perm [2,3,0,1]
  v += lane_exchange<0xb1>(v);             // 1: quad_perm [1,0,3,2]
  return v;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < int(blockDim.x >> 6); ++i) r += sh[i];
  return r;
}


}  // namespace stencil
}  // namespace dd4dvar
