// Temperature tables of the LTE line and of the source functions.
//
// The paper precomputes its level populations on a grid and interpolates
// them at run time ("Grid Precomputation"). Here, with LTE populations, the
// per-cell quantities that depend on temperature alone are
//   FL(T) = f_l(T) (1 - e^{-dE/T}),  f_l = g_l e^{-E_l/T} / Z(T)
//   J(T)  = T0 / expm1(T0 / T)       (Planck source in RJ kelvin)
//   JL(T) = T0 / expm1(dE / T)       (LTE line source; = J when dE = T0)
// so kappa_L = kL X n_H2 FL(T) / b(T). Each is evaluated exactly in FP64
// (partition sum over J = 0..j_max) at the nodes of a grid in u = log2(T)
// with kTabPerOctave intervals per octave over T in [2^kTabOct0, 2^kTabOct1),
// and stored per interval as the cubic Hermite polynomial
//   y(t) = y0 + t (m0 + t (c2 + t c3)),  t in [0, 1),
// built from the values and exact u-derivatives at both ends. Its
// interpolation error is below 1e-9 relative over the grid, far under FP32
// rounding. Temperatures outside the grid use the direct formulas.

#include "device_util.h"

namespace iris {

// Value and derivative d/du (u = log2 T) of FL, J and JL at T, in FP64.
struct TabNode {
  double fl, dfl, j, dj, jl, djl;
};

constexpr int kNodeLanes = 16;  // lanes of a node's partition sum (one DPP row)

// The node at u by a row of 16 lanes (r = lane in the row): the terms of the
// partition sum and the exponentials of the source functions are spread over
// the lanes; every lane returns the node.
__device__ __forceinline__ TabNode tab_node(const TabParams& tp, double u, int r) {
  const double T = exp2(u);
  const double rT = 1.0 / T;
  const double ln2 = 0.69314718055994530942;
  TabNode t;
  // Partition sum and its E-weighted sum, E_J = theta J(J+1), and the lower
  // level's own exponential.
  double Z = 0.0, ZE = 0.0, el = 0.0;
  for (int J = r; J <= tp.j_max; J += kNodeLanes) {
    const double E = tp.theta * J * (J + 1.0);
    const double e = exp(-E * rT);
    const double w = (2.0 * J + 1.0) * e;
    Z += w;
    ZE += w * E;
    if (J == tp.j_l) el = e;
  }
  Z = row_allsum64(Z);
  ZE = row_allsum64(ZE);
  el = row_allsum64(el);
  const double El = tp.theta * tp.j_l * (tp.j_l + 1.0);
  // e^{-dE/T} - 1, e^{T0/T} - 1 and e^{dE/T} - 1 in lanes 0, 1 and 2.
  const double x = tp.T0 * rT, y = tp.dE * rT;
  const double m1 = expm1(r == 0 ? -y : r == 1 ? x : y);
  const double stim = -__shfl(m1, 0, kNodeLanes);
  const double ex = __shfl(m1, 1, kNodeLanes), ey = __shfl(m1, 2, kNodeLanes);
  t.fl = tp.g_l * el * stim / Z;
  // d ln FL / dT = E_l/T^2 - <E>/T^2 - (dE/T^2) e^{-dE/T} / (1 - e^{-dE/T}),
  // the last quotient 1 / (e^{dE/T} - 1).
  const double dln = (El - ZE / Z - tp.dE / ey) * rT * rT;
  t.dfl = t.fl * dln * T * ln2;
  t.j = tp.T0 / ex;
  t.dj = t.j * t.j * (ex + 1.0) * ln2 * rT;
  t.jl = tp.T0 / ey;
  t.djl = tp.T0 * (ey + 1.0) * y * ln2 / (ey * ey);
  return t;
}

__device__ inline float4 hermite(double y0, double d0, double y1, double d1, double h) {
  const double m0 = d0 * h, m1 = d1 * h;
  const double c2 = 3.0 * (y1 - y0) - 2.0 * m0 - m1;
  const double c3 = 2.0 * (y0 - y1) + m0 + m1;
  return make_float4((float)y0, (float)m0, (float)c2, (float)c3);
}

// One interval per 32 lanes, a row of 16 for each end. Every call rebuilds the
// tables before its march, so this is a latency in front of all of them: with
// one interval per thread (eight workgroups, each thread 82 exponentials in a
// row) it took 12.3 us, spread like this 4.0 us.
__global__ __launch_bounds__(256) void pop_table_kernel(const TabParams tp, float4* tab) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = t / (2 * kNodeLanes);  // the grid is exactly kTabN intervals
  const int r = t % kNodeLanes, end = (t / kNodeLanes) & 1;
  const double h = 1.0 / kTabPerOctave;
  const TabNode a = tab_node(tp, kTabOct0 + (i + end) * h, r);
  TabNode b;  // the other end
  b.fl = __shfl_xor(a.fl, kNodeLanes, 64);
  b.dfl = __shfl_xor(a.dfl, kNodeLanes, 64);
  b.j = __shfl_xor(a.j, kNodeLanes, 64);
  b.dj = __shfl_xor(a.dj, kNodeLanes, 64);
  b.jl = __shfl_xor(a.jl, kNodeLanes, 64);
  b.djl = __shfl_xor(a.djl, kNodeLanes, 64);
  if (end == 0 && r < 3)
    tab[r * kTabN + i] = r == 0   ? hermite(a.fl, a.dfl, b.fl, b.dfl, h)
                         : r == 1 ? hermite(a.j, a.dj, b.j, b.dj, h)
                                  : hermite(a.jl, a.djl, b.jl, b.djl, h);
}

int launch_pop_table(const TabParams& tp, void* tab, void* stream) {
  static_assert(kTabN * 2 * kNodeLanes % 256 == 0, "whole workgroups");
  hipLaunchKernelGGL(pop_table_kernel, dim3(kTabN * 2 * kNodeLanes / 256), dim3(256), 0,
                     (hipStream_t)stream, tp, (float4*)tab);
  return (int)hipGetLastError();
}

}  // namespace iris
