// Adjoint of the DG Euler right-hand side with one thread per line, the
// scheme of kern_vjp.hip for N = 7 and 8, bitwise the same result; with STAGE
// the reverse LSERK45 stage around it too.
//
// A workgroup of three waves owns an element, wave d its lines along direction d: the neighbours' traces of Q and lifted traces
// of g, the transposed Lax-Friedrichs Jacobian of both ends of the line, and
// the transposed contraction and flux Jacobian at its nodes, all in one
// thread's registers; the three directions' parts are added in LDS in the
// order x, y, z.  LDS per node: Q (5), g (5) and the sum (5), whose place the
// neighbour traces had before: 41 and 61 KB an element, against 95 and 139 KB
// for a thread per node with the x-neighbours and the face adjoints beside
// them (24^3 p=6 581 -> 341 us, 24^3 p=7 1781 -> 779).  At N = 8 the 256
// registers a lane has with two waves on a SIMD do not hold it: 60 (product)
// and 69 (reverse stage) are spilled, 232 and 280 bytes of scratch a lane.

#include "dg_internal.h"
#include "stage_line.h"
#include "vjp_dev.h"

namespace {

using dgdev::along;
using dgdev::Block;
using dgdev::imin;
using dgdev::LineLds;
using dgdev::LineTables;

template <int N>
struct ALine {
  static_assert(N >= 7 && dg_line_elems(N) == 1, "one element per workgroup");
  static constexpr int N2 = N * N, N3 = N2 * N;
  static constexpr int SF = dgdev::LineSmem<N, 1>::SF;
  static constexpr int NT = 192;
  static constexpr int TD = 10 * N2;   // per direction [side][5][N2], g's traces, then Q's
  static constexpr int WORK = 5 * SF > 3 * TD ? 5 * SF : 3 * TD;
  static constexpr int size = 10 * SF + WORK;
};

// Orders this wave's LDS accesses (they execute in order; the compiler must
// keep them so).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// G = (dR/dQ)^T g, or with STAGE the reverse stage G += dt (dR/dQ)^T g in
// place and gres = a g (g is not gres).
template <int N, bool STAGE>
__global__ void __launch_bounds__(192) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_vjp_line(DGTables tb, const double* __restrict__ Q, const double* __restrict__ g, double* __restrict__ G,
           double* __restrict__ gres, double rka, double dt, DGOrder ord) {
  using V = ALine<N>;
  using L = LineLds<N>;
  constexpr int N2 = V::N2, N3 = V::N3, SF = V::SF;
  __shared__ __align__(16) double smem[V::size];
  double* sQ = smem;              // [5][SF]
  double* sG = smem + 5 * SF;     // [5][SF]
  double* sA = smem + 10 * SF;    // [5][SF]

  const Block blk = dgdev::block_of<1>(tb, ord, blockIdx.x, gridDim.x);
  const int e0 = blk.e0, nx = tb.nx, plane = tb.nx * tb.ny;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool px = wave == 0;
  const int64_t EN3 = (int64_t)tb.E * N3;
  const LineTables<N> tab{tb};
  double* sT = sA + wave * V::TD;

  // ---- loads: own Q and g (node pairs over the whole workgroup), then the
  //      wave's neighbour lines (as k_visc_line), Q's and, field by field as
  //      those are used up, g's
  constexpr int NU = (N3 + 1) / 2, PU = (5 * NU + V::NT - 1) / V::NT;
  const int64_t span = (int64_t)e0 * N3;
  const int cnt = blk.ne * N3;   // N3; known to the compiler, N = 8 spills a third more registers
  double2 oq[PU], og[PU];
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    const int64_t p = f * EN3 + span + imin(2 * (x - f * NU), cnt - 2);
    __builtin_memcpy(&oq[u], Q + p, 16);
    __builtin_memcpy(&og[u], g + p, 16);
  }
  const dgdev::PairLane<N, 1> pl(imin(lane, 2 * dgdev::LinePairs<N, 1>::LPF - 1));
  int64_t i0, i1 = 0;   // first nodes of the lane's neighbour lines
  int step = 1;
  if (px) {
    const int el = blk.x0 == 0 ? e0 + nx - 1 : e0 - 1;
    const int er = blk.x0 + 1 == nx ? e0 - blk.x0 : e0 + 1;
    const int pt = imin(lane, N2 - 1);
    i0 = (int64_t)el * N3 + pt * N;
    i1 = (int64_t)er * N3 + pt * N;
  } else {
    const int ey = blk.y, ez = blk.z;
    const bool y = wave == 1;
    const int em = y ? (ey == 0 ? e0 + (tb.ny - 1) * nx : e0 - nx) : (ez == 0 ? e0 + (tb.nz - 1) * plane : e0 - plane);
    const int ep = y ? (ey == tb.ny - 1 ? e0 - (tb.ny - 1) * nx : e0 + nx)
                     : (ez == tb.nz - 1 ? e0 - (tb.nz - 1) * plane : e0 + plane);
    step = y ? N : N2;
    i0 = (int64_t)(pl.side ? ep : em) * N3 + (y ? dgdev::tnode<N>(1, 0, pl.pt) : pl.pt);
  }
  double2 w[5][N];
  auto load_line = [&](const double* X, int f) {
    const double* b0 = X + f * EN3 + i0;
    if (px) {
      const double* b1 = X + f * EN3 + i1;
#pragma unroll
      for (int m = 0; m < N; m += 2) {
        if (m + 1 < N) {
          double2 v;
          __builtin_memcpy(&v, b0 + m, 16);
          w[f][m].x = v.x;
          w[f][m + 1 < N ? m + 1 : m].x = v.y;
          __builtin_memcpy(&v, b1 + m, 16);
          w[f][m].y = v.x;
          w[f][m + 1 < N ? m + 1 : m].y = v.y;
        } else {
          w[f][m].x = b0[m];
          w[f][m].y = b1[m];
        }
      }
    } else {
#pragma unroll
      for (int m = 0; m < N; ++m) __builtin_memcpy(&w[f][m], b0 + m * step, 16);
    }
  };
#pragma unroll
  for (int f = 0; f < 5; ++f) load_line(Q, f);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    const int n = f * SF + L::node(imin(2 * (x - f * NU), cnt - 2));
    sQ[n] = oq[u].x;
    sQ[n + 1] = oq[u].y;
    sG[n] = og[u].x;
    sG[n + 1] = og[u].y;
  }
  // traces of the lane's two lines (LIFT: lifted, l / w), the FMA chain of line_sum
  const int s0 = px ? 0 : pl.side, s1 = px ? 1 : pl.side;
  double q0[5], q1[5], g0[5], g1[5];
  auto trace = [&](int f, bool lift, double& t0, double& t1) {
    double v0 = 0.0, v1 = 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const double cm = lift ? tab.liftm(m) : tab.lm(m), cp = lift ? tab.liftp(m) : tab.lp(m);
      v0 = fma(s0 ? cm : cp, w[f][m].x, v0);
      v1 = fma(s1 ? cm : cp, w[f][m].y, v1);
    }
    asm volatile("" : "+v"(v0), "+v"(v1));
    t0 = v0;
    t1 = v1;
  };
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    trace(f, false, q0[f], q1[f]);
    load_line(g, f);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int f = 0; f < 5; ++f) trace(f, true, g0[f], g1[f]);
  // hands the lane's traces to the lines' threads
  auto give = [&](const double* t0, const double* t1) {
    if (px) {
      if (lane < N2) {
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          sT[f * N2 + lane] = t0[f];
          sT[(5 + f) * N2 + lane] = t1[f];
        }
      }
    } else if (lane < 2 * dgdev::LinePairs<N, 1>::LPF) {
      double* t = sT + pl.side * 5 * N2 + pl.pt;
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        t[f * N2] = t0[f];
        t[f * N2 + 1] = t1[f];
      }
    }
  };
  give(g0, g1);
  __syncthreads();

  // ---- the thread's line: line `lane`, (a, b) its tangential indices
  const bool act = lane < N2;
  const int ln = imin(lane, N2 - 1);
  const int b = ln / N, a = ln - b * N;
  int o[N];
#pragma unroll
  for (int m = 0; m < N; ++m)
    o[m] = px ? L::row(0, b, a) + m : wave == 1 ? L::row(0, b, m) + a : L::row(0, m, b) + a;

  // ---- end traces: the line's own, from LDS, and (after `give` and this) the
  //      neighbours' at sT[side][field][ln]
  auto own_ends = [&](const double* X, bool lift, double* tl, double* tr) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double x = 0.0, y = 0.0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const double v = X[f * SF + o[m]];
        x = fma(lift ? tab.liftm(m) : tab.lm(m), v, x);
        y = fma(lift ? tab.liftp(m) : tab.lp(m), v, y);
      }
      asm volatile("" : "+v"(x), "+v"(y));
      tl[f] = x;
      tr[f] = y;
    }
    wave_order();
  };
  const double sc = tb.sc[px ? 0 : wave == 1 ? 1 : 2];
  double tl[5], tr[5], fl[5], fr[5];   // f: adjoints of the two face fluxes
  own_ends(sG, true, tl, tr);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    fl[f] = sc * (tl[f] - sT[f * N2 + ln]);
    fr[f] = sc * (sT[(5 + f) * N2 + ln] - tr[f]);
    asm volatile("" : "+v"(fl[f]), "+v"(fr[f]));
  }
  wave_order();
  give(q0, q1);
  wave_order();
  own_ends(sQ, false, tl, tr);

  // ---- adjoints hl, hr of the line's end traces (one side at a time: the
  //      terms of both do not fit the registers), then v[f][m], the flux
  //      Jacobian transpose at its nodes
  double hl[5], hr[5], v[5][N];
  along(wave, [&](auto dir) {
    constexpr int D = decltype(dir)::d;
    double nb[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) nb[f] = sT[f * N2 + ln];
    dgdev::lf_vjp_d<D>(nb, tl, tb.gamma, tb.gm1, fl, false, hl);
#pragma unroll
    for (int f = 0; f < 5; ++f) asm volatile("" : "+v"(hl[f]));
#pragma unroll
    for (int f = 0; f < 5; ++f) nb[f] = sT[(5 + f) * N2 + ln];
    dgdev::lf_vjp_d<D>(tr, nb, tb.gamma, tb.gm1, fr, true, hr);
#pragma unroll
    for (int f = 0; f < 5; ++f) asm volatile("" : "+v"(hr[f]));
    // the transposed contraction takes each field's line, the flux Jacobian
    // transpose each node's values, in place
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double gg[N];
#pragma unroll
      for (int m = 0; m < N; ++m) gg[m] = sG[f * SF + o[m]];
#pragma unroll
      for (int m = 0; m < N; ++m) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) s = fma(tab.dh(i, m), gg[i], s);
        v[f][m] = sc * s;
      }
#pragma unroll
      for (int m = 0; m < N; ++m) asm volatile("" : "+v"(v[f][m]));
    }
#pragma unroll
    for (int m = 0; m < N; ++m) {
      double gF[5], q[5], out[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        gF[f] = v[f][m];
        q[f] = sQ[f * SF + o[m]];
        out[f] = 0.0;
      }
      dgdev::flux_vjp<D>(q, gF, tb.gm1, out);
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        v[f][m] = out[f];
        asm volatile("" : "+v"(v[f][m]));
      }
    }
  });
  __syncthreads();   // last reads of the neighbour traces: the sum takes their place
  auto add = [&](bool first) {
    if (!act) return;
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double r[N];
#pragma unroll
      for (int m = 0; m < N; ++m) r[m] = first ? 0.0 : sA[f * SF + o[m]];
#pragma unroll
      for (int m = 0; m < N; ++m) {
        r[m] += v[f][m];
        r[m] += tab.lp(m) * hr[f] + tab.lm(m) * hl[f];
        sA[f * SF + o[m]] = r[m];
      }
    }
  };
  if (wave == 0) add(true);
  __syncthreads();
  if (wave == 1) add(false);
  __syncthreads();
  // what the output updates in place, read before the last sum
  double2 old[STAGE ? PU : 1];
  if constexpr (STAGE) {
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
      __builtin_memcpy(&old[u], G + f * EN3 + span + imin(2 * (x - f * NU), cnt - 2), 16);
    }
  }
  if (wave == 2) add(false);
  __syncthreads();   // (also: a pair taken twice has been read before it is written)
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    const int n = imin(2 * (x - f * NU), cnt - 2);
    const int64_t p = f * EN3 + span + n;
    const int l = f * SF + L::node(n);
    double2 r = {sA[l], sA[l + 1]};
    if constexpr (STAGE) {
      const double2 z = {rka * sG[l], rka * sG[l + 1]};
      r.x = fma(dt, r.x, old[u].x);
      r.y = fma(dt, r.y, old[u].y);
      __builtin_memcpy(gres + p, &z, 16);
    }
    __builtin_memcpy(G + p, &r, 16);
  }
}

template <int N>
int launch_n(const dg_ctx* c, const double* Q, const double* g, double* G, double* gres, double a, double dt) {
  unsigned grid;
  const DGOrder ord = dg_order(c, 1, &grid, true, 16);
  if (gres)
    hipLaunchKernelGGL((k_vjp_line<N, true>), dim3(grid), dim3(192), 0, c->stream, c->tab, Q, g, G, gres, a, dt, ord);
  else
    hipLaunchKernelGGL((k_vjp_line<N, false>), dim3(grid), dim3(192), 0, c->stream, c->tab, Q, g, G, gres, a, dt, ord);
  return (int)hipGetLastError();
}

}  // namespace

int dg_launch_vjp_line(const dg_ctx* c, const double* Q, const double* g, double* G, double* gres, double a,
                       double dt) {
  return c->N == 7   ? launch_n<7>(c, Q, g, G, gres, a, dt)
         : c->N == 8 ? launch_n<8>(c, Q, g, G, gres, a, dt)
                     : (int)hipErrorInvalidValue;
}
