// Viscous (Navier-Stokes) stage with one thread per line, the scheme of
// kern_visc.hip (BR1) for degrees 1..7:
//   k_visc_line    Q -> R and the face traces of the viscous flux: the
//                  inviscid rate of the standard form (with RATE; else R
//                  holds one already), the gradients, the viscous flux, and
//                  the element's own part of its weak derivative, added to R;
//   k_visc_update  the neighbours' part, the lift of half their traces, added
//                  to R (MODE 0) or folded with R into the LSERK45 update of
//                  Q and res in place (MODE 1, MODE 2 for the first stage).
// The weak derivative is linear in the traces, so what an element needs of
// its neighbours' viscous fluxes is 4 values per face point: 24 N^2 doubles
// an element change hands instead of 12 N^3 that six neighbours read whole.
// A node and stage moves 40 + 40 + 192 / N bytes in the first launch (Q, R,
// traces) and 200 + 192 / N in the second (traces, R, Q, res; Q, res):
// 357 at N = 5.
//
// k_visc_line: a workgroup of three waves owns a block of elements of one
// x-row, wave d its lines along direction d.  The three directions' loads,
// traces, fluxes and contractions run side by side; their sums are added to
// the shared nodal values in the order x, y, z, so the inviscid rate is that
// of the inviscid kernels bit for bit.  48^3 p=4: 983 us, and 632 for
// k_visc_update (5.2 TB/s), against 1130 + 990 with a node per thread and the
// nodal flux between them.  LDS per node: the state (5), the rate
// (5), and in the place that the neighbour traces had before, the viscous
// stress and heat flux (9): 38 KB a block at N = 4 and 5, four blocks or
// twelve waves a CU.

#include "dg_internal.h"
#include "stage_line.h"

namespace {

using dgdev::add_line;
using dgdev::along;
using dgdev::Block;
using dgdev::Dir;
using dgdev::imin;
using dgdev::LineLds;
using dgdev::LineTables;

template <int N>
struct VLine {
  static constexpr int EPB = dg_line_elems(N);
  static constexpr int N2 = N * N, N3 = N2 * N, FP = EPB * N2;
  static constexpr int SF = dgdev::LineSmem<N, EPB>::SF;
  static constexpr int NT = 192;
  // neighbour traces: per direction [side][5 conserved, 4 primitive][FP]
  static constexpr int TD = 18 * FP;
  static constexpr int WORK = 14 * SF > 3 * TD ? 14 * SF : 3 * TD;
  static constexpr int size = 5 * SF + WORK;
};

// (u, v, w, T) of a conserved state, T = p / rho with Eq. (3)'s pressure.
__device__ __forceinline__ void primitive(const double* q, double gm1, double* P) {
  const double r = dgdev::recip(q[0]);
  P[0] = q[1] * r;
  P[1] = q[2] * r;
  P[2] = q[3] * r;
  const double ke = 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) * r;
  P[3] = gm1 * (q[4] - ke) * r;
}

// Adds a node to a line's conserved trace (weight c, the FMA chain of
// chunk_trace) and primitive trace.
template <bool CONS>
__device__ __forceinline__ void add_trace(const double* q, double c, double gm1, double* cons, double* prim) {
  double p[4];
  primitive(q, gm1, p);
  if (CONS) {
#pragma unroll
    for (int f = 0; f < 5; ++f) cons[f] = fma(c, q[f], cons[f]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) prim[k] = fma(c, p[k], prim[k]);
}

// Place of stress tau_kd among the nine nodal values xx yy zz xy xz yz qx qy qz.
__device__ __forceinline__ constexpr int stress(int k, int d) { return k == d ? k : k + d + 2; }

template <int N, bool RATE>
__global__ void __launch_bounds__(192) __attribute__((amdgpu_waves_per_eu(N <= 6 ? 3 : 2, 8)))
k_visc_line(DGTables tb, const double* __restrict__ Q, double* __restrict__ T, double* __restrict__ R, double mu,
            double kappa, DGOrder ord) {
  using V = VLine<N>;
  using L = LineLds<N>;
  constexpr int EPB = V::EPB, N2 = V::N2, N3 = V::N3, FP = V::FP, SF = V::SF;
  __shared__ __align__(16) double smem[V::size];
  double* sS = smem;             // [5][SF] state
  double* sA = smem + 5 * SF;    // [5][SF] rate
  double* sG = sA + 5 * SF;      // [9][SF] stress and heat flux

  const Block blk = dgdev::block_of<EPB>(tb, ord, blockIdx.x, gridDim.x);
  const int e0 = blk.e0, ne = blk.ne, nx = tb.nx, plane = tb.nx * tb.ny;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t EN3 = (int64_t)tb.E * N3;
  const LineTables<N> tab{tb};
  const double g1 = tb.gm1;
  double* sT = sA + wave * V::TD;   // this direction's neighbour traces

  // ---- loads: own state (node pairs of the contiguous per-field spans over
  //      the whole workgroup), then the wave's neighbour lines
  constexpr int NU = (EPB * N3 + 1) / 2, PU = (5 * NU + V::NT - 1) / V::NT;
  const int64_t span = (int64_t)e0 * N3;
  const int cnt = ne * N3;
  double2 own[PU], rin[RATE ? 1 : PU];
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    const int64_t g = f * EN3 + span + imin(2 * (x - f * NU), cnt - 2);
    __builtin_memcpy(&own[u], Q + g, 16);
    if constexpr (!RATE) __builtin_memcpy(&rin[u], R + g, 16);
  }
  // y, z: pairs of face points as PairLane, both points of a pair in x and y.
  // x: EPB > 1 the outer neighbours' lines, lanes [0, N^2) the left one's,
  // [N^2, 2 N^2) the right one's, in x; EPB = 1 left in x, right in y.
  const dgdev::PairLane<N, EPB> pl(imin(lane, 2 * dgdev::LinePairs<N, EPB>::LPF - 1));
  const int xside = lane >= N2;
  const bool px = wave == 0;
  const double *b0, *b1;
  int step = 1;
  if (px) {
    const int el = blk.x0 == 0 ? e0 + nx - 1 : e0 - 1;
    const int er = blk.x0 + ne == nx ? e0 - blk.x0 : e0 + ne;
    const int pt = imin(EPB == 1 ? lane : lane - xside * N2, N2 - 1);
    b0 = Q + (int64_t)(EPB > 1 && xside ? er : el) * N3 + pt * N;
    b1 = Q + (int64_t)er * N3 + pt * N;
  } else {
    const int ey = blk.y, ez = blk.z;
    const bool y = wave == 1;
    const int em = y ? (ey == 0 ? e0 + (tb.ny - 1) * nx : e0 - nx) : (ez == 0 ? e0 + (tb.nz - 1) * plane : e0 - plane);
    const int ep = y ? (ey == tb.ny - 1 ? e0 - (tb.ny - 1) * nx : e0 + nx)
                     : (ez == tb.nz - 1 ? e0 - (tb.nz - 1) * plane : e0 + plane);
    step = y ? N : N2;
    b0 = b1 = Q + (int64_t)(pl.side ? ep : em) * N3 + imin(pl.fel, ne - 1) * N3 +
              (y ? dgdev::tnode<N>(1, 0, pl.pt) : pl.pt);
  }
  // two nodes of the lines at a time; at N = 6 and 8 the registers hold two
  // such parts in flight beside the traces, else all
  constexpr int PARTS = (N + 1) / 2, AHEAD = N == 6 || N == 8 ? 2 : PARTS;
  double2 w[5][N];
  auto load_part = [&](int c) {
    const int m = 2 * c;
    if (px) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        if (m + 1 < N) {
          double2 v;
          __builtin_memcpy(&v, b0 + f * EN3 + m, 16);
          w[f][m].x = v.x;
          w[f][m + 1 < N ? m + 1 : m].x = v.y;
          if (EPB == 1) {   // (else the second points are not used)
            __builtin_memcpy(&v, b1 + f * EN3 + m, 16);
            w[f][m].y = v.x;
            w[f][m + 1 < N ? m + 1 : m].y = v.y;
          }
        } else {
          w[f][m].x = b0[f * EN3 + m];
          if (EPB == 1) w[f][m].y = b1[f * EN3 + m];
        }
      }
    } else {
#pragma unroll
      for (int h = m; h < N && h < m + 2; ++h)
#pragma unroll
        for (int f = 0; f < 5; ++f) __builtin_memcpy(&w[f][h], b0 + f * EN3 + h * step, 16);
    }
  };
#pragma unroll
  for (int c = 0; c < AHEAD; ++c) load_part(c);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    double* s = sS + f * SF + L::node(imin(2 * (x - f * NU), cnt - 2));
    s[0] = own[u].x;
    s[1] = own[u].y;
  }
  // ---- the neighbours' traces
  {
    double t0[9], t1[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) t0[c] = t1[c] = 0.0;
    const int s0 = px ? (EPB > 1 ? xside : 0) : pl.side, s1 = px ? (EPB > 1 ? xside : 1) : pl.side;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const double v0[5] = {w[0][m].x, w[1][m].x, w[2][m].x, w[3][m].x, w[4][m].x};
      const double v1[5] = {w[0][m].y, w[1][m].y, w[2][m].y, w[3][m].y, w[4][m].y};
      add_trace<RATE>(v0, s0 ? tab.lm(m) : tab.lp(m), g1, t0, t0 + 5);
      add_trace<RATE>(v1, s1 ? tab.lm(m) : tab.lp(m), g1, t1, t1 + 5);
#pragma unroll
      for (int c = RATE ? 0 : 5; c < 9; ++c) asm volatile("" : "+v"(t0[c]), "+v"(t1[c]));
      if (m % 2 && m / 2 + AHEAD < PARTS) load_part(m / 2 + AHEAD);
    }
    if (px) {
      if (EPB > 1) {
        if (lane < 2 * N2) {
          double* t = sT + (xside ? 9 * FP + (ne - 1) * N2 + lane - N2 : lane);
#pragma unroll
          for (int c = RATE ? 0 : 5; c < 9; ++c) t[c * FP] = t0[c];
        }
      } else if (lane < N2) {
#pragma unroll
        for (int c = RATE ? 0 : 5; c < 9; ++c) {
          sT[c * FP + lane] = t0[c];
          sT[(9 + c) * FP + lane] = t1[c];
        }
      }
    } else if (lane < 2 * dgdev::LinePairs<N, EPB>::LPF) {
      double* t = sT + pl.side * 9 * FP + pl.fel * N2 + pl.pt;
#pragma unroll
      for (int c = RATE ? 0 : 5; c < 9; ++c) {
        t[c * FP] = t0[c];
        t[c * FP + 1] = t1[c];
      }
    }
  }
  __syncthreads();

  // ---- the thread's line: line `lane` = (el, pt), pt = (a, b) tangential
  const bool act = lane < FP;
  const int ln = imin(lane, FP - 1);
  const int el = ln / N2, pt = ln - el * N2;
  const int b = pt / N, a = pt - b * N;
  int o[N];   // LDS places of the line's nodes
#pragma unroll
  for (int m = 0; m < N; ++m)
    o[m] = wave == 0 ? L::row(el, b, a) + m : wave == 1 ? L::row(el, b, m) + a : L::row(el, m, b) + a;

  // ---- phase 1: the line's face terms and inviscid sums.  v holds what the
  //      wave adds next to the nodal values: the inviscid sums, then the
  //      gradients, then the viscous rate (one array: in arrays of their own
  //      they would all be held through every wave's turn).
  double v[5][N], hm[4], hp[4];
  along(wave, [&](auto dir) {
    constexpr int D = decltype(dir)::d;
    // own end traces, primitive and conserved, each from the line read from
    // LDS for it (held, the line and the flux's terms do not fit the registers)
    double pl4[4] = {0.0, 0.0, 0.0, 0.0}, pr4[4] = {0.0, 0.0, 0.0, 0.0}, tl[5], tr[5];
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const double q[5] = {sS[o[m]], sS[SF + o[m]], sS[2 * SF + o[m]], sS[3 * SF + o[m]], sS[4 * SF + o[m]]};
      double p[4];
      primitive(q, g1, p);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pl4[k] = fma(tab.lm(m), p[k], pl4[k]);
        pr4[k] = fma(tab.lp(m), p[k], pr4[k]);
        asm volatile("" : "+v"(pl4[k]), "+v"(pr4[k]));
      }
    }
    if constexpr (RATE) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        double x = 0.0, y = 0.0;
#pragma unroll
        for (int m = 0; m < N; ++m) {
          const double q = sS[f * SF + o[m]];
          x = fma(tab.lm(m), q, x);
          y = fma(tab.lp(m), q, y);
        }
        asm volatile("" : "+v"(x), "+v"(y));
        tl[f] = x;
        tr[f] = y;
      }
    }
    if (D == 0 && EPB > 1) {
      // neighbours inside the block take this line's end traces
      const bool give_r = act && el + 1 < ne, give_l = act && el > 0 && el < ne;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (give_r) sT[(5 + k) * FP + ln + N2] = pr4[k];
        if (give_l) sT[(14 + k) * FP + ln - N2] = pl4[k];
      }
      if constexpr (RATE) {
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          if (give_r) sT[f * FP + ln + N2] = tr[f];
          if (give_l) sT[(9 + f) * FP + ln - N2] = tl[f];
        }
      }
      // (the wave's own LDS accesses stay in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      hm[k] = 0.5 * (pl4[k] + sT[(5 + k) * FP + ln]);
      hp[k] = 0.5 * (pr4[k] + sT[(14 + k) * FP + ln]);
      asm volatile("" : "+v"(hm[k]), "+v"(hp[k]));
    }
    if constexpr (RATE) {
      double fl[5], fr[5], nbr[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) nbr[f] = sT[f * FP + ln];
      dgdev::lf_flux_d<D>(nbr, tl, tb.gamma, g1, fl);
#pragma unroll
      for (int f = 0; f < 5; ++f) asm volatile("" : "+v"(fl[f]));
#pragma unroll
      for (int f = 0; f < 5; ++f) nbr[f] = sT[(9 + f) * FP + ln];
      dgdev::lf_flux_d<D>(tr, nbr, tb.gamma, g1, fr);
#pragma unroll
      for (int f = 0; f < 5; ++f) asm volatile("" : "+v"(fr[f]));
#pragma unroll
      for (int f = 0; f < 5; ++f)
#pragma unroll
        for (int m = 0; m < N; ++m) v[f][m] = sS[f * SF + o[m]];
      // the inviscid sums, as EulerLine::rate; each field's take the place of
      // its line (held in order: interleaved, they do not fit the registers)
      double pr[N], ud[N];
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const double rinv = dgdev::recip(v[0][c]);
        pr[c] = g1 * (v[4][c] - 0.5 * (v[1][c] * v[1][c] + v[2][c] * v[2][c] + v[3][c] * v[3][c]) * rinv);
        ud[c] = v[1 + D][c] * rinv;
        asm volatile("" : "+v"(pr[c]), "+v"(ud[c]));
      }
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        double F[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
          if (f == 0) F[c] = v[1 + D][c];
          else if (f == 4) F[c] = (v[4][c] + pr[c]) * ud[c];
          else F[c] = v[f][c] * ud[c] + (D == f - 1 ? pr[c] : 0.0);
        }
#pragma unroll
        for (int m = 0; m < N; ++m) {
          double x = 0.0;
#pragma unroll
          for (int c = 0; c < N; ++c) x = fma(tab.dh(m, c), F[c], x);
          x = fma(tab.liftm(m), fl[f], x);
          v[f][m] = fma(-tab.liftp(m), fr[f], x);
        }
#pragma unroll
        for (int m = 0; m < N; ++m) asm volatile("" : "+v"(v[f][m]));
      }
    }
  });
  __syncthreads();   // last reads of the neighbour traces: rate and stress take their place
  if constexpr (!RATE) {
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
      double* r = sA + f * SF + L::node(imin(2 * (x - f * NU), cnt - 2));
      r[0] = rin[u].x;
      r[1] = rin[u].y;
    }
  }
  // inviscid sums into the rate
  auto add_rate = [&](auto dir) {
    constexpr int D = decltype(dir)::d;
    if (!RATE || !act) return;
    const double sc = tb.sc[D];
#pragma unroll
    for (int f = 0; f < 5; ++f) add_line<N>(sA + f * SF, o, sc, v[f], D == 0);
  };
  // gradients of (u, v, w, T) along the line
  auto gradient = [&](auto dir) {
    constexpr int D = decltype(dir)::d;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const double q[5] = {sS[o[m]], sS[SF + o[m]], sS[2 * SF + o[m]], sS[3 * SF + o[m]], sS[4 * SF + o[m]]};
      double p[4];
      primitive(q, g1, p);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k][m] = p[k];
    }
    const double sc = tb.sc[D];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double P[N];
#pragma unroll
      for (int m = 0; m < N; ++m) P[m] = v[k][m];
#pragma unroll
      for (int m = 0; m < N; ++m) {
        double vol = 0.0;
#pragma unroll
        for (int c = 0; c < N; ++c) vol = fma(tab.dh(m, c), P[c], vol);
        v[k][m] = sc * (tab.liftp(m) * hp[k] - tab.liftm(m) * hm[k] - vol);
      }
#pragma unroll
      for (int m = 0; m < N; ++m) asm volatile("" : "+v"(v[k][m]));
    }
  };
  // their part of stress and heat flux
  auto add_stress = [&](auto dir) {
    constexpr int D = decltype(dir)::d;
    if (!act) return;
    const double a4 = mu * (4.0 / 3.0), a2 = -(mu * (2.0 / 3.0));
    // diagonal: mu (2 d_D u_D delta_kD - 2/3 d_D u_D)
#pragma unroll
    for (int k = 0; k < 3; ++k) add_line<N>(sG + k * SF, o, k == D ? a4 : a2, v[D], D == 0);
    // off the diagonal: mu d_D u_k into tau_kD
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k != D) add_line<N>(sG + stress(k, D) * SF, o, mu, v[k], D == 0 || (D == 1 && k == 2));
    add_line<N>(sG + (6 + D) * SF, o, kappa, v[3], true);
  };
  // every sum in the order x, y, z; a wave forms its gradients while the
  // next one adds its inviscid sums
  if (wave == 0) add_rate(Dir<0>{});
  __syncthreads();
  if (wave == 0) gradient(Dir<0>{});
  else if (wave == 1) add_rate(Dir<1>{});
  __syncthreads();
  if (wave == 0) add_stress(Dir<0>{});
  else if (wave == 1) gradient(Dir<1>{});
  else add_rate(Dir<2>{});
  __syncthreads();
  if (wave == 1) add_stress(Dir<1>{});
  else if (wave == 2) gradient(Dir<2>{});
  __syncthreads();
  if (wave == 2) add_stress(Dir<2>{});
  __syncthreads();

  // ---- phase 2: viscous flux on the line, its end traces out, its
  //      derivative with half the own traces
  along(wave, [&](auto dir) {
    constexpr int D = decltype(dir)::d;
    double F[4][N];
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const double ri = dgdev::recip(sS[o[m]]);
      double en = sG[(6 + D) * SF + o[m]];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        F[k][m] = sG[stress(k, D) * SF + o[m]];
        en = fma(sS[(1 + k) * SF + o[m]] * ri, F[k][m], en);
      }
      F[3][m] = en;
    }
    const int64_t EN2 = (int64_t)tb.E * N2;
    double* Tl = T + (int64_t)(2 * D * 4) * EN2 + (int64_t)e0 * N2 + ln;
    const double sc = tb.sc[D];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double fl = 0.0, fr = 0.0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        fl = fma(tab.lm(m), F[k][m], fl);
        fr = fma(tab.lp(m), F[k][m], fr);
      }
      fl *= 0.5;
      fr *= 0.5;
      if (act && el < ne) {
        Tl[k * EN2] = fl;
        Tl[(4 + k) * EN2] = fr;
      }
#pragma unroll
      for (int m = 0; m < N; ++m) {
        double vol = 0.0;
#pragma unroll
        for (int c = 0; c < N; ++c) vol = fma(tab.dh(m, c), F[k][c], vol);
        v[k][m] = sc * (tab.liftp(m) * fr - tab.liftm(m) * fl - vol);
      }
#pragma unroll
      for (int m = 0; m < N; ++m) asm volatile("" : "+v"(v[k][m]));
    }
  });
  auto add2 = [&] {
    if (!act) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) add_line<N>(sA + (1 + k) * SF, o, 1.0, v[k], false);
  };
  if (wave == 0) add2();
  __syncthreads();
  if (wave == 1) add2();
  __syncthreads();
  if (wave == 2) add2();
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PU; ++u) {
    const int x = imin(tid + V::NT * u, 5 * NU - 1), f = x / NU;
    const int n = imin(2 * (x - f * NU), cnt - 2);
    const double* r = sA + f * SF + L::node(n);
    const double2 v = {r[0], r[1]};
    __builtin_memcpy(R + f * EN3 + span + n, &v, 16);
  }
}

// The neighbours' part of the viscous rate.  One wave per block of elements
// of one x-row; it streams R, Q and res, so their bytes bound it.
template <int N, int MODE>
__global__ void __launch_bounds__(64)
k_visc_update(DGTables tb, const double* __restrict__ T, double* __restrict__ R, double* __restrict__ Q,
              double* __restrict__ res, double rka, double rkb, double dt, DGOrder ord) {
  using V = VLine<N>;
  constexpr int EPB = V::EPB, N2 = V::N2, N3 = V::N3, FP = V::FP;
  constexpr int UPT = ((EPB * N3 + 1) / 2 + 63) / 64;
  __shared__ double sT[24 * FP];     // [2 d + side][4][FP]: half the trace of the neighbour across face (d, side)
  __shared__ double sL[6 * N];       // [2 d + side][N]: +-(2/h_d) l(+-1) / w
  const Block blk = dgdev::block_of<EPB>(tb, ord, blockIdx.x, gridDim.x);
  const int e0 = blk.e0, ne = blk.ne, x0 = blk.x0, nx = tb.nx, plane = tb.nx * tb.ny, lane = threadIdx.x;
  const int64_t EN3 = (int64_t)tb.E * N3, EN2 = (int64_t)tb.E * N2, span = (int64_t)e0 * N3;
  const int cnt = ne * N3;
  constexpr int F0 = MODE == 0 ? 1 : 0;   // the mass equation has no viscous part
  const int ln = imin(lane, FP - 1), el = imin(ln / N2, ne - 1), pt = ln % N2;
  const int xl = el > 0 ? e0 + el - 1 : x0 == 0 ? e0 + nx - 1 : e0 - 1;
  const int xr = el + 1 < ne ? e0 + el + 1 : x0 + ne == nx ? e0 - x0 : e0 + ne;
  const int yl = e0 + el + (blk.y == 0 ? (tb.ny - 1) * nx : -nx);
  const int yr = e0 + el + (blk.y == tb.ny - 1 ? -(tb.ny - 1) * nx : nx);
  const int zl = e0 + el + (blk.z == 0 ? (tb.nz - 1) * plane : -plane);
  const int zr = e0 + el + (blk.z == tb.nz - 1 ? -(tb.nz - 1) * plane : plane);
  const int en[6] = {xl, xr, yl, yr, zl, zr};
  double t[6][4];
#pragma unroll
  for (int face = 0; face < 6; ++face)
#pragma unroll
    for (int k = 0; k < 4; ++k) t[face][k] = T[((face ^ 1) * 4 + k) * EN2 + (int64_t)en[face] * N2 + pt];
  // node pairs two at a time (from N = 7 there are three or four per lane)
  constexpr int UG = UPT < 2 ? UPT : 2;
  // Q and res are updated in place and the last pair may be taken twice, so
  // both takings have to fall into the last two rows of pairs
  static_assert(UPT <= UG || (EPB == 1 && (N3 + 1) / 2 > 64 * (UPT - 1)), "repeated pairs are loaded together");
  double2 r[UG][5], q[UG][5], x[UG][5];
  auto load = [&](int u0) {
#pragma unroll
    for (int u = 0; u < UG; ++u) {
      if (u0 + u >= UPT) continue;
      const int64_t g = span + imin(2 * (lane + 64 * (u0 + u)), cnt - 2);
#pragma unroll
      for (int f = F0; f < 5; ++f) {
        r[u][f] = dgdev::load_pair_nt(R + f * EN3 + g);
        if (MODE != 0) __builtin_memcpy(&q[u][f], Q + f * EN3 + g, 16);
        if (MODE == 1) x[u][f] = dgdev::load_pair_nt(res + f * EN3 + g);
      }
    }
  };
  load(0);
  if (lane < N) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double lm = 0.0, lp = 0.0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        lm = lane == m ? tb.liftm[m] : lm;
        lp = lane == m ? tb.liftp[m] : lp;
      }
      sL[2 * d * N + lane] = -tb.sc[d] * lm;
      sL[(2 * d + 1) * N + lane] = tb.sc[d] * lp;
    }
  }
#pragma unroll
  for (int face = 0; face < 6; ++face)
#pragma unroll
    for (int k = 0; k < 4; ++k) sT[(face * 4 + k) * FP + ln] = t[face][k];
  __syncthreads();
  // viscous rate of node n of the block from the neighbours' traces
  auto lift = [&](int n, double* v) {
    const int e = n / N3, i = n % N, j = n / N % N, k = n / N2 % N;
    const int at[3] = {e * N2 + j + N * k, e * N2 + i + N * k, e * N2 + i + N * j};
    const int m[3] = {i, j, k};
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = 0.0;
#pragma unroll
    for (int face = 0; face < 6; ++face) {
      const double l = sL[face * N + m[face / 2]];
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = fma(l, sT[(face * 4 + c) * FP + at[face / 2]], v[c]);
    }
  };
#pragma unroll
  for (int u0 = 0; u0 < UPT; u0 += UG) {
    if (u0 > 0) load(u0);
#pragma unroll
    for (int u = 0; u < UG; ++u) {
      if (u0 + u >= UPT) continue;
      const int n = imin(2 * (lane + 64 * (u0 + u)), cnt - 2);
      double v0[4], v1[4];
      lift(n, v0);
      lift(n + 1, v1);
      const int64_t g = span + n;
#pragma unroll
      for (int f = F0; f < 5; ++f) {
        double2 rate = r[u][f];
        if (f > 0) {
          rate.x += v0[f > 0 ? f - 1 : 0];
          rate.y += v1[f > 0 ? f - 1 : 0];
        }
        if (MODE == 0) {
          __builtin_memcpy(R + f * EN3 + g, &rate, 16);
        } else {
          double2 y;
          y.x = MODE == 2 ? dt * rate.x : fma(rka, x[u][f].x, dt * rate.x);
          y.y = MODE == 2 ? dt * rate.y : fma(rka, x[u][f].y, dt * rate.y);
          dgdev::store_pair_nt(res + f * EN3 + g, y);
          y.x = fma(rkb, y.x, q[u][f].x);
          y.y = fma(rkb, y.y, q[u][f].y);
          __builtin_memcpy(Q + f * EN3 + g, &y, 16);
        }
      }
    }
  }
}

template <int N>
int launch_n(const dg_ctx* c, const double* Q, double* T, double* R, double* Qu, double* res, int mode, double a,
             double b, double dt, int first, bool rate) {
  unsigned grid;
  const DGOrder ord = dg_order(c, VLine<N>::EPB, &grid, true);
  if (rate)
    hipLaunchKernelGGL((k_visc_line<N, true>), dim3(grid), dim3(192), 0, c->stream, c->tab, Q, T, R, c->mu, c->kappa,
                       ord);
  else
    hipLaunchKernelGGL((k_visc_line<N, false>), dim3(grid), dim3(192), 0, c->stream, c->tab, Q, T, R, c->mu, c->kappa,
                       ord);
#define DG_LAUNCH(m) \
  hipLaunchKernelGGL((k_visc_update<N, m>), dim3(grid), dim3(64), 0, c->stream, c->tab, T, R, Qu, res, a, b, dt, ord)
  if (mode == 0) DG_LAUNCH(0);
  else if (first) DG_LAUNCH(2);
  else DG_LAUNCH(1);
#undef DG_LAUNCH
  return (int)hipGetLastError();
}

}  // namespace

int dg_launch_visc_line(const dg_ctx* c, const double* Q, double* T, double* R, double* Qu, double* res, int mode,
                        double a, double b, double dt, int first, bool rate) {
  switch (c->N) {
    case 2: return launch_n<2>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 3: return launch_n<3>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 4: return launch_n<4>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 5: return launch_n<5>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 6: return launch_n<6>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 7: return launch_n<7>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    case 8: return launch_n<8>(c, Q, T, R, Qu, res, mode, a, b, dt, first, rate);
    default: return (int)hipErrorInvalidValue;
  }
}
