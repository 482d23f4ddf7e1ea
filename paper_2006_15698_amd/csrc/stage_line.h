// Device code of the FP64 DG Euler stage with one thread per line.
//
// Same arithmetic, in the same order, as stage_nb_body (stage_nb.h), so the
// results are bitwise the same; the work is split differently.  A thread owns
// one 1-D line of nodes of its element per direction, held in registers, so
// that
//   - the volume contraction (N outputs from N inputs) reads each flux from
//     a register and the 1-D tables from scalar registers (one thread per
//     node read 5 N fluxes and N table entries from LDS per direction);
//   - the same thread forms both end traces, both Lax-Friedrichs fluxes and
//     their lift, so face fluxes never pass through LDS and no lane idles in
//     a face phase;
//   - a workgroup is one wave, with no barrier to wait at: every wave moves
//     through its load, compute and store phases on its own.
// LDS holds the state of the block (S) and its rate (A), both addressed by
// node: a thread reads the y- and z-lines of S, and the rate of the three
// directions is summed through A.  State, residual and results move between
// HBM and LDS in 16-byte pieces of the contiguous per-field spans.
#pragma once

#include "stage_nb.h"

namespace dgdev {

// LDS index of node (row j of plane k, element el), first node of the row.
// At N = 2, 4, 8 the rows of plane k are permuted by j ^ k: the y-lines of a
// wave (same j, all k) would otherwise fall on a quarter of the banks.
template <int N>
struct LineLds {
  static constexpr int N2 = N * N, N3 = N2 * N;
  static constexpr bool SWZ = (N & (N - 1)) == 0;
  __host__ __device__ static constexpr int row(int el, int k, int j) {
    return el * N3 + k * N2 + (SWZ ? (j ^ k) : j) * N;
  }
  // node g of the block's contiguous per-field span (g = el N^3 + ...)
  __host__ __device__ static constexpr int node(int g) {
    if (!SWZ) return g;
    const int el = g / N3, n = g % N3;
    return row(el, n / N2, (n / N) % N) + n % N;
  }
};

// 16-byte accesses at 8-byte alignment that mark their line as not reused
// (the residual: no other workgroup of the launch reads it, and it would push
// the state its neighbours do read out of the L2).
typedef double pair_nt __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ double2 load_pair_nt(const double* p) {
  const pair_nt v = __builtin_nontemporal_load((const pair_nt*)p);
  return double2{v[0], v[1]};
}
__device__ __forceinline__ void store_pair_nt(double* p, double2 v) {
  __builtin_nontemporal_store(pair_nt{v.x, v.y}, (pair_nt*)p);
}

// The 1-D tables of one degree as a thread uses them, halves only: the rule's
// reflection symmetry holds to the last bit (dg_build_tables), so the other
// half is read mirrored, and the N^2 / 2 + 2 N values fit the scalar registers.
template <int N>
struct LineTables {
  const DGTables& tb;
  __device__ __forceinline__ double dh(int m, int a) const {
    const int k = m * N + a;
    return k < N * N / 2 ? tb.Dh[k] : 2 * k + 1 == N * N ? 0.0 : -tb.Dh[N * N - 1 - k];
  }
  __device__ __forceinline__ double lm(int m) const { return tb.lm[m]; }
  __device__ __forceinline__ double lp(int m) const { return tb.lm[N - 1 - m]; }
  __device__ __forceinline__ double liftm(int m) const { return tb.liftm[m]; }
  __device__ __forceinline__ double liftp(int m) const { return tb.liftm[N - 1 - m]; }
};

// A wave's direction as a compile-time constant (uniform over the wave), where
// the three waves of a workgroup take a direction each.
template <int D>
struct Dir {
  static constexpr int d = D;
};
template <class F>
__device__ __forceinline__ void along(int wave, F&& f) {
  if (wave == 0) f(Dir<0>{});
  else if (wave == 1) f(Dir<1>{});
  else f(Dir<2>{});
}

template <int N, int EPB>
struct LineSmem {
  // per-field strides are even, so that pairs stay 16-byte aligned at even N
  static constexpr int SF = (EPB * N * N * N + 1) & ~1;
  static constexpr int size = 10 * SF;
};

// Pairs of neighbour-line points as PairLane (stage_nb.h), on a wave of its
// own: lanes [0, LPF) the - face, [LPF, 2 LPF) the + face.
template <int N, int EPB>
struct LinePairs {
  static constexpr int P = (N + 1) / 2, LPF = EPB * N * P;
};

// One field of the neighbour lines of a pair: w[m] the pair's nodes at
// position m of the line along D.
template <int N, int D>
__device__ __forceinline__ void load_pair_line(const double* qf, double2 (&w)[N]) {
#pragma unroll
  for (int m = 0; m < N; ++m) __builtin_memcpy(&w[m], qf + m * (D == 1 ? N : N * N), 16);
}

// The traces of one field of a pair (the FMA chain of chunk_trace) into h[0],
// h[1].  (An overlapping pair writes its first point's trace a second time,
// the same value.)
template <int N>
__device__ __forceinline__ void store_pair_trace(const double2 (&w)[N], const double (&c)[N], double* h) {
  double v0 = 0.0, v1 = 0.0;
#pragma unroll
  for (int m = 0; m < N; ++m) {
    v0 = fma(c[m], w[m].x, v0);
    v1 = fma(c[m], w[m].y, v1);
  }
  h[0] = v0;
  h[1] = v1;
}

// x[o[m]] = fma(c, v[m], x[o[m]]) along a line in LDS (or = fma(c, v[m], 0)):
// all reads before the first write, which the compiler, not knowing the
// places distinct, would have to wait for one by one.
template <int N>
__device__ __forceinline__ void add_line(double* x, const int (&o)[N], double c, const double (&v)[N], bool first) {
  double r[N];
#pragma unroll
  for (int m = 0; m < N; ++m) r[m] = first ? 0.0 : x[o[m]];
#pragma unroll
  for (int m = 0; m < N; ++m) x[o[m]] = fma(c, v[m], r[m]);
}

// Volume contraction of direction D on the thread's line q[field][node] plus
// the lift of its two face fluxes fl, fr, handed to `emit(f, s)` for every
// field (2/h_D times s[node] is the rate).
template <int N, int D, class Emit>
__device__ __forceinline__ void line_rate(const LineTables<N>& t, const double (&q)[5][N], const double* fl,
                                          const double* fr, Emit&& emit) {
  double pr[N], ud[N];
#pragma unroll
  for (int a = 0; a < N; ++a) {
    const double rinv = recip(q[0][a]);
    pr[a] = t.tb.gm1 * (q[4][a] - 0.5 * (q[1][a] * q[1][a] + q[2][a] * q[2][a] + q[3][a] * q[3][a]) * rinv);
    ud[a] = q[1 + D][a] * rinv;
  }
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    double F[N], s[N];
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if (f == 0) F[a] = q[1 + D][a];
      else if (f == 4) F[a] = (q[4][a] + pr[a]) * ud[a];
      else F[a] = q[f][a] * ud[a] + (D == f - 1 ? pr[a] : 0.0);
    }
#pragma unroll
    for (int m = 0; m < N; ++m) {
      double v = 0.0;
#pragma unroll
      for (int a = 0; a < N; ++a) v = fma(t.dh(m, a), F[a], v);
      v = fma(t.liftm(m), fl[f], v);
      s[m] = fma(-t.liftp(m), fr[f], v);
    }
    emit(f, s);
  }
}

// The standard form's rate of direction D: line_rate with the two
// Lax-Friedrichs fluxes, on an active lane, after `pre()` on every lane.
// tl, tr: the line's own end traces; nl, nr: the - and + neighbour's traces.
template <int N>
struct EulerLine {
  static constexpr bool BULK = false;   // rates are handed out field by field
  LineTables<N> tab;
  template <int D, class Pre, class Emit>
  __device__ __forceinline__ void rate(const double (&q)[5][N], const double* tl, const double* tr, const double* nl,
                                       const double* nr, bool act, Pre&& pre, Emit&& emit) const {
    const LineTables<N>& t = tab;
    pre();
    if (!act) return;
    double fl[5], fr[5];
    lf_flux_d<D>(nl, tl, t.tb.gamma, t.tb.gm1, fl);
    lf_flux_d<D>(tr, nr, t.tb.gamma, t.tb.gm1, fr);
    line_rate<N, D>(t, q, fl, fr, emit);
  }
};

// Both end traces of a line (the FMA chain of line_trace).
template <int N>
__device__ __forceinline__ void end_traces(const LineTables<N>& t, const double (&q)[5][N], double* tl,
                                           double* tr) {
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      a = fma(t.lm(m), q[f][m], a);
      b = fma(t.lp(m), q[f][m], b);
    }
    tl[f] = a;
    tr[f] = b;
  }
}

// The elements of block blk, 1 <= ne <= EPB, on one wave, with the rate of the
// volume form `form` (EulerLine; kern_split.hip has another); the other
// arguments and MODE as for stage_nb_body.  smem: LineSmem<N, EPB>::size doubles.
// nt: mark the new state as not reused, for states that the next launch would
// not find in the last-level cache anyway (DGOrder::size): their stores then
// do not push the state that the neighbours read out of the L2.
template <int N, int MODE, int EPB, class Form>
__device__ __forceinline__ void stage_line_body(const Form& form, const DGTables& tb, const double* __restrict__ Qin,
                                                double* __restrict__ Qout, double* __restrict__ RR, double rka,
                                                double rkb, double dt, int first, const Block& blk, double* smem,
                                                int lane, bool nt) {
  using L = LineLds<N>;
  constexpr int N2 = N * N, N3 = N2 * N, FP = EPB * N2, SF = LineSmem<N, EPB>::SF;
  constexpr int UPT = ((EPB * N3 + 1) / 2 + 63) / 64;   // node pairs per lane and field
  constexpr int HP = N / 2;                              // 16-byte pieces of an x-line (plus one node at odd N)
  static_assert(N >= 2 && FP <= 64 && 2 * LinePairs<N, EPB>::LPF <= 64, "one line and one pair per lane");
  static_assert(EPB == 1 || 2 * N2 <= 64, "one outer x-line per lane");

  double* sS = smem;             // [5][SF] state
  double* sA = smem + 5 * SF;    // [5][SF] rate
  double* sT = sA;               // [2][5][FP] neighbour traces, before the rate is first written
  // a form that hands out its rates at its end (Form::BULK) leaves the y- and
  // z-traces in LDS beside each other until then, which frees 40 registers
  constexpr bool KEEP = Form::BULK && 20 * FP <= 5 * SF;

  const int nx = tb.nx, ny = tb.ny, nz = tb.nz;
  const int64_t EN3 = (int64_t)tb.E * N3;
  const int e0 = blk.e0, ne = blk.ne, x0 = blk.x0, ey = blk.y, ez = blk.z;
  const int plane = nx * ny;
  const int eym = ey == 0 ? e0 + (ny - 1) * nx : e0 - nx;
  const int eyp = ey == ny - 1 ? e0 - (ny - 1) * nx : e0 + nx;
  const int ezm = ez == 0 ? e0 + (nz - 1) * plane : e0 - plane;
  const int ezp = ez == nz - 1 ? e0 - (nz - 1) * plane : e0 + plane;
  const int exl = x0 == 0 ? e0 + nx - 1 : e0 - 1;
  const int exr = x0 + ne == nx ? e0 - x0 : e0 + ne;
  const int cnt = ne * N3;

  // ---- A: loads.  Own state, outer x-lines and y-lines are issued before
  //         the first is waited for; then every consumed field of the x- and
  //         y-lines issues the field of the y- and z-lines that takes its
  //         registers.
  const LineTables<N>& tab = form.tab;
  // own state, node pairs of the contiguous per-field span (past its end the
  // last pair is read, and written, again)
  const int64_t span = (int64_t)e0 * N3;
  double2 own[UPT][5];
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
    const int g = imin(2 * (lane + 64 * u), cnt - 2);
#pragma unroll
    for (int f = 0; f < 5; ++f) __builtin_memcpy(&own[u][f], Qin + f * EN3 + span + g, 16);
  }
  // x-lines of the outer x-neighbours: EPB >= 2: lanes [0, N^2) the left
  // one's, [N^2, 2 N^2) the right one's; EPB = 1: both in every lane
  constexpr int XL = EPB == 1 ? 2 : 1;
  double xo[XL][5][N];
  const int xside = lane >= N2;
#pragma unroll
  for (int s = 0; s < XL; ++s) {
    const int right = EPB == 1 ? s : xside;
    const int pt = EPB == 1 ? imin(lane, N2 - 1) : imin(lane - right * N2, N2 - 1);
    const double* xb = Qin + (int64_t)(right ? exr : exl) * N3 + pt * N;
#pragma unroll
    for (int f = 0; f < 5; ++f) {
#pragma unroll
      for (int h = 0; h < HP; ++h) {
        double2 v;
        __builtin_memcpy(&v, xb + f * EN3 + 2 * h, 16);
        xo[s][f][2 * h] = v.x;
        xo[s][f][2 * h + 1] = v.y;
      }
      if (N % 2) xo[s][f][N - 1] = xb[f * EN3 + N - 1];
    }
  }
  // pairs of neighbour-line points on the y- and z-faces.  Lanes past the
  // pairs and pairs of absent elements repeat a valid pair (unconditional
  // loads: one under a condition is waited for where the branches join).
  const PairLane<N, EPB> pl(imin(lane, 2 * LinePairs<N, EPB>::LPF - 1));
  const bool paired = lane < 2 * LinePairs<N, EPB>::LPF;
  const int pfel = imin(pl.fel, ne - 1) * N3;
  const double* yb = Qin + (int64_t)(pl.side ? eyp : eym) * N3 + pfel + tnode<N>(1, 0, pl.pt);
  const double* zb = Qin + (int64_t)(pl.side ? ezp : ezm) * N3 + pfel + tnode<N>(2, 0, pl.pt);
  double* pT = sT + pl.side * 5 * FP + pl.fel * N2 + pl.pt;
  double pc[N];
#pragma unroll
  for (int m = 0; m < N; ++m) pc[m] = pl.side ? tab.lm(m) : tab.lp(m);
  double2 w[5][N];
  // from N = 6 the registers do not hold the y-lines beside the x-lines
  constexpr bool YLATE = EPB == 1;
  if (!YLATE) {
#pragma unroll
    for (int f = 0; f < 5; ++f) load_pair_line<N, 1>(yb + f * EN3, w[f]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
    const int g = imin(2 * (lane + 64 * u), cnt - 2);
    // (at even N a pair never leaves its row)
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double* s = sS + f * SF + L::node(g);
      s[0] = own[u][f].x;
      s[1] = own[u][f].y;
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- B: the thread's lines: line `lane` = (el, pt), pt = (a, b) the
  //         tangential indices, lower axis fastest; the neighbours' traces
  //         change lanes through sT
  const bool act = lane < FP;
  const int ln = imin(lane, FP - 1);
  const int el = ln / N2, pt = ln - el * N2;
  const int b = pt / N, a = pt - b * N;
  double q[5][N], tl[5], tr[5], nl[3][5], nr[3][5];
  auto take = [&](int d, int off = 0) {
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      nl[d][f] = sT[off + f * FP + ln];
      nr[d][f] = sT[off + (5 + f) * FP + ln];
    }
    __syncthreads();
  };
  if constexpr (EPB == 1) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double u = 0.0, v = 0.0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        u = fma(tab.lp(m), xo[0][f][m], u);   // left neighbour: its right end
        v = fma(tab.lm(m), xo[XL - 1][f][m], v);   // right neighbour: its left end
      }
      // (formed here, before the y-line takes the registers: left to itself
      // the compiler sinks the chains to the first use of the traces)
      asm volatile("" : "+v"(u), "+v"(v));
      nl[0][f] = u;
      nr[0][f] = v;
      if (YLATE) load_pair_line<N, 1>(yb + f * EN3, w[f]);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    double c[N];
#pragma unroll
    for (int m = 0; m < N; ++m) c[m] = xside ? tab.lm(m) : tab.lp(m);
    double* t = sT + (xside ? 5 * FP + (ne - 1) * N2 + lane - N2 : lane);
    if (lane < 2 * N2) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        double v = 0.0;
#pragma unroll
        for (int m = 0; m < N; ++m) v = fma(c[m], xo[0][f][m], v);
        t[f * FP] = v;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  auto read_x = [&] {
    const double* s = sS + L::row(el, b, a);   // x-line: j = a, k = b
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
      for (int m = 0; m < N; ++m) q[f][m] = s[f * SF + m];
    end_traces<N>(tab, q, tl, tr);
  };
  __syncthreads();
  if constexpr (EPB > 1) {
    read_x();
    // neighbours inside the block take this line's end traces
    if (act && el + 1 < ne) {
#pragma unroll
      for (int f = 0; f < 5; ++f) sT[f * FP + ln + N2] = tr[f];
    }
    if (act && el > 0 && el < ne) {
#pragma unroll
      for (int f = 0; f < 5; ++f) sT[(5 + f) * FP + ln - N2] = tl[f];
    }
    take(0);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if (paired) store_pair_trace<N>(w[f], pc, pT + f * FP);
    load_pair_line<N, 2>(zb + f * EN3, w[f]);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (!KEEP) take(1);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if (paired) store_pair_trace<N>(w[f], pc, pT + (KEEP ? 10 * FP : 0) + f * FP);
  }
  if (!KEEP) take(2);
  // (read again where it was not held through the loads above)
  if constexpr (EPB == 1 || Form::BULK) read_x();

  // ---- C: the three directions, summed through sA in the order x, y, z
  {
    int o[N];
#pragma unroll
    for (int m = 0; m < N; ++m) o[m] = L::row(el, b, a) + m;
    const double sc = tb.sc[0];
    form.template rate<0>(
          q, tl, tr, nl[0], nr[0], act,
          [&] {
            if (KEEP) {
              take(1);
              take(2, 10 * FP);
            }
          },
          [&](int f, const double(&s)[N]) { add_line<N>(sA + f * SF, o, sc, s, true); });
  }
  __syncthreads();
  double2 r[UPT][5];
  auto read_res = [&] {
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
      const int g = imin(2 * (lane + 64 * u), cnt - 2);
#pragma unroll
      for (int f = 0; f < 5; ++f) r[u][f] = load_pair_nt(RR + f * EN3 + span + g);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the residual: its latency overlaps the y- and z-lines where their rates
  // leave its registers free
  if (MODE == 1 && !Form::BULK) read_res();
  {
    int o[N];   // y-line: i = a, k = b
#pragma unroll
    for (int m = 0; m < N; ++m) o[m] = L::row(el, b, m) + a;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
      for (int m = 0; m < N; ++m) q[f][m] = sS[f * SF + o[m]];
    end_traces<N>(tab, q, tl, tr);
    const double sc = tb.sc[1];
    form.template rate<1>(q, tl, tr, nl[1], nr[1], act, [] {}, [&](int f, const double(&s)[N]) {
        add_line<N>(sA + f * SF, o, sc, s, false);
      });
  }
  __syncthreads();
  {
    int o[N];   // z-line: i = a, j = b
#pragma unroll
    for (int m = 0; m < N; ++m) o[m] = L::row(el, m, b) + a;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
      for (int m = 0; m < N; ++m) q[f][m] = sS[f * SF + o[m]];
    end_traces<N>(tab, q, tl, tr);
    const double sc = tb.sc[2];
    form.template rate<2>(q, tl, tr, nl[2], nr[2], act, [] {}, [&](int f, const double(&s)[N]) {
        add_line<N>(sA + f * SF, o, sc, s, false);
      });
  }
  if (MODE == 1 && Form::BULK) read_res();
  __syncthreads();

  // ---- D: output, node pairs of the per-field spans
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
    const int g = imin(2 * (lane + 64 * u), cnt - 2);
    const int n = L::node(g);
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      const double a0 = sA[f * SF + n], a1 = sA[f * SF + n + 1];
      double2 v;
      if (MODE == 0) {
        v.x = a0;
        v.y = a1;
        __builtin_memcpy(RR + f * EN3 + span + g, &v, 16);
      } else {
        v.x = (MODE == 2 || first) ? dt * a0 : fma(rka, r[u][f].x, dt * a0);
        v.y = (MODE == 2 || first) ? dt * a1 : fma(rka, r[u][f].y, dt * a1);
        double2 qn;
        qn.x = fma(rkb, v.x, sS[f * SF + n]);
        qn.y = fma(rkb, v.y, sS[f * SF + n + 1]);
        if (nt) store_pair_nt(Qout + f * EN3 + span + g, qn);
        else __builtin_memcpy(Qout + f * EN3 + span + g, &qn, 16);
        store_pair_nt(RR + f * EN3 + span + g, v);
      }
    }
  }
}

}  // namespace dgdev
