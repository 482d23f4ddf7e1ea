// Stage kernel of the variable-degree mesh with one thread per line: the
// arithmetic of k_varp (kern_varp.hip), in the same order, so bitwise its
// results, split over threads as stage_line_body (stage_line.h) splits the
// single-degree stage: a lane holds a 1-D line of its element per direction,
// a workgroup is one wave, the 1-D tables sit in scalar registers.  What
// differs is where a line's neighbours are: the elements of a workgroup are
// any entries of the group's list, and a face either has a neighbour of the
// same size and degree (its state is read along the normal line, also where
// the neighbour is in the same workgroup) or a projected flux in the face-flux
// buffer.  A lane whose face has a flux reads a line of its own element like
// the others, so that those loads keep their constant strides (offsets of the
// instruction; with strides per lane 48^3 p = 4 took 646 us a stage against
// 635, 32^3 p = 6 602 against 552) and no branch, and the blocks with such a
// face fetch the fluxes afterwards.

#include "dg_varp.h"
#include "stage_line.h"

namespace dgdev {
namespace {

// An entry of the face table.
struct VFace {
  long long raw;
  __device__ __forceinline__ bool flux() const { return (raw & 3) == DG_FACE_MORTAR; }
  __device__ __forceinline__ long long place() const { return raw >> 2; }
};

// 40^3 cells, degrees 3..5, 7.8% refined (us a stage per group, k_varp before):
// p = 3 52 (60), p = 4 252 and 85 (320, 97), p = 5 294 (392); of the last, the
// traces for the next stage take 20.
template <int N, int MODE, bool TR>
__global__ void __launch_bounds__(64, 2)
k_varp_line(const DGTables tb, const DGVarpMesh mesh, int first, int count, const double* __restrict__ Qin,
            double* __restrict__ Qout, double* __restrict__ RR, double rka, double rkb, double dt) {
  constexpr int EPB = dg_line_elems(N);
  using L = LineLds<N>;
  constexpr int N2 = N * N, N3 = N2 * N, FP = EPB * N2, SF = LineSmem<N, EPB>::SF;
  constexpr int PPE = (N3 + 1) / 2;                 // node pairs of an element (the last may overlap at odd N)
  constexpr int UPT = (EPB * PPE + 63) / 64;        // node pairs per lane and field
  constexpr int TASKS = 6 * EPB;
  static_assert(N >= 2 && FP <= 64 && 2 * LinePairs<N, EPB>::LPF <= 64, "one line and one pair per lane");
  __shared__ __align__(16) double smem[LineSmem<N, EPB>::size];
  __shared__ long long sOff[EPB];
  __shared__ long long sFace[TASKS];   // [face][element] the face table's entries
  __shared__ long long sNb[TASKS];     // the neighbours' first nodes (own, where the face has a flux)
  double* sS = smem;             // [5][SF] state
  double* sA = smem + 5 * SF;    // [5][SF] rate
  double* sT = sA;               // [2][5][FP] neighbour traces or fluxes, before the rate is first written

  const int lane = threadIdx.x;
  // each XCD takes a contiguous part of the list
  const int blk0 = xcd_block(blockIdx.x, gridDim.x) * EPB;
  const int ne = imin(count - blk0, EPB);
  const int64_t T = mesh.T;
  const LineTables<N> tab{tb};

  // ---- A: the block's places in the state and its faces (absent elements
  //         repeat the last one)
  bool any = false;   // a face of the block has a flux
#pragma unroll
  for (int i = 0; i < (TASKS + 63) / 64; ++i) {
    const int t = imin(lane + 64 * i, TASKS - 1);
    const int face = t / EPB, fel = t - face * EPB;
    const int e = mesh.list[first + blk0 + imin(fel, ne - 1)];
    const VFace fc{mesh.face[(int64_t)e * 6 + face]};
    const long long off = mesh.off[e];
    if (i == 0 && lane < EPB) sOff[lane] = off;
    sFace[t] = fc.raw;
    sNb[t] = fc.flux() ? off : fc.place();
    any = any || __ballot(fc.flux()) != 0ull;
  }
  __syncthreads();

  int pn[UPT];          // node in LDS and
  long long pg[UPT];    // in the state of the lane's pairs (past the block's end the last one)
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
    const int i = imin(lane + 64 * u, ne * PPE - 1);
    const int e = i / PPE, n = imin(2 * (i - e * PPE), N3 - 2);
    pn[u] = L::node(e * N3 + n);
    pg[u] = sOff[e] + n;
  }
  double2 own[UPT][5];
#pragma unroll
  for (int u = 0; u < UPT; ++u)
#pragma unroll
    for (int f = 0; f < 5; ++f) __builtin_memcpy(&own[u][f], Qin + f * T + pg[u], 16);

  // line `lane` = (el, pt), pt = (a, b) the tangential indices, lower axis
  // fastest
  const bool act = lane < FP;
  const int ln = imin(lane, FP - 1);
  const int el = ln / N2, pt = ln - el * N2;
  const int b = pt / N, a = pt - b * N;
  // the x-neighbours' lines
  double xo[2][5][N];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const double* xb = Qin + sNb[s * EPB + el] + pt * N;
#pragma unroll
    for (int f = 0; f < 5; ++f) {
#pragma unroll
      for (int h = 0; h < N / 2; ++h) {
        double2 v;
        __builtin_memcpy(&v, xb + f * T + 2 * h, 16);
        xo[s][f][2 * h] = v.x;
        xo[s][f][2 * h + 1] = v.y;
      }
      if (N % 2) xo[s][f][N - 1] = xb[f * T + N - 1];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      double* s = sS + f * SF + pn[u];
      s[0] = own[u][f].x;
      s[1] = own[u][f].y;
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- B: the neighbours' traces.  On the y- and z-faces a lane forms those
  //         of a pair of points, which change lanes through sT; each consumed
  //         field of the x- and y-lines issues the field of the y- and z-lines
  //         that takes its registers.
  const PairLane<N, EPB> pl(imin(lane, 2 * LinePairs<N, EPB>::LPF - 1));
  const bool paired = lane < 2 * LinePairs<N, EPB>::LPF;
  const double* yb = Qin + sNb[(2 + pl.side) * EPB + pl.fel] + tnode<N>(1, 0, pl.pt);
  const double* zb = Qin + sNb[(4 + pl.side) * EPB + pl.fel] + tnode<N>(2, 0, pl.pt);
  double* pT = sT + pl.side * 5 * FP + pl.fel * N2 + pl.pt;
  double pc[N];
#pragma unroll
  for (int m = 0; m < N; ++m) pc[m] = pl.side ? tab.lm(m) : tab.lp(m);
  double2 w[5][N];
  double q[5][N], tl[5], tr[5], nl[3][5], nr[3][5];
  auto take = [&](int d) {
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      nl[d][f] = sT[f * FP + ln];
      nr[d][f] = sT[(5 + f) * FP + ln];
    }
    __syncthreads();
  };
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    double u = 0.0, v = 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      u = fma(tab.lp(m), xo[0][f][m], u);   // left neighbour: its right end
      v = fma(tab.lm(m), xo[1][f][m], v);   // right neighbour: its left end
    }
    asm volatile("" : "+v"(u), "+v"(v));   // formed here, before the y-line takes the registers
    nl[0][f] = u;
    nr[0][f] = v;
    load_pair_line<N, 1>(yb + f * T, w[f]);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if (paired) store_pair_trace<N>(w[f], pc, pT + f * FP);
    load_pair_line<N, 2>(zb + f * T, w[f]);
    __builtin_amdgcn_sched_barrier(0);
  }
  take(1);
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if (paired) store_pair_trace<N>(w[f], pc, pT + f * FP);
  }
  take(2);
  // faces that have a flux take it in the neighbour's trace's place
  bool ml[3] = {}, mr[3] = {};
  if (any) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const VFace fl{sFace[2 * d * EPB + el]}, fr{sFace[(2 * d + 1) * EPB + el]};
      ml[d] = fl.flux();
      mr[d] = fr.flux();
      if (ml[d]) {
#pragma unroll
        for (int f = 0; f < 5; ++f) nl[d][f] = mesh.fbuf[fl.place() + f * N2 + pt];
      }
      if (mr[d]) {
#pragma unroll
        for (int f = 0; f < 5; ++f) nr[d][f] = mesh.fbuf[fr.place() + f * N2 + pt];
      }
    }
  }

  // ---- C: the three directions, summed through sA in the order x, y, z
  auto line = [&](auto dir) {
    constexpr int D = decltype(dir)::value;
    int o[N];
#pragma unroll
    for (int m = 0; m < N; ++m) o[m] = D == 0 ? L::row(el, b, a) + m : D == 1 ? L::row(el, b, m) + a : L::row(el, m, b) + a;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
      for (int m = 0; m < N; ++m) q[f][m] = sS[f * SF + o[m]];
    end_traces<N>(tab, q, tl, tr);
    if (act) {
      const double sc = tb.sc[D];
      double fl[5], fr[5];
      lf_flux_d<D>(nl[D], tl, tb.gamma, tb.gm1, fl);
      lf_flux_d<D>(tr, nr[D], tb.gamma, tb.gm1, fr);
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        fl[f] = ml[D] ? nl[D][f] : fl[f];
        fr[f] = mr[D] ? nr[D][f] : fr[f];
      }
      line_rate<N, D>(tab, q, fl, fr, [&](int f, const double(&s)[N]) {
        add_line<N>(sA + f * SF, o, sc, s, D == 0);
      });
    }
    __syncthreads();
  };
  line(std::integral_constant<int, 0>{});
  double2 r[UPT][5];
  // the residual: its latency overlaps the y- and z-lines
  if (MODE == 1) {
#pragma unroll
    for (int u = 0; u < UPT; ++u)
#pragma unroll
      for (int f = 0; f < 5; ++f) r[u][f] = load_pair_nt(RR + f * T + pg[u]);
    __builtin_amdgcn_sched_barrier(0);
  }
  line(std::integral_constant<int, 1>{});
  line(std::integral_constant<int, 2>{});

  // ---- D: output
#pragma unroll
  for (int u = 0; u < UPT; ++u) {
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      const double a0 = sA[f * SF + pn[u]], a1 = sA[f * SF + pn[u] + 1];
      double2 v;
      if (MODE == 0) {
        v.x = a0;
        v.y = a1;
        __builtin_memcpy(RR + f * T + pg[u], &v, 16);
      } else {
        v.x = MODE == 2 ? dt * a0 : fma(rka, r[u][f].x, dt * a0);
        v.y = MODE == 2 ? dt * a1 : fma(rka, r[u][f].y, dt * a1);
        double2 qn;
        qn.x = fma(rkb, v.x, sS[f * SF + pn[u]]);
        qn.y = fma(rkb, v.y, sS[f * SF + pn[u] + 1]);
        __builtin_memcpy(Qout + f * T + pg[u], &qn, 16);
        store_pair_nt(RR + f * T + pg[u], v);
        own[u][f] = qn;
      }
    }
  }
  // ---- E: the new state's traces on the faces that take their flux from
  //         fbuf, for the next stage's face launches
  if (TR && any) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        double* s = sS + f * SF + pn[u];
        s[0] = own[u][f].x;
        s[1] = own[u][f].y;
      }
    }
    __syncthreads();
    if (act && el < ne) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (!ml[d] && !mr[d]) continue;
        double* hl = mesh.tbuf + VFace{sFace[2 * d * EPB + el]}.place() + pt;
        double* hr = mesh.tbuf + VFace{sFace[(2 * d + 1) * EPB + el]}.place() + pt;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          double u = 0.0, v = 0.0;
#pragma unroll
          for (int m = 0; m < N; ++m) {
            const int o = d == 0 ? L::row(el, b, a) + m : d == 1 ? L::row(el, b, m) + a : L::row(el, m, b) + a;
            const double x = sS[f * SF + o];
            u = fma(tab.lm(m), x, u);
            v = fma(tab.lp(m), x, v);
          }
          if (ml[d]) hl[f * N2] = u;
          if (mr[d]) hr[f * N2] = v;
        }
      }
    }
  }
}

template <int N>
int launch_n(hipStream_t stream, const DGTables& tb, const DGVarpMesh& m, int first, int count, const double* Qin,
             double* Qout, double* RR, int mode, double a, double b, double dt, bool tr) {
  const dim3 grid((unsigned)((count + dg_line_elems(N) - 1) / dg_line_elems(N))), blk(64);
#define VARP_LAUNCH(MODE, TR) \
  hipLaunchKernelGGL((k_varp_line<N, MODE, TR>), grid, blk, 0, stream, tb, m, first, count, Qin, Qout, RR, a, b, dt)
  if (mode == 0)
    VARP_LAUNCH(0, false);
  else if (mode == 1 && tr)
    VARP_LAUNCH(1, true);
  else if (mode == 1)
    VARP_LAUNCH(1, false);
  else if (tr)
    VARP_LAUNCH(2, true);
  else
    VARP_LAUNCH(2, false);
#undef VARP_LAUNCH
  return (int)hipGetLastError();
}

}  // namespace
}  // namespace dgdev

int dg_launch_varp_line(hipStream_t stream, int N, const DGTables& tb, const DGVarpMesh& m, int first, int count,
                        const double* Qin, double* Qout, double* RR, int mode, double a, double b, double dt,
                        bool traces) {
  using namespace dgdev;
  if (count <= 0) return 0;
#define CALL(n) launch_n<n>(stream, tb, m, first, count, Qin, Qout, RR, mode, a, b, dt, traces && mode != 0)
  switch (N) {
    case 2: return CALL(2);
    case 3: return CALL(3);
    case 4: return CALL(4);
    case 5: return CALL(5);
    case 6: return CALL(6);
    case 7: return CALL(7);
    default: return (int)hipErrorInvalidValue;
  }
#undef CALL
}
