// Internal declarations shared by the host library and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dg.h"

#define DG_MAXN 8
#define DG_NF 5

// Per-context constant tables, passed by value as a kernel argument.
// Section II-B: collocated Gauss-Legendre nodal basis (Eqs. (6)-(7)).
struct DGTables {
  double Dh[DG_MAXN * DG_MAXN];  // Dh[i*N+a] = w_a l_i'(xi_a) / w_i: the
                                 // volume term of Eq. (5) on one 1-D line,
                                 // mass matrix already divided out
  double lm[DG_MAXN];            // l_i(-1): face interpolation weights
  double lp[DG_MAXN];            // l_i(+1)
  double liftm[DG_MAXN];         // l_i(-1) / w_i: surface term of Eq. (5)
  double liftp[DG_MAXN];         // l_i(+1) / w_i   lifted by M^{-1}
  double w[DG_MAXN];             // Gauss-Legendre weights
  double rs[DG_MAXN];            // rs[i] = sum_a Dh[i*N+a] (free-stream identity:
                                 // (l_i(1) - l_i(-1)) / w_i up to rounding)
  float Dh32[DG_MAXN * DG_MAXN]; // Dh rounded to FP32 (matrix-core variant)
  float lm32[DG_MAXN];           // l_i(-1), l_i(+1) rounded to FP32
  float lp32[DG_MAXN];
  double liftm32[DG_MAXN];       // the FP32 form's lift weights (FP64)
  double liftp32[DG_MAXN];
  double sc[3];                  // 2 / h_d (reference-to-physical metric)
  double hinv[3];                // 1 / h_d
  double J;                      // h_x h_y h_z / 8 (volume Jacobian)
  double gamma;                  // ratio of specific heats, Eq. (3)
  double gm1;                    // gamma - 1
  int nx, ny, nz;
  int E;                         // nx*ny*nz
};

struct dg_ctx {
  int nx, ny, nz, p, N;
  int64_t E;
  double gamma;
  double L[3];
  double xi[DG_MAXN], w[DG_MAXN];
  hipStream_t stream;
  int precision;
  char* ws;
  size_t ws_bytes;
  DGTables tab;
  int timing_on;
  void* timing;   // DGTiming*, owned, created by dg_set_timing
  int exchange;   // DG_EXCHANGE_TRACES or DG_EXCHANGE_NEIGHBOUR (FP64 path)
  int xcd_remap;  // XCD-aware workgroup -> block mapping (neighbour path)
  int order;      // DG_ORDER_LINEAR or DG_ORDER_PENCIL
  int pencil_x;   // pencil extent along x in elements (0: whole row)
  int pencil_z;   // pencil extent along z in element planes
  int pencil_z_set;  // pencil_z was chosen by the caller (DG_OPT_PENCIL_Z_AUTO 0)
  int visc_fused; // viscous FP64 standard form: inviscid rate inside the viscous-flux launch
  // viscous terms (dg_set_viscosity): dynamic viscosity, Prandtl number and
  // conductivity mu gamma / ((gamma - 1) Pr); mu = 0 is the Euler equations
  double mu, prandtl, kappa;
  int volume_form;  // DG_VOLUME_STANDARD or DG_VOLUME_KEP (dg_set_volume_form)
  // graph replay of whole steps (dg_rk_graph_steps): one executable graph
  // per place of a step in the ping-pong, valid while the arrays, dt and `epoch` (bumped by
  // every setter that changes what a launch does) are unchanged
  unsigned epoch;
  hipStream_t gstream;
  hipEvent_t ev_in, ev_out;
  hipGraphExec_t gexec[3];
  const double* gQ;
  const double* gR;
  double gdt;
  unsigned gepoch;
};

// n / d for 0 <= n < 2^31 by a multiplication: with s = ceil(log2 d) and
// m = floor(2^32 (2^s - d) / d) + 1 the quotient is (mulhi(n, m) + n) >> s.
// (A division costs a wave about 25 dependent instructions, and a block's
// place in the visiting order takes four of them.)
struct DGDiv {
  unsigned m;
  int s;
};
inline DGDiv dg_div(unsigned d) {
  DGDiv v;
  v.s = 0;
  while ((1ull << v.s) < d) ++v.s;
  v.m = (unsigned)((((1ull << v.s) - d) << 32) / d + 1);
  return v;
}
__host__ __device__ __forceinline__ int dg_quot(int n, DGDiv v) {
  return (int)(((unsigned)(((unsigned long long)(unsigned)n * v.m) >> 32) + (unsigned)n) >> v.s);
}

// Elements of a wave of the one-thread-per-line kernels: as many as have their
// N^2 lines, and their pairs of y/z neighbour points, in 64 lanes.
constexpr int dg_line_elems(int N) { return N == 2 ? 16 : N == 3 ? 5 : N == 4 ? 4 : N == 5 ? 2 : 1; }

// How the arrays of a stage compare with the 256 MB last-level cache: within
// it; the three together beyond it; a state above 144 MiB, so that the next
// launch finds next to nothing of the new one there; a state above 400 MiB.
enum { DG_CACHED = 0, DG_BEYOND = 1, DG_STREAMED = 2, DG_HUGE = 3 };

// Order in which a neighbour-read stage launch visits its element blocks
// (kernel argument).  A block is EPB consecutive elements of one x-row (the
// last block of a row may be short).  Blocks are visited z-slab by z-slab
// (tz planes), inside a slab pencil by pencil along x (tx blocks), inside a
// pencil y-row by y-row, and inside that z-plane by z-plane, x fastest.
// Index order is the special case of whole-row pencils one plane deep.
struct DGOrder {
  int xcd;      // the XCDs share every `share` blocks, each taking a contiguous eighth
  int nxb;      // blocks per x-row
  int tx;       // blocks of a pencil along x
  int tz;       // element planes of a pencil along z
  int slab;     // blocks of a whole slab
  int share;    // blocks the XCDs share at a time: whole slabs, or all
  int full;     // whole shares
  int q;        // share / 8
  int size;     // DG_CACHED .. DG_HUGE
  DGDiv dslab, dq, dpen, drow, dtx;   // by slab, q, and a whole pencil's blocks, blocks per y-row, blocks along x
};

// Bytes of the arrays that a stage streams (state in and out, residual), and
// whether they exceed the 256 MB last-level cache.
inline int64_t dg_stage_bytes(const dg_ctx* c) {
  return 3 * DG_NF * (int64_t)sizeof(double) * c->E * c->N * c->N * c->N;
}
inline bool dg_beyond_cache(const dg_ctx* c) { return dg_stage_bytes(c) > ((int64_t)256 << 20); }

#define DG_PENCIL_Z 8   // planes of a pencil unless the caller chose

// Planes of a pencil in a launch of c (before the mesh's own height).
inline int dg_pencil_depth(const dg_ctx* c, bool line) {
  const bool chosen = c->pencil_z_set || c->order != DG_ORDER_PENCIL || !c->xcd_remap || !dg_beyond_cache(c);
  return chosen ? c->pencil_z : line ? 1 : 4;
}

// Visiting order and grid size of a neighbour-read launch with EPB elements
// per block; `line` for the one-thread-per-line kernels.
//
// Within the 256 MB last-level cache the XCDs take an eighth of the order
// each.  Where the arrays of a stage (state in and out, residual) exceed it
// they share every slab, and slabs are one (line kernels) or four planes deep
// unless the caller chose a depth: the XCDs then work on the same few planes
// and the neighbours of their parts come from HBM once.  With an eighth of
// the whole order each, they were spread over the mesh: k_stage_line 636
// against 534 us a stage at 48^3 p=4, 264 / 232 at 48^3 p=3, 1084 / 864 at
// 40^3 p=6; k_split 950 / 925 (4 planes) at 48^3 p=4; the viscous pair
// 2166 / 2125; k_stage_nb32 738 / 717.  Within the cache the eighths are as
// fast or faster (us a stage, sharing slabs of 8 planes / eighths: 32^3 p=3
// 66.7 / 65.2, 24^3 p=4 65.8 / 62.9, 16^3 p=5 38.7 / 37.6), by far where a slab
// has few blocks (4x4x1024 p=3 47.5 / 34.3, 8x8x512 p=3 87.7 / 63.2).
//
// A plane of few blocks gives an XCD next to nothing of its own neighbours:
// below `thin` blocks (6 per XCD) they share up to 512 blocks of whole slabs
// (a plane / 512 blocks: 4x4x8192 p=3, 4 blocks, 354 / 265; 8x8x2048 p=3, 16
// blocks, 313 / 268; 12x12x300 p=3, 36 blocks, 102 / 96; above, 100x2x300
// p=3, 50 blocks, 126 / 130; 12x12x300 p=4, 72 blocks, 203 / 212).  The
// adjoint's kernels, of which a CU holds one to three workgroups, do so only
// below 16 blocks (16x1x4096 p=3, 4 blocks, 206 / 193, p=5, 16 blocks, 1117 /
// 1165, 4x4x1024 p=6, 16 blocks, 373 / 416).
inline DGOrder dg_order(const dg_ctx* c, int epb, unsigned* grid, bool line = false, int thin = 48) {
  DGOrder o;
  const bool pencil = c->order == DG_ORDER_PENCIL;
  const bool hbm = dg_beyond_cache(c);
  o.xcd = c->xcd_remap;
  const int64_t state = dg_stage_bytes(c) / 3;
  o.size = !hbm ? DG_CACHED : state <= ((int64_t)144 << 20) ? DG_BEYOND : state <= ((int64_t)400 << 20) ? DG_STREAMED : DG_HUGE;
  o.nxb = (c->nx + epb - 1) / epb;
  const int px = pencil && c->pencil_x > 0 && c->pencil_x < c->nx ? c->pencil_x : c->nx;
  o.tx = (px + epb - 1) / epb;
  o.tz = !pencil || c->pencil_z < 1 ? 1 : dg_pencil_depth(c, line);
  if (o.tz > c->nz) o.tz = c->nz;
  *grid = (unsigned)((int64_t)o.nxb * c->ny * c->nz);
  o.slab = o.nxb * c->ny * o.tz;
  o.share = hbm ? o.slab : (int)*grid;
  if (hbm && o.nxb * c->ny < thin && o.slab < 512) o.share = o.slab * (512 / o.slab);
  if (o.share > (int)*grid) o.share = (int)*grid;
  o.full = (int)(*grid / (unsigned)o.share);
  o.q = o.share >> 3;
  o.dslab = dg_div(o.slab);
  o.dq = dg_div(o.q > 0 ? o.q : 1);
  o.dpen = dg_div(c->ny * o.tz * o.tx);
  o.drow = dg_div(o.tz * o.tx);
  o.dtx = dg_div(o.tx);
  return o;
}

// Workspace carve-up (byte offsets, each 256-aligned).
struct DGWorkspace {
  size_t trace_bytes;   // one face-trace buffer: 30 * N^2 * E doubles
  size_t off_trace0, off_trace1;
  size_t off_red;       // reduction partials
  size_t off_vjp;       // adjoint scratch: two state-sized buffers
  size_t off_q2;        // second state buffer of the neighbour-read path
  size_t off_visc_r;    // viscous terms only (mu > 0): the inviscid rate of a stage (5 N^3 E doubles)
  size_t off_visc_fv;   //   and the nodal viscous flux (12 N^3 E doubles) or its face traces (24 N^2 E)
  size_t total;
};
DGWorkspace dg_workspace_layout(const dg_ctx* c);

// Number of blocks used by the reduction kernels (fixed: the summation
// order, and hence the result, does not depend on the device).
#define DG_RED_BLOCKS 1024
#define DG_RED_VALS 8

// ---- launchers (return hipError_t as int) -------------------------------
// Face traces of Q on all six faces of every element.
int dg_launch_trace(const dg_ctx* c, const double* Q, double* T);
// RHS: R = dQ/dt using traces Tin of Q.
int dg_launch_rhs(const dg_ctx* c, const double* Q, const double* Tin, double* R);
// One RK stage in place; writes the traces of the updated Q to Tout when
// Tout != nullptr.
int dg_launch_stage(const dg_ctx* c, double* Q, double* res, const double* Tin,
                    double* Tout, double a, double b, double dt, int first);
// Neighbour-read stage: Qin -> Qout; mode 0 writes RR = dQ/dt, mode 1 the
// RK update (res = RR in place).
int dg_launch_stage_nb(const dg_ctx* c, const double* Qin, double* Qout, double* RR, int mode, double a, double b,
                       double dt, int first);
// Reductions: per-block partials then a fixed-order final pass into
// red[DG_RED_BLOCKS*DG_RED_VALS .. +DG_RED_VALS).
int dg_launch_reduce(const dg_ctx* c, const double* Q, double* red);
// Adjoint RHS.
int dg_launch_vjp(const dg_ctx* c, const double* Q, const double* gR, double* gQ, char* scratch);

// Reverse RK stage with neighbour reads: gQ += dt (dR/dQ)^T g in place and
// gres = a g.
int dg_launch_vjp_stage(const dg_ctx* c, const double* Q, const double* g, double* gQ, double* gres, double a,
                        double dt);

// Viscous terms (kern_visc.hip): the nodal viscous flux of Q into Fv (with
// `rate` also the inviscid rate of the standard form into R), then mode 0:
// R += the viscous rate; mode 1: the LSERK45 stage in place on Qu and res
// with R the inviscid rate of the stage.
int dg_launch_visc(const dg_ctx* c, const double* Q, double* Fv, double* R, double* Qu, double* res, int mode,
                   double a, double b, double dt, int first, bool rate);

// Kinetic-energy-preserving split form (kern_split.hip): mode 0 RR = dQ/dt;
// mode 1 the LSERK45 stage Qin -> Qout with res = RR in place; mode 2 the
// first stage.
int dg_launch_split(const dg_ctx* c, const double* Qin, double* Qout, double* RR, int mode, double a, double b,
                    double dt);

// Gradient of the kinetic-energy integral with respect to Q.
int dg_launch_ke_grad(const dg_ctx* c, const double* Q, double* G);

int dg_launch_axpy(const dg_ctx* c, int64_t n, const double* x, double b, const double* y, double* out);
int dg_launch_rk_reverse(const dg_ctx* c, int64_t n, const double* v, double dt, double a, const double* gtot,
                         double* gQ, double* gres);

// FP32 matrix-core variants.  Their trace buffers hold FP32 deviations
// [face][field][E][N^2] followed (256-aligned) by FP64 anchors [field][E];
// they fit in the same workspace regions as the FP64 traces.
int dg_launch_trace_f32(const dg_ctx* c, const double* Q, char* buf);
int dg_launch_rhs_f32(const dg_ctx* c, const double* Q, const char* tin, double* R);
int dg_launch_stage_f32(const dg_ctx* c, double* Q, double* res, const char* tin, char* tout, double a,
                        double b, double dt, int first);
bool dg_f32_supported(int N);
int dg_launch_stage_nb_f32(const dg_ctx* c, const double* Qin, double* Qout, double* RR, int mode, double a,
                           double b, double dt, int first);
