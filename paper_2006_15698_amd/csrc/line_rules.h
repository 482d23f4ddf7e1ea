// Which launches take the kernels with one thread per line (stage_line.h) and
// which those with one thread per node.  Host code.
//
// A wave that holds whole lines runs longer than the waves that hold its nodes
// one a thread, so lines need enough waves to fill the chip; and a wave of lines
// takes up to dg_line_elems(N) elements of ONE x-row, so on short rows its
// lanes idle where a node kernel with an element per workgroup loses nothing.
// "waves" below are blocks of up to dg_line_elems(N) elements; all figures are
// us a stage, lines / nodes.
#pragma once

#include "dg_internal.h"

// Blocks of up to epb elements of one x-row.
inline int64_t dg_row_blocks(const dg_ctx* c, int epb) { return (int64_t)((c->nx + epb - 1) / epb) * c->ny * c->nz; }

// Whether 100 nx >= percent times the elements that the row's blocks have room for.
inline bool dg_rows_filled(const dg_ctx* c, int epb, int percent) {
  return 100LL * c->nx >= (int64_t)percent * ((c->nx + epb - 1) / epb) * epb;
}

// Stage of the standard form (k_stage_line / k_stage_nb).  Up to 512 waves (two
// per CU) a stage takes as long as one workgroup: 8^3 p=3 7.5 / 6.5, 8^3 p=5
// 12.6 / 12.0, 8^3 p=7 18.9 / 17.6; above, 14^3 p=3 11.7 / 11.8, 10^3 p=5
// 13.9 / 15.8, 9^3 p=7 21.7 / 24.5.
inline bool dg_stage_line_pays(const dg_ctx* c) {
  const int N = c->N;
  if (N < 2) return false;
  const int64_t waves = dg_row_blocks(c, dg_line_elems(N));
  if (N == 3) {
    // Its node kernel reads one point per lane and is the slower at small
    // sizes (8^3 7.5 / 8.1), but takes 9 elements a block to the lines' 5:
    // where those fill the rows better and the arrays are in the cache the
    // node kernel is ahead from 4096 waves on (36^3 54.2 / 51.0, 6x82x82 11%;
    // 24^3, rows filled better by the lines, 19.7 / 22.3; beyond the cache
    // lines 8x8x2048 167 / 173).
    const int line = (c->nx + 4) / 5 * 5, node = (c->nx + 8) / 9 * 9;
    return line <= node || waves <= 4096 || dg_beyond_cache(c);
  }
  if (waves <= 512) return false;
  // N = 4: 2048 waves are resident at once; a second round of them ends well
  // after the node kernel's workgroups, of which more fit (full rows in the
  // cache: 16^3, 1024 waves, 12.2 / 13.7, 21^3 25.7 / 23.8, 24^3 32.9 / 31.4;
  // 28^3, 5488 waves, even, 30^3 58.9 / 59.6).
  if (N == 4 && waves > 2048 && waves <= 4608 && dg_rows_filled(c, 4, 90) && !dg_beyond_cache(c)) return false;
  // N = 8: one wave per SIMD, 1024 at once; up to three rounds a last one that
  // is nearly empty costs what the lines gain (10^3 24.4 / 29.6, 5x16x16
  // 37.9 / 34.9, 13x13x12 5% and 14x14x13 7% behind, 15x15x16 even, 1x64x64 77 /
  // 87, 17x16x17 12% ahead).
  if (N == 8 && waves > 1024 && waves <= 3072) return false;
  return true;
}

// Split form (k_split_line / k_split, one element per workgroup).
inline bool dg_split_line_pays(const dg_ctx* c) {
  const int N = c->N, nx = c->nx;
  if (N < 2) return false;
  const int64_t waves = dg_row_blocks(c, dg_line_elems(N));
  switch (N) {
    case 2: return nx > 1 || waves <= 2048;   // 1x64x64 18.2 / 14.9, 1x16x4096 205 / 132; 1x24x24 0.71, 2x69x69 0.76
    case 3: return nx > 1 || waves <= 512;    // 1x64x64 25.2 / 18.3, 1x39x39 18% behind, 1x24x24 even; 2x39x39 0.93
    case 4:
      // 9^3 10.4 / 9.3, 12x10x11 12.6 / 13.1; rows of one or two elements
      // 1x64x64 33.1 / 24.0, 2x35x35 13% behind, 2x45x45, not yet a second round,
      // 13% ahead, 2x48x48 27.3 / 25.2, 2x77x77 2% ahead; 3x20x20 even
      return waves > 384 && nx > 1 && (nx > 2 || (waves > 1536 && waves <= 2048) || waves > 4096);
    case 5:
      // 10^3 15.4 / 13.8, 11^3 16.5 / 16.4, 12^3 17.3 / 18.4; with half-empty
      // blocks 1x64x64 40.6 / 33.0, 3x20x20 16.2 / 14.5, 3x45x45 even; just over
      // the 2048 waves of one round 2x48x48 38 / 36, 18x17x17 5% ahead again
      return waves > 704 && nx > 1 && (nx != 3 || waves > 4096) && !(waves > 2048 && waves <= 2400);
    case 6: return waves > 512;   // 8^3 16.6 / 14.8, 9x8x8 17.8 / 19.0
    case 7: return waves > 384;   // 7x7x8 18.2 / 19.0 at 392
    default: return waves > 512;  // 8^3 24.9 / 22.8, 9x8x8 26.1 / 31.5
  }
}

// Viscous stage (k_visc_line + k_visc_update / k_visc_flux + k_visc_apply, one
// element per workgroup).  The node pair hands a nodal flux of 12 values from
// launch to launch; while that, the state, the rate and the residual (216
// bytes a node) fit the cache it is close to the lines and any idle lane
// decides, beyond it the lines gain 30 to 40%.
inline bool dg_visc_line_pays(const dg_ctx* c) {
  const int N = c->N, nx = c->nx;
  if (N < 2) return false;
  const int64_t waves = dg_row_blocks(c, dg_line_elems(N));
  const bool cached = 216 * c->E * N * N * N <= (int64_t)256 << 20;
  switch (N) {
    case 2: return nx > 2 || waves <= 512;   // 1x64x64 43 / 25, 2x155x155 10% behind, 2x20x20 9% and 3x57x57 24% ahead
    case 3: return nx > 2 || waves <= 256;   // 1x64x64 54 / 30, 2x48x48 38.3 / 35.1; 3x22x22 12% ahead
    case 4:
      // 12x14x14 27.8 / 27.0, 16x13x14 28.5 / 29.8; 5x49x49 17% and 6x45x45 5%
      // behind, 17x16x16 9% ahead; beyond the cache 2x126x126 even, 5x80x80 15%
      // ahead, 1x179x179 73% behind
      return waves > 640 && (cached ? dg_rows_filled(c, 4, 85) : nx > 2);
    case 5:
      // 11x10x10 29.9 / 28.9, 10x11x12 30.7 / 32.1; 3x45x45 12%, 5x35x35 and
      // 7x17x17 and 9x15x15 5% behind; beyond the cache 3x103x103 22% ahead, 1x126x126 6% behind
      return waves > 600 && (cached ? dg_rows_filled(c, 2, 92) : nx > 1);
    // a block's 36 lines leave two fifths of the lanes idle: 17^2x18 140 / 137, 18^2x19 162 / 180
    case 6: return waves > 5632;
    case 7: return waves > 512;    // 8x7x8 32.5 / 32.7 at 448, 9^3 44 / 48
    default: return waves > 2816;  // 14x14x13 182 / 177, 15x14x15 225 / 235 (registers and LDS leave few waves)
  }
}

// Batched stage of one degree (k_batch_degree / k_batch_nodes), N = 2..6, of
// `items` blocks: from one per CU on (one mesh 6^3 p=3, 72 items, 9.6 / 8.9,
// p=4 11.3 / 10.4; two 6^3 p=3, 144, 9.7 / 9.2; four 4^3 p=5, 256, even; four
// 6^3 p=3, 288, 8% and eight 4^3 p=4, 256, 9% ahead).  At N = 3 lines are ahead at
// every size (one 4^3 3%).
inline bool dg_batch_line_pays(int N, int items) { return N == 3 || items >= 256; }

// Variable-degree stage of one group (k_varp_line / k_varp), N = 2..7.  At N = 2
// and 3 lines are ahead at every size (512 elements 6.7 / 8.1 and 7.9 / 8.3); at
// N = 4..7 from two waves per CU on (128 waves of N = 4 8.7 / 7.6, 784 11.7 /
// 12.9; N = 5 256 10.8 / 9.6, 792 12.9 / 15.7; N = 6 512 13.5 / 12.6, 900 13.5 /
// 15.8; N = 7 448 14.7 / 15.0); at N = 8, where a wave takes a SIMD's registers
// and the tables' scalar registers spill, at none (1728 elements 59.8 / 50.1).
// N = 4: 1792 waves are resident at once, and a second round of a few costs more
// than the lines gain (1805 waves 0.98, 2000 24.3 / 23.2, 2x2x2048 24.6 / 22.3,
// 2310 even).
inline bool dg_varp_line_pays(int N, int count) {
  if (N < 2 || N > 7) return false;
  if (N <= 3) return true;
  const int epb = dg_line_elems(N), waves = (count + epb - 1) / epb;
  return waves > 512 && !(N == 4 && waves > 1792 && waves <= 2112);
}

// Adjoint of the right-hand side (k_vjp_line / k_vjp_nb).  Below N = 7 the node
// kernel is the faster one at every size (32^3 p=3 111 / 104, 48^3 p=4 867 / 801,
// 32^3 p=5 657 / 583): the transposed Lax-Friedrichs Jacobians hold both, and it
// too forms them one face point a thread.  At N = 7 and 8 its LDS (95 and 139 KB
// an element) leaves one workgroup on a CU (24^3 p=6 341 / 581, 24^3 p=7 779 /
// 1781); at N = 8 it is ahead in the product while there is no more than half of
// one (4^3 19.1 / 17.5, 5^3 19.7 / 17.6, 180 elements 22.0 / 26.3; N = 7 4^3 even),
// but not in the reverse stage (4^3 24.2 / 28.8).
inline bool dg_vjp_line_pays(const dg_ctx* c, bool reverse_stage) {
  return c->N == 7 || (c->N == 8 && (reverse_stage || c->E > 128));
}
