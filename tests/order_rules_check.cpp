// Host check of what dg_order (dg_internal.h) decides for a mesh: how many
// blocks the XCDs share at a time.  Usage: order_rules_check; exit status 0
// and "ok" on success.
#include <cstdio>
#include <vector>

#include "dg_internal.h"
#include "stage_nb.h"

static dg_ctx mesh(int nx, int ny, int nz, int N) {
  dg_ctx c{};
  c.nx = nx; c.ny = ny; c.nz = nz; c.N = N;
  c.E = (int64_t)nx * ny * nz;
  c.order = DG_ORDER_PENCIL; c.pencil_x = 16; c.pencil_z = 8; c.xcd_remap = 1;
  return c;
}

static int fails = 0;
#define CHECK(cond, ...)                  \
  do {                                    \
    if (!(cond)) {                        \
      printf(__VA_ARGS__);                \
      printf(" (%s)\n", #cond);             \
      ++fails;                            \
    }                                     \
  } while (0)

// Every block of the launch once.
static bool covers(const dg_ctx& c, const DGOrder& o, unsigned grid, int epb) {
  DGTables tb{};
  tb.nx = c.nx; tb.ny = c.ny; tb.nz = c.nz; tb.E = (int)c.E;
  std::vector<char> hits(c.E, 0);
  for (unsigned w = 0; w < grid; ++w) {
    const dgdev::Block b = epb == 1   ? dgdev::block_of<1>(tb, o, (int)w, (int)grid)
                           : epb == 2 ? dgdev::block_of<2>(tb, o, (int)w, (int)grid)
                           : epb == 4 ? dgdev::block_of<4>(tb, o, (int)w, (int)grid)
                           : epb == 5 ? dgdev::block_of<5>(tb, o, (int)w, (int)grid)
                                      : dgdev::block_of<16>(tb, o, (int)w, (int)grid);
    for (int k = 0; k < b.ne; ++k)
      if (b.e0 + k < 0 || b.e0 + k >= c.E || hits[b.e0 + k]++) return false;
  }
  for (char h : hits)
    if (h != 1) return false;
  return true;
}

int main() {
  struct Mesh { int nx, ny, nz, N; };
  // arrays of a stage within the 256 MB cache: an eighth of the order per XCD
  for (Mesh m : {Mesh{32, 32, 32, 4}, Mesh{4, 4, 1024, 4}, Mesh{24, 24, 24, 5}, Mesh{2, 2, 2048, 5}, Mesh{16, 16, 128, 3}})
    for (bool line : {true, false}) {
      const dg_ctx c = mesh(m.nx, m.ny, m.nz, m.N);
      unsigned grid;
      const int epb = dg_line_elems(m.N);
      const DGOrder o = dg_order(&c, epb, &grid, line);
      CHECK(o.share == (int)grid, "%dx%dx%d N=%d line=%d share %d of %u", m.nx, m.ny, m.nz, m.N, line, o.share, grid);
      CHECK(covers(c, o, grid, epb), "%dx%dx%d N=%d line=%d", m.nx, m.ny, m.nz, m.N, line);
    }
  // beyond it: a slab at a time where a plane gives every XCD several blocks,
  // else some hundreds of blocks of whole slabs
  for (Mesh m : {Mesh{40, 40, 40, 4}, Mesh{48, 48, 48, 5}, Mesh{20, 20, 100, 5}, Mesh{16, 16, 600, 5}})
    for (bool line : {true, false}) {
      const dg_ctx c = mesh(m.nx, m.ny, m.nz, m.N);
      unsigned grid;
      const int epb = dg_line_elems(m.N);
      const DGOrder o = dg_order(&c, epb, &grid, line);
      CHECK(o.share == o.slab && o.slab == o.nxb * m.ny * (line ? 1 : 4), "%dx%dx%d N=%d line=%d share %d slab %d", m.nx,
            m.ny, m.nz, m.N, line, o.share, o.slab);
      CHECK(covers(c, o, grid, epb), "%dx%dx%d N=%d line=%d", m.nx, m.ny, m.nz, m.N, line);
    }
  for (Mesh m : {Mesh{4, 4, 8192, 4}, Mesh{8, 8, 2048, 4}, Mesh{16, 1, 4096, 5}, Mesh{2, 2, 2048, 7}, Mesh{4, 8, 4000, 5},
                 Mesh{1, 1, 6000, 8}, Mesh{7, 3, 1500, 6}})
    for (bool line : {true, false}) {
      const dg_ctx c = mesh(m.nx, m.ny, m.nz, m.N);
      unsigned grid;
      const int epb = dg_line_elems(m.N);
      const DGOrder o = dg_order(&c, epb, &grid, line);
      CHECK(o.share >= 256 && o.share <= 512 && o.share % o.slab == 0, "%dx%dx%d N=%d line=%d share %d slab %d", m.nx,
            m.ny, m.nz, m.N, line, o.share, o.slab);
      CHECK(covers(c, o, grid, epb), "%dx%dx%d N=%d line=%d", m.nx, m.ny, m.nz, m.N, line);
    }
  // the adjoint's limit
  for (int nx : {16, 15}) {
    const dg_ctx c = mesh(nx, 1, 4096, 6);
    unsigned grid;
    const DGOrder o = dg_order(&c, 1, &grid, false, 16);
    CHECK(nx < 16 ? o.share > 256 : o.share == o.slab, "%dx1x4096 share %d slab %d", nx, o.share, o.slab);
    CHECK(covers(c, o, grid, 1), "%dx1x4096", nx);
  }
  // size classes: three arrays against the cache, then the state alone
  {
    struct Case { Mesh m; int size; };
    for (Case k : {Case{{32, 32, 32, 4}, DG_CACHED}, Case{{16, 16, 16, 8}, DG_CACHED}, Case{{17, 17, 17, 8}, DG_BEYOND},
                   Case{{36, 36, 36, 4}, DG_BEYOND}, Case{{24, 24, 24, 6}, DG_BEYOND}, Case{{72, 72, 72, 2}, DG_BEYOND},
                   Case{{48, 48, 48, 3}, DG_BEYOND}, Case{{31, 31, 31, 5}, DG_BEYOND}, Case{{22, 22, 22, 7}, DG_BEYOND},
                   Case{{39, 39, 39, 4}, DG_STREAMED}, Case{{26, 26, 26, 6}, DG_STREAMED}, Case{{32, 32, 32, 5}, DG_STREAMED},
                   Case{{80, 80, 80, 2}, DG_STREAMED}, Case{{24, 24, 24, 7}, DG_STREAMED}, Case{{48, 48, 48, 5}, DG_HUGE},
                   Case{{36, 36, 36, 7}, DG_HUGE}, Case{{40, 40, 40, 7}, DG_HUGE}}) {
      const dg_ctx c = mesh(k.m.nx, k.m.ny, k.m.nz, k.m.N);
      unsigned grid;
      const DGOrder o = dg_order(&c, dg_line_elems(k.m.N), &grid, true);
      CHECK(o.size == k.size, "%dx%dx%d N=%d size %d", k.m.nx, k.m.ny, k.m.nz, k.m.N, o.size);
    }
  }
  // never more than the launch
  {
    dg_ctx c = mesh(1, 1, 5, 8);
    c.order = DG_ORDER_LINEAR;
    unsigned grid;
    const DGOrder o = dg_order(&c, 1, &grid, true);
    CHECK(o.share <= (int)grid && covers(c, o, grid, 1), "1x1x5 share %d", o.share);
  }
  if (!fails) printf("ok\n");
  return fails != 0;
}
