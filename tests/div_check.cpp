// Host check of dg_quot (dg_internal.h), the multiplication that stands for
// n / d in the visiting order: every divisor up to 4096 and a spread of
// larger ones, at n around every power of two, around multiples of d and at
// the end of the range; and of the line kernel's LDS index (stage_line.h):
// the nodes of a block fill their places one to one, rows whole and at even
// places where pairs are read; of the visiting order with shared slabs; and of the shared windows of a list.  Exit status 0 and "ok" on success.
#include <cstdio>
#include <vector>

#include "dg_internal.h"
#include "stage_line.h"

template <int N, int EPB>
static bool lds_map() {
  using L = dgdev::LineLds<N>;
  const int nodes = EPB * N * N * N;
  std::vector<int> hits(nodes, 0);
  for (int g = 0; g < nodes; ++g) {
    const int a = L::node(g);
    if (a < 0 || a >= nodes || hits[a]++) return false;
    if (g % N && a != L::node(g - 1) + 1) return false;
    if (N % 2 == 0 && g % 2 == 0 && a % 2) return false;
    const int n = g % (N * N * N);
    if (a != L::row(g / (N * N * N), n / (N * N), n / N % N) + n % N) return false;
  }
  return true;
}

// With the slabs shared among the XCDs (the line kernel, and every kernel
// beyond the last-level cache) each element is still covered exactly once.
template <int EPB>
static bool shared_slabs(int nx, int ny, int nz, int N, bool line, int pencil_z) {
  dg_ctx c{};
  c.nx = nx; c.ny = ny; c.nz = nz; c.N = N;
  c.E = (int64_t)nx * ny * nz;
  c.order = DG_ORDER_PENCIL; c.pencil_x = 16; c.pencil_z = 8; c.xcd_remap = 1;
  if (pencil_z) { c.pencil_z = pencil_z; c.pencil_z_set = 1; }
  DGTables tb{};
  tb.nx = nx; tb.ny = ny; tb.nz = nz; tb.E = (int)c.E;
  unsigned grid;
  const DGOrder o = dg_order(&c, EPB, &grid, line);
  std::vector<char> hits(c.E, 0);
  for (unsigned w = 0; w < grid; ++w) {
    const dgdev::Block b = dgdev::block_of<EPB>(tb, o, (int)w, (int)grid);
    if (b.ne < 1 || b.ne > EPB || b.x0 < 0 || b.x0 + b.ne > nx || b.y < 0 || b.y >= ny || b.z < 0 || b.z >= nz ||
        b.e0 != (b.z * ny + b.y) * nx + b.x0)
      return false;
    for (int k = 0; k < b.ne; ++k)
      if (hits[b.e0 + k]++) return false;
  }
  for (char h : hits)
    if (h != 1) return false;
  return true;
}

// The windows of items that the XCDs share cover every block once.
static bool windows(int nblk, int per) {
  std::vector<int> hits(nblk, 0);
  for (int w = 0; w < nblk; ++w) {
    const int i = dgdev::xcd_window(w, nblk, per);
    if (i < 0 || i >= nblk || hits[i]++) return false;
  }
  return true;
}

int main() {
  for (int nblk : {1, 7, 8, 9, 1023, 1024, 1025, 2047, 2048, 5000, 441031})
    for (int per : {1, 3, 128})
      if (!windows(nblk, per)) {
        printf("window of %d per XCD over %d blocks\n", per, nblk);
        return 1;
      }
  for (int nx : {1, 3, 16, 31})
    for (int ny : {1, 5, 24})
      for (int nz : {1, 2, 7, 25})
        for (int pz : {0, 1, 3})
          for (bool line : {false, true})
            for (int N : {2, 8})
              if (!(shared_slabs<1>(nx, ny, nz, N, line, pz) && shared_slabs<4>(nx, ny, nz, N, line, pz) &&
                    shared_slabs<5>(nx, ny, nz, N, line, pz))) {
                printf("order %d %d %d N %d line %d planes %d\n", nx, ny, nz, N, (int)line, pz);
                return 1;
              }
  if (!(lds_map<2, 16>() && lds_map<3, 5>() && lds_map<4, 4>() && lds_map<5, 2>() && lds_map<6, 1>() &&
        lds_map<7, 1>() && lds_map<8, 1>())) {
    printf("LDS map\n");
    return 1;
  }
  const long long top = 0x7fffffffLL;
  long long checks = 0;
  for (long long d = 1; d <= top; d = d < 4096 ? d + 1 : d + d / 7 + 1) {
    const DGDiv v = dg_div((unsigned)d);
    auto ok = [&](long long n) {
      if (n < 0 || n > top) return true;
      ++checks;
      if (dg_quot((int)n, v) == n / d) return true;
      printf("%lld / %lld gave %d\n", n, d, dg_quot((int)n, v));
      return false;
    };
    for (int b = 0; b < 32; ++b)
      for (long long e = -2; e <= 2; ++e)
        if (!ok((1LL << b) + e)) return 1;
    for (long long k : {1LL, 2LL, 3LL, top / d / 3, top / d / 2, top / d - 1, top / d, top / d + 1})
      for (long long e = -1; e <= 1; ++e)
        if (!ok(k * d + e)) return 1;
    if (!ok(top) || !ok(0)) return 1;
  }
  printf("%lld ok\n", checks);
  return 0;
}
