// Host check of the rules that choose between the kernels with a thread per
// line and those with a thread per node (line_rules.h), at sizes on both sides
// of each line.  Exit status 0 and "ok" on success.
#include <cstdio>

#include "line_rules.h"

struct Case {
  const char* form;
  int N, nx, ny, nz;
  bool line;
};

static dg_ctx mesh(const Case& k) {
  dg_ctx c{};
  c.nx = k.nx; c.ny = k.ny; c.nz = k.nz; c.N = k.N;
  c.E = (int64_t)k.nx * k.ny * k.nz;
  c.order = DG_ORDER_PENCIL; c.pencil_x = 16; c.pencil_z = 8; c.xcd_remap = 1;
  return c;
}

static int fails = 0;
template <class F>
static void check(const char* form, F&& pays, std::initializer_list<Case> cases) {
  for (const Case& k : cases) {
    const dg_ctx c = mesh(k);
    if (pays(&c) == k.line) continue;
    ++fails;
    printf("%s N=%d %dx%dx%d: %s expected\n", form, k.N, k.nx, k.ny, k.nz, k.line ? "lines" : "nodes");
  }
}

int main() {
  check("stage", dg_stage_line_pays,
        {{"", 1, 64, 64, 64, false},
         {"", 2, 16, 16, 32, false}, {"", 2, 16, 16, 33, true}, {"", 2, 1, 64, 64, true},
         // 9 elements a block fill rows of 36, 27, 9, 6 better than 5 do
         {"", 3, 36, 36, 36, false}, {"", 3, 27, 27, 27, false}, {"", 3, 6, 82, 82, false}, {"", 3, 16, 16, 128, false},
         {"", 3, 1, 1, 1, true}, {"", 3, 8, 8, 8, true}, {"", 3, 9, 30, 30, true}, {"", 3, 28, 28, 28, true},
         {"", 3, 40, 40, 40, true}, {"", 3, 45, 45, 45, true}, {"", 3, 8, 8, 2048, true},
         {"", 4, 8, 16, 16, false}, {"", 4, 12, 14, 14, true}, {"", 4, 16, 16, 32, true}, {"", 4, 16, 16, 33, false},
         {"", 4, 24, 24, 24, false}, {"", 4, 26, 26, 25, false}, {"", 4, 24, 26, 26, false}, {"", 4, 28, 28, 28, true}, {"", 4, 30, 30, 30, true},
         {"", 4, 32, 32, 32, true}, {"", 4, 1, 64, 64, true}, {"", 4, 9, 37, 37, true}, {"", 4, 48, 48, 48, true},
         {"", 5, 8, 8, 16, false}, {"", 5, 8, 8, 17, true}, {"", 6, 8, 8, 8, false}, {"", 6, 8, 8, 9, true},
         {"", 7, 8, 8, 8, false}, {"", 7, 8, 8, 9, true},
         {"", 8, 8, 8, 8, false}, {"", 8, 8, 8, 9, true}, {"", 8, 8, 8, 16, true}, {"", 8, 5, 16, 16, false},
         {"", 8, 16, 16, 12, false}, {"", 8, 16, 16, 13, true}, {"", 8, 1, 64, 64, true}, {"", 8, 20, 20, 20, true}});
  check("split", dg_split_line_pays,
        {{"", 1, 64, 64, 64, false},
         {"", 2, 1, 64, 64, false}, {"", 2, 1, 1, 4096, false}, {"", 2, 1, 24, 24, true}, {"", 2, 2, 69, 69, true},
         {"", 2, 1, 1, 1, true}, {"", 2, 33, 5, 4, true},
         {"", 3, 1, 64, 64, false}, {"", 3, 1, 39, 39, false}, {"", 3, 2, 39, 39, true}, {"", 3, 7, 5, 4, true},
         {"", 4, 9, 9, 9, false}, {"", 4, 12, 12, 12, true}, {"", 4, 1, 64, 64, false}, {"", 4, 2, 35, 35, false},
         {"", 4, 2, 45, 45, true}, {"", 4, 2, 48, 48, false}, {"", 4, 2, 77, 77, true}, {"", 4, 3, 20, 20, true},
         {"", 4, 1, 16, 4096, false},
         {"", 5, 10, 10, 10, false}, {"", 5, 12, 12, 12, true}, {"", 5, 1, 64, 64, false}, {"", 5, 3, 20, 20, false},
         {"", 5, 3, 73, 73, true}, {"", 5, 2, 48, 48, false}, {"", 5, 18, 17, 17, true}, {"", 5, 48, 48, 48, true},
         {"", 6, 8, 8, 8, false}, {"", 6, 9, 9, 9, true}, {"", 7, 7, 7, 7, false}, {"", 7, 7, 7, 8, true},
         {"", 8, 8, 8, 8, false}, {"", 8, 9, 8, 8, true}});
  check("viscous", dg_visc_line_pays,
        {{"", 1, 64, 64, 64, false},
         {"", 2, 1, 64, 64, false}, {"", 2, 2, 48, 48, false}, {"", 2, 2, 20, 20, true}, {"", 2, 3, 57, 57, true},
         {"", 2, 1, 16, 4096, false}, {"", 2, 33, 5, 4, true},
         {"", 3, 1, 24, 24, false}, {"", 3, 2, 48, 48, false}, {"", 3, 3, 22, 22, true}, {"", 3, 7, 5, 4, true},
         {"", 4, 12, 14, 14, false}, {"", 4, 16, 13, 14, true}, {"", 4, 2, 48, 48, false}, {"", 4, 5, 49, 49, false},
         {"", 4, 17, 16, 16, true}, {"", 4, 5, 80, 80, true}, {"", 4, 1, 179, 179, false}, {"", 4, 48, 48, 48, true},
         {"", 5, 10, 11, 10, false}, {"", 5, 12, 12, 12, true}, {"", 5, 3, 45, 45, false}, {"", 5, 5, 35, 35, false}, {"", 5, 9, 15, 15, false},
         {"", 5, 3, 103, 103, true}, {"", 5, 1, 126, 126, false}, {"", 5, 48, 48, 48, true},
         {"", 6, 17, 17, 18, false}, {"", 6, 18, 18, 19, true}, {"", 6, 2, 48, 48, false},
         {"", 7, 8, 8, 8, false}, {"", 7, 9, 8, 8, true}, {"", 8, 14, 14, 13, false}, {"", 8, 15, 14, 15, true}});
  for (int N = 2; N <= 6; ++N)
    for (int items : {1, 72, 255, 256, 4000})
      if (dg_batch_line_pays(N, items) != (N == 3 || items > 255)) {
        ++fails;
        printf("batch N=%d items %d\n", N, items);
      }
  check("adjoint", [](const dg_ctx* c) { return dg_vjp_line_pays(c, false); },
        {{"", 6, 48, 48, 48, false}, {"", 7, 1, 1, 1, true}, {"", 8, 4, 4, 8, false}, {"", 8, 43, 3, 1, true},
         {"", 8, 6, 6, 6, true}});
  check("reverse stage", [](const dg_ctx* c) { return dg_vjp_line_pays(c, true); },
        {{"", 6, 48, 48, 48, false}, {"", 7, 1, 1, 1, true}, {"", 8, 1, 1, 1, true}, {"", 8, 6, 6, 6, true}});
  struct Group { int N, count; bool line; };
  for (Group g : {Group{1, 9999, false}, Group{2, 1, true}, Group{3, 1, true}, Group{4, 2048, false}, Group{4, 2049, true},
                  Group{4, 7168, true}, Group{4, 7169, false}, Group{4, 8000, false}, Group{4, 8448, false},
                  Group{4, 8449, true}, Group{5, 1024, false}, Group{5, 1025, true}, Group{6, 512, false},
                  Group{6, 513, true}, Group{7, 512, false}, Group{7, 513, true}, Group{8, 9999, false}})
    if (dg_varp_line_pays(g.N, g.count) != g.line) {
      ++fails;
      printf("variable degree N=%d count %d\n", g.N, g.count);
    }
  if (!fails) printf("ok\n");
  return fails != 0;
}
