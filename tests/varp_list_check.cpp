// Host check of the variable-degree builder's element lists where the arrays
// of a stage exceed the last-level cache (each XCD's part of a list takes an
// eighth of every one-plane slab in turn, but for planes of few cells), compiled with the builder's own
// source as varp_mesh_check.cpp is.  Every element stands once, in its group's
// range; a group's elements of one plane and part follow one another; and an
// eighth of a wide mesh's list holds an eighth of every plane, within one.
// Exit status 0 and "ok" on success.
#include "varp_api.cpp"

#include <cstdio>
#include <random>

static int fails = 0;
#define CHECK(cond, ...)          \
  do {                            \
    if (!(cond)) {                \
      if (fails++ < 20) {         \
        printf(__VA_ARGS__);      \
        printf("\n");             \
      }                           \
    }                             \
  } while (0)

static void check(int nx, int ny, int nz, double refined, int plo, int phi, bool beyond) {
  std::mt19937 rng(nx * 131 + nz);
  std::vector<int> ref(nx * ny * nz), plane;
  for (int c = 0; c < nx * ny * nz; ++c) {
    ref[c] = std::uniform_real_distribution<double>(0, 1)(rng) < refined;
    for (int k = 0; k < (ref[c] ? 8 : 1); ++k) plane.push_back(c / (nx * ny));
  }
  const int E = (int)plane.size();
  std::vector<int> deg(E);
  for (int& d : deg) d = std::uniform_int_distribution<int>(plo, phi)(rng);
  const double L[3] = {1.0, 0.8, 1.2};
  dg_varp* v = dg_varp_create_refined(nx, ny, nz, ref.data(), deg.data(), L, 1.4);
  if (!v) {
    printf("create failed: %s\n", dg_last_error());
    ++fails;
    return;
  }
  CHECK((120 * v->T > ((int64_t)256 << 20)) == beyond, "%dx%dx%d: %lld nodes", nx, ny, nz, (long long)v->T);
  std::vector<int> seen(E, 0);
  for (int N = 1; N <= DG_VARP_MAXN; ++N)
    for (int lev = 0; lev < 2; ++lev) {
      const int first = v->first[N][lev], count = v->count[N][lev];
      std::vector<std::vector<int>> per(8, std::vector<int>(nz, 0));
      std::vector<int> total(nz, 0);
      for (int i = 0; i < count; ++i) {
        const int e = v->list[first + i];
        CHECK(e >= 0 && e < E, "entry %d out of range", e);
        if (e < 0 || e >= E) continue;
        ++seen[e];
        CHECK(deg[e] + 1 == N && v->level[e] == lev, "element %d in the wrong group", e);
        ++total[plane[e]];
        ++per[(int64_t)i * 8 / count][plane[e]];
      }
      // planes of few cells: the order of eight-plane slabs stays whole
      if (beyond && nx * ny < 48)
        for (int i = 1; i < count; ++i)
          CHECK(plane[v->list[first + i]] / 8 >= plane[v->list[first + i - 1]] / 8, "%dx%dx%d N=%d: slab order at %d", nx, ny,
                nz, N, i);
      // parts of near-equal length: their borders drift by less than one
      // element a plane, here at most a plane's own eighth
      if (beyond && refined == 0.0 && plo == phi && nx * ny >= 64)
        for (int x = 0; x < 8; ++x)
          for (int z = 0; z < nz; ++z)
            CHECK(per[x][z] * 8 >= total[z] - 8 * nz && per[x][z] * 8 <= total[z] + 8 * nz, "part %d plane %d: %d of %d", x, z,
                  per[x][z], total[z]);
    }
  for (int e = 0; e < E; ++e) CHECK(seen[e] == 1, "element %d listed %d times", e, seen[e]);
  dg_varp_destroy(v);
}

int main() {
  check(24, 22, 20, 0.15, 5, 7, true);
  check(24, 22, 20, 0.15, 0, 7, true);
  check(3, 2, 900, 0.0, 7, 7, true);
  check(1, 1, 5000, 0.1, 6, 7, true);
  check(130, 131, 1, 0.0, 5, 5, true);
  check(67, 61, 9, 0.0, 3, 3, true);
  check(40, 40, 40, 0.08, 2, 5, true);
  check(16, 16, 16, 0.15, 1, 4, false);
  if (!fails) printf("ok\n");
  return fails != 0;
}
