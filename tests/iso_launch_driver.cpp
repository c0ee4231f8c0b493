// The launches of iso-parametric blocks (iso_next): over blocks from none to 2^31
// elements they cover every element once, in order, each with fewer than 2^32
// threads.  Built and run by tests/test_iso_launches.py with the host compiler only.
#include <cstdio>
#include <vector>

#include "../paper_2604_04644_amd/csrc/shp_internal.hpp"

using namespace shp;

static int fails = 0;
#define CHECK(c)                                               \
  do {                                                         \
    if (!(c)) {                                                \
      std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
      ++fails;                                                 \
    }                                                          \
  } while (0)

// the block entry of work-group w, as the kernel finds it
static int entry(const IsoMesh& m, long long w) {
  int i = 0;
  for (int j = 1; j < ISO_MAX_BLK; ++j) i += w >= m.wg0[j] ? 1 : 0;
  return i;
}

static int run(int P, const std::vector<long long>& ne) {
  const IsoShape sh = iso_shape(P);
  const int n = (int)ne.size();
  std::vector<int> blk(n);
  std::vector<long long> done(n, 0);  // elements covered so far
  for (int i = 0; i < n; ++i) blk[i] = 1000 + n - i;
  IsoMesh m{};
  int launches = 0, last = -1;
  for (IsoCursor c; iso_next(m, c, P, n, blk.data(), ne.data()); ++launches) {
    const long long wgs = m.wg0[m.nblk];
    CHECK(m.nblk >= 1 && m.nblk <= ISO_MAX_BLK && wgs > 0);
    CHECK(wgs * sh.NT < (1LL << 32));
    for (int k = 0; k < m.nblk; ++k) {
      const long long w0 = k == 0 ? 0 : m.wg0[k], w1 = m.wg0[k + 1];
      CHECK(w1 > w0);
      CHECK(entry(m, w0) == k && entry(m, w1 - 1) == k);
      const int b = 1000 + n - m.blk[k];
      CHECK(b >= last && b < n);
      last = b;
      // first element of the first work-group, elements of the last one
      CHECK((w0 - m.wg0[k]) * sh.E == done[b]);
      const long long e1 = (w1 - m.wg0[k]) * sh.E;
      CHECK((w1 - 1 - m.wg0[k]) * sh.E < ne[b]);
      done[b] = e1 < ne[b] ? e1 : ne[b];
    }
  }
  for (int i = 0; i < n; ++i) CHECK(done[i] == ne[i]);
  return launches;
}

int main() {
  const long long big = 1LL << 31;
  for (int P = 1; P <= MAX_P; ++P) {
    const IsoShape sh = iso_shape(P);
    const long long lim = 0xffffffffLL / sh.NT, full = lim * sh.E;  // elements of a full launch
    CHECK(run(P, {}) == 0);
    CHECK(run(P, {0}) == 0);
    CHECK(run(P, {1}) == 1);
    CHECK(run(P, {full}) == 1);
    CHECK(run(P, {full + 1}) == 2);
    CHECK(run(P, {full - 1, 1, 1}) == 2);
    CHECK(run(P, {0, full / 2, 0, full, 0, 3, 0}) == 2);
    CHECK(run(P, {big, 0, big, 5}) >= 2);
    std::vector<long long> many(MAX_BLK);
    for (int i = 0; i < MAX_BLK; ++i) many[i] = i % 5 == 2 ? 0 : 1 + 7 * i;
    run(P, many);
    many[20] = big;
    run(P, many);
  }
  std::printf("%s: %d failures\n", fails ? "FAILED" : "ok", fails);
  return fails ? 1 : 0;
}
