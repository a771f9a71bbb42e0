// CPU check of the resident multi-shift kernel's block decomposition and addressing
// (res_geom, res_site): on every lattice of a list the blocks tile the sites, the launch
// fits its limits, a neighbour inside the block is found in LDS, and what a site reads from
// another workgroup's face is what the neighbouring site wrote there.  Built by hipcc for
// the host; prints "res_geom ok".
#include <cstdio>
#include <vector>

#include "ov_host.hpp"
#include "ov_kernels.hpp"

using namespace ov;

static int fails = 0;
#define CHECK(c, d)                                                                       \
  do {                                                                                    \
    if (!(c)) {                                                                           \
      if (fails++ < 10)                                                                   \
        std::printf("failed: %s (line %d) at %dx%dx%dx%d\n", #c, __LINE__, (d)[0], (d)[1], \
                    (d)[2], (d)[3]);                                                      \
    }                                                                                     \
  } while (0)

template <class R>
static void check(const int* d, int ncu, bool fits) {
  const int maxK = sizeof(R) == sizeof(double) ? 1 : 2;
  const ResGeom q = res_geom(d, (int)sizeof(c2<R>), ncu, maxK);
  CHECK((q.G > 0) == fits, d);
  if (q.G == 0) return;
  CHECK(q.G <= ncu && q.K <= maxK && q.threads % 64 == 0 && q.threads <= RES_MAX_THREADS, d);
  CHECK(q.threads * q.K >= q.S && (q.S + 1) * RES_SITE<R> <= RES_MAX_LDS, d);
  const int V = d[0] * d[1] * d[2] * d[3];
  CHECK(q.G * q.S == V, d);
  ResRun U{};
  U.G = q.G;
  U.FT = q.FT;
  for (int m = 0; m < 4; ++m) {
    U.b[m] = q.b[m];
    U.nb[m] = q.nb[m];
    CHECK(q.b[m] * q.nb[m] == d[m] && (q.nb[m] == 1 || q.b[m] >= 2), d);
  }
  const Geo g{d[0], d[1], d[2], d[3], V, -1};
  std::vector<ResSite> at(V);
  std::vector<int> wg(V, -1);
  const unsigned fb = (unsigned)(q.G * q.FT * sizeof(c2<R>));
  std::vector<char> used(fb / 8, 0);
  for (int w = 0; w < q.G; ++w)
    for (int j = 0; j < q.S; ++j) {
      const ResSite s = res_site<R>(U, g, w, j);
      CHECK(s.gi >= 0 && s.gi < V && wg[s.gi] < 0, d);
      at[s.gi] = s;
      wg[s.gi] = w;
      for (int m = 0; m < 4; ++m) {
        if (s.st[m] == RES_OOB) continue;
        // bytes of the two components: FP64 F values apart, FP32 side by side
        const unsigned F = (unsigned)(q.S / q.b[m]) * (unsigned)sizeof(c2<R>);
        for (int k = 0; k < 2; ++k) {
          const unsigned o = s.st[m] + (sizeof(R) == sizeof(double) ? k * F : k * 8u);
          CHECK(o + sizeof(c2<R>) <= fb && !used[o / 8], d);
          if (o + sizeof(c2<R>) <= fb) used[o / 8] = 1;
        }
      }
    }
  for (int i = 0; i < V; ++i) {
    const ResSite& s = at[i];
    int st = 1, r = i;
    for (int m = 0; m < 4; ++m) {
      const int c = r % d[m];
      r /= d[m];
      const int up = c + 1 < d[m] ? i + st : i + st - st * d[m];
      const int dn = c > 0 ? i - st : i - st + st * d[m];
      for (int side = 0; side < 2; ++side) {
        const ResSite& n = at[side ? dn : up];
        const bool cut = s.fl & ((side ? 2u : 1u) << 2 * m);
        if (cut) {
          CHECK((side ? s.nb[m] >> 16 : s.nb[m] & 0xffffu) == (unsigned)q.S, d);  // zero site
          CHECK(s.ld[m] == n.st[m] && n.st[m] != RES_OOB, d);
          // the sender's face is the one that looks at the receiver
          CHECK(n.fl & ((side ? 1u : 2u) << 2 * m), d);
        } else {
          CHECK(wg[n.gi] == wg[i], d);
          CHECK((side ? s.nb[m] >> 16 : s.nb[m] & 0xffffu) == (unsigned)n.j, d);
        }
      }
      st *= d[m];
    }
    const int t = i / (d[0] * d[1] * d[2]);
    CHECK(((s.fl & 256u) != 0) == (t == d[3] - 1) && ((s.fl & 512u) != 0) == (t == 0), d);
  }
  // a thread beyond the block sends and receives nothing
  const ResSite x = res_site<R>(U, g, q.G - 1, q.S);
  for (int m = 0; m < 4; ++m) CHECK(x.st[m] == RES_OOB && x.ld[m] == RES_OOB, d);
}

int main() {
  const int small[][4] = {{2, 2, 2, 2}, {4, 4, 4, 4}, {2, 4, 6, 8}, {6, 4, 2, 10}, {2, 2, 2, 64},
                          {64, 2, 2, 2}, {8, 8, 8, 8}, {12, 6, 10, 14}, {14, 14, 14, 14},
                          {16, 16, 8, 4}, {2, 26, 2, 38}, {12, 12, 12, 12}, {16, 16, 16, 16},
                          {16, 16, 16, 32}, {6, 22, 10, 42}};
  for (const auto& d : small) {
    check<double>(d, 256, true);
    check<float>(d, 256, true);
  }
  const int big[4] = {24, 24, 24, 48};  // 2592 sites per compute unit
  check<double>(big, 256, false);
  check<float>(big, 256, false);
  if (fails == 0) std::printf("res_geom ok\n");
  return fails != 0;
}
