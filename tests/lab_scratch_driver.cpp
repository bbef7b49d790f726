// Layout checks of the label recovery's scratch over a sweep of sizes (host code; no GPU call).
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "nlr_internal.hpp"

using namespace nlr;

int main() {
  const int64_t ns[] = {1, 2, 5, 64, 257, 500, 1100, 5766, 10996, 60000, 127464, 614822, 1000000, 20000000};
  const int32_t ds[] = {1, 2, 8, 16, 51, 64, 130, 200, 768};
  const int32_t rs[] = {1, 2, 3, 4, 5, 7, 8, 13, 16, 30, 33, 64, 65, 100, 128, 129, 200, 300, 448};
  long cases = 0, fails = 0;
  for (int64_t n : ns)
    for (int32_t d : ds)
      for (int32_t r : rs)
        for (int form = 0; form < 8; ++form) {
          if (r > n) continue;
          const Geometry g = make_geometry(n, d, r, 1, form & 1, form & 2, form & 4);
          Bufs b;
          char* base = reinterpret_cast<char*>((uintptr_t)1 << 20);
          const size_t total = carve_workspace(g, base, &b);
          const int32_t kmax = std::min(r, kLabMaxK);
          for (int32_t K : {1, std::max(1, kmax / 2), kmax}) {
            char* lo = reinterpret_cast<char*>(b.theta_part);
            const LabScratch L = carve_lab_scratch(n, r, K, lo, b.union_bytes);
            const size_t r64 = L.r64, r32 = (size_t)(r + 31) / 32 * 32, k32 = (size_t)(K + 31) / 32 * 32, rk = (size_t)r * K;
            // arrays in use at the same time: inside the region and apart (the Gram partials and
            // the cluster sums share one place)
            std::vector<std::pair<const char*, size_t>> a = {
                {(char*)L.gpart, std::max((size_t)L.GU * r * r * 8, (size_t)L.W * (rk * 8 + (size_t)K * 4))},
                {(char*)L.A, r64 * r64 * 8}, {(char*)L.V, r64 * r64 * 8}, {(char*)L.Q, r64 / 64 * 4096 * 8},
                {(char*)L.jpart, 2 * kLabJacParts * 8}, {(char*)L.P, rk * 8}, {(char*)L.Pt, rk * 8},
                {(char*)L.Mimg, r32 * k32 * 4}, {(char*)L.Mt, rk * 8}, {(char*)L.centT, (size_t)K * K * 8},
                {(char*)L.cn, (size_t)K * 8}, {(char*)L.cscale, (size_t)r * 8}, {(char*)L.cinv, (size_t)r * 8},
                {(char*)L.minv, (size_t)K * 8}, {(char*)L.ubound, (size_t)r * 8}, {(char*)L.scal, 24},
                {(char*)L.seeds, (size_t)K * 8}, {(char*)L.grp, (size_t)K * 4}, {(char*)L.lead, (size_t)K * 4}, {(char*)L.flag, 64}};
            std::sort(a.begin(), a.end());
            bool ok = a.front().first >= lo && (size_t)(a.back().first + a.back().second - lo) <= b.union_bytes &&
                      b.union_bytes <= total && (char*)L.spart == (char*)L.gpart &&
                      (char*)L.cpart == (char*)L.spart + (size_t)L.W * rk * 8;
            for (size_t i = 0; i + 1 < a.size(); ++i) ok = ok && a[i].first + a[i].second <= a[i + 1].first;
            // the rows are shared out: up to 64 columns a chunk never takes more than 1024 rows before
            // 48 chunks are reached, above that never more than a tenth of them at 1e5 rows and more
            const int64_t full = (n + 255) / 256;
            const int64_t want = r <= 64 ? std::min<int64_t>(std::max<int64_t>(full / 4, 1), 48) : (n >= 100000 ? 10 : 1);
            ok = ok && L.GU >= want && L.W >= want && L.GU <= full && L.W <= full;
            ++cases;
            if (!ok && ++fails <= 20)
              std::printf("n %lld d %d r %d K %d form %d: GU %d W %d region %zu\n", (long long)n, d, r, K, form, L.GU,
                          L.W, b.union_bytes);
          }
        }
  std::printf("%ld cases, %ld failed\n", cases, fails);
  return fails ? 1 : 0;
}
