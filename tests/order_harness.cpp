// CPU check of the prefill's XCD-aware order (paper_2511_20982_amd/csrc/plan.hpp)
// at a given XCD count: every (request, q tile, head) item is taken by exactly
// one place, every index stays in range, heads stay on the XCDs the rule gives
// them, and the XCDs get equal shares.
// Usage: order_harness <xcds>; prints "ok <cases>" or the first failure.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>
#include <vector>

#include "../paper_2511_20982_amd/csrc/plan.hpp"

using namespace dopd;

static int fail(const char* what, long a, long b) {
  std::printf("FAIL %s (%ld, %ld)\n", what, a, b);
  return 1;
}

static int check(const std::vector<int32_t>& lens, const std::vector<int32_t>& prefix, int hq, int hkv,
                 int64_t kv_bytes, int xcds, bool split_requests = true) {
  const int n = (int)lens.size(), g = hq / hkv;
  std::vector<int32_t> cu(n + 1, 0);
  for (int r = 0; r < n; ++r) cu[r + 1] = cu[r] + lens[r];
  PfOrder o;
  pf_build_order(o, cu.data(), prefix.empty() ? nullptr : prefix.data(), n, hq, hkv, kv_bytes, xcds,
                 split_requests);
  if (!split_requests)  // whole requests: the fused step's order
    for (int k = 0; k < o.n; ++k)
      if (o.e[k].tile0 != 0 || o.e[k].nt != (o.e[k].len + kPfTileRows - 1) / kPfTileRows)
        return fail("part of a request", k, o.e[k].nt);
  if (o.n < 0 || o.n > kPfMaxOrdered) return fail("entries", o.n, n);
  std::map<std::tuple<int, int, int>, int> seen;
  std::vector<long> got(xcds, 0);
  std::vector<std::map<int, int>> heads(xcds);
  int64_t last = -1;
  for (int k = 0; k < o.n; ++k) {
    const PfEntry& e = o.e[k];
    const int r = e.req;
    if (r < 0 || r >= n || e.nt < 1 || e.tile0 < 0) return fail("entry", k, r);
    if (e.seq0 != cu[r] || e.len != lens[r] || e.prefix != (prefix.empty() ? 0 : prefix[r]))
      return fail("entry's rows", k, r);
    const int64_t w = (prefix.empty() ? 0 : prefix[r]) +
                      std::min<int64_t>(lens[r], (int64_t)(e.tile0 + e.nt) * kPfTileRows);
    if (last >= 0 && w > last) return fail("entries not heaviest first", k, (long)w);
    last = w;
    const int places = e.incl - (k ? o.e[k - 1].incl : 0);
    for (int x = 0; x < xcds; ++x)
      for (int local = 0; local < places; ++local) {
        int back = -1, h = -1;
        if (!pf_entry_item(o, e.rot, e.nt, x, local, back, h)) continue;
        const int tile = e.tile0 + e.nt - 1 - back, head = h / g;
        if (h < 0 || h >= hq || back < 0 || back >= e.nt) return fail("item", h, back);
        if (tile < 0 || tile >= (lens[r] + kPfTileRows - 1) / kPfTileRows) return fail("tile", tile, lens[r]);
        ++seen[{r, tile, h}];
        ++got[x];
        heads[x][head] = 1;
      }
  }
  long items = 0;
  for (int r = 0; r < n; ++r) items += (long)((lens[r] + kPfTileRows - 1) / kPfTileRows) * hq;
  if ((long)seen.size() != items) return fail("items not covered", (long)seen.size(), items);
  for (auto& s : seen)
    if (s.second != 1) return fail("item taken more than once", std::get<0>(s.first), std::get<1>(s.first));
  // the kernel's way from a workgroup to its XCD, place and split, where the order
  // says that its divisions hold
  for (int nsplit : {1, 3, kPfMaxSplits}) {
    if (!pf_order_fits(o, nsplit)) return fail("order does not fit", nsplit, o.n);
    const FastDiv by_split = fast_div((uint32_t)nsplit);
    const int64_t blocks = (int64_t)pf_order_places(o) * nsplit * xcds;
    for (int64_t b = 0; b < blocks; b += blocks > 20000 ? 7 : 1) {
      const int s = fast_quot((int)b, o.by_xcds), place = fast_quot(s, by_split);
      if (s != b / xcds || place != s / nsplit) return fail("workgroup's place", (long)b, nsplit);
    }
  }
  if (hkv % xcds == 0 || xcds % hkv == 0) {
    long lo = got[0], hi = got[0];
    for (int x = 0; x < xcds; ++x) {
      lo = std::min(lo, got[x]);
      hi = std::max(hi, got[x]);
      if (hkv >= xcds ? (int)heads[x].size() > hkv / xcds : (int)heads[x].size() > 1)
        return fail("heads of an XCD", x, (long)heads[x].size());
    }
    if (hi - lo > 1) return fail("unequal shares", lo, hi);  // the odd items go round in turn
  }
  return 0;
}

static int check_fast_div() {
  std::mt19937_64 rng(3);
  for (uint32_t d : {1u, 2u, 3u, 6u, 7u, 8u, 28u, 56u, 64u, 100u, 4096u, 65535u})
    for (int i = 0; i < 20000; ++i) {
      const uint64_t top = std::min<uint64_t>(((uint64_t)1 << 32) / d, INT32_MAX);
      const int x = i < 200 ? i : i < 400 ? (int)(top - 1 - (i - 200)) : (int)(rng() % top);
      if (x >= 0 && fast_quot(x, fast_div(d)) != x / (int)d) return fail("fast_quot", x, d);
    }
  return 0;
}

// Orders too large for divisions by multiplication say so, and the ones just below
// divide exactly at their last workgroup.
static int check_fits(int xcds) {
  bool some_fit = false, some_do_not = false;
  for (int hq : {32, 64})
    for (int nsplit : {1, 16}) {
      bool fits = true;
      for (int64_t len = 1 << 20; len <= INT32_MAX; len += len / 3) {
        const int32_t cu[2] = {0, (int32_t)len};
        PfOrder o;
        pf_build_order(o, cu, nullptr, 1, hq, 8, 512, xcds);
        const int64_t places = (int64_t)pf_order_places(o) * nsplit, blocks = places * xcds;
        const bool now = pf_order_fits(o, nsplit);
        if (now && !fits) return fail("a larger order fits", (long)len, nsplit);
        fits = now;
        some_fit |= now;
        some_do_not |= !now;
        if (!now || blocks > INT32_MAX / 2) continue;  // (refused before the order is asked)
        const FastDiv by_split = fast_div((uint32_t)nsplit);
        if (fast_quot((int)(blocks - 1), o.by_xcds) != places - 1 ||
            fast_quot((int)(places - 1), by_split) != pf_order_places(o) - 1)
          return fail("last workgroup of an order that fits", (long)len, nsplit);
        int back = -1, h = -1;
        for (int x = 0; x < xcds; ++x)
          if (!o.sliced && pf_entry_item(o, o.e[0].rot, o.e[0].nt, x, pf_order_places(o) - 1, back, h) &&
              (back < 0 || back >= o.e[0].nt || h < 0 || h >= hq))
            return fail("last item of an order that fits", back, h);
      }
    }
  if (!some_fit || !some_do_not) return fail("orders on one side of the limit only", some_fit, some_do_not);
  return 0;
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  const int xcds = std::atoi(argv[1]);
  std::mt19937 rng(7);
  int cases = 0;
  if (check_fast_div()) return 1;
  const int heads[][2] = {{32, 32}, {64, 8}, {28, 4}, {8, 2}, {5, 1}, {6, 3}, {12, 12}, {10, 5}, {16, 16}, {24, 24}};
  for (auto& h : heads)
    for (int t = 0; t < 24; ++t) {
      const int n = t < 4 ? 1 : 1 + (int)(rng() % 64);
      std::vector<int32_t> lens(n), prefix;
      for (auto& x : lens) x = t % 5 == 0 ? 512 : (int)(rng() % (t % 3 ? 700 : 3000));
      if (t % 2)
        for (int r = 0; r < n; ++r) prefix.push_back((int)(rng() % 5000));
      for (int64_t kv : {256, 512})
        if (check(lens, prefix, h[0], h[1], kv, xcds)) return 1;
      if (t < 12 && check(lens, prefix, h[0], h[1], 256, xcds, false)) return 1;
      ++cases;
    }
  if (check_fits(xcds)) return 1;
  if (check({128}, {}, 32, 32, 512, xcds) || check({0, 1, 0, 129}, {}, 28, 4, 512, xcds)) return 1;
  std::printf("ok %d\n", cases + 2);
  return 0;
}
