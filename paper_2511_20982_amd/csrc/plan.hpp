// Launch planning of the attention kernels: pure integer arithmetic on the
// host copies of the lengths and the machine shape (CU and XCD counts), with
// no HIP dependency, so the same functions size the launches in the library
// and are checked on the CPU at several machine shapes.  The few formulas the
// kernels evaluate too are constexpr (host and device).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace dopd {

// Compute units and XCDs of the device a call runs on.
struct MachineShape {
  int cus;
  int xcds;
};
// Used when no device answers the query (only host-side sizing can run then).
constexpr MachineShape kDefaultMachine{256, 8};

// Four-wave workgroups resident per CU for the decode and prefill kernels
// (both are launched with __launch_bounds__(256, 2)).
constexpr int kWgPerCu = 2;

// Grid of `blocks` workgroups in one or two dimensions: a dimension holds fewer than
// 2^32 threads, which 2^23 workgroups of 512 reach.  Workgroup (x, y) is block
// grid_block(x, y); those from `blocks` on, in the last row, have no work.
constexpr unsigned kGridRow = 1u << 22;
constexpr int64_t kGridMaxBlocks = (int64_t)INT32_MAX - kGridRow;  // every index fits an int
struct GridShape {
  unsigned x, y;
};
constexpr GridShape grid_shape(int64_t blocks) {
  return blocks <= kGridRow ? GridShape{(unsigned)blocks, 1}
                            : GridShape{kGridRow, (unsigned)((blocks + kGridRow - 1) / kGridRow)};
}
constexpr int grid_block(unsigned x, unsigned y) { return (int)(y * kGridRow + x); }

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- decode partition ------------------------------------------------------
// The keys of every (request r, KV head c) are cut into pairs of pages (32
// tokens); (r, c) is a span of seg + pairs work units, spans laid out r-major
// then c; workgroup b takes units [b * total / nwg, (b+1) * total / nwg).
constexpr int kDecSegCost = 8;          // work units of a segment start, in bf16 pairs
constexpr int64_t kDecMaxUnits = INT32_MAX / 2;  // of a call (the kernels count them in an int)
constexpr int kDecMaxSplitTokens = 4096;
constexpr int64_t kDecMinPairsPerWg = 4;  // one pair per wave at least

// How the decode of one kind of pool is laid on the machine: seg, the work
// units a segment start counts, and the resident workgroups per CU, in
// quarters, that the automatic partition fills.
struct DecodeShape {
  int seg = kDecSegCost;
  int quarter_wgs = 4 * kWgPerCu;
};

constexpr int64_t dec_slice_begin(int64_t b, int64_t total, int64_t nwg) {
  return b * total / nwg;
}

inline int64_t decode_total_units(const int32_t* ctx, int32_t n, int hkv, int seg = kDecSegCost) {
  int64_t units = 0;
  for (int32_t r = 0; r < n; ++r) units += (int64_t)(seg + (ctx[r] + 31) / 32) * hkv;
  return units;
}

// Resident decode workgroup slots the automatic partition fills: quarter_wgs / 4
// workgroups per CU.
inline int64_t decode_slots(const MachineShape& m, int quarter_wgs = 4 * kWgPerCu) {
  return std::max<int64_t>(1, (int64_t)std::max(1, m.cus) * std::max(1, quarter_wgs) / 4);
}

// Workgroups of the partition: split_tokens / 32 units each when given, else
// one slice per resident slot (one round).
inline int64_t decode_nwg(int64_t total_units, int32_t split_tokens, const MachineShape& m,
                          int quarter_wgs = 4 * kWgPerCu) {
  if (total_units <= 0) return 0;
  if (split_tokens > 0) {
    const int64_t per = split_tokens / 32;
    return (total_units + per - 1) / per;
  }
  const int64_t slots = decode_slots(m, quarter_wgs);
  return std::max<int64_t>(1, std::min(slots, (total_units + kDecMinPairsPerWg - 1) /
                                                  kDecMinPairsPerWg));
}

// Work units of a segment start in a call's partition: ds.seg where the call fills
// the machine.  Smaller calls have one slice per kDecMinPairsPerWg units, counted
// with kDecSegCost, one pair a wave: heavier starts would make it two (E4M3, d 64,
// one request of 1000 tokens, 8 KV heads, 8.5 us against 7.7).  An explicit
// split_tokens counts kDecSegCost too, as do totals that would not fit an int.
inline int decode_seg(const int32_t* ctx, int32_t n, int hkv, int32_t split_tokens, const MachineShape& m,
                      const DecodeShape& ds) {
  const int64_t nwg = decode_nwg(decode_total_units(ctx, n, hkv), split_tokens, m, ds.quarter_wgs);
  if (split_tokens > 0 || nwg < decode_slots(m, ds.quarter_wgs)) return kDecSegCost;
  return decode_total_units(ctx, n, hkv, ds.seg) <= kDecMaxUnits ? ds.seg : kDecSegCost;
}

// Does a call with the automatic partition run one workgroup of
// kDecDirectWaves waves per whole (r, c) instead (no partials, no second
// kernel)?  A route's steps are the pairs one of its waves takes one after the
// other: of the longest context here, of a slice and its segment starts (ds.seg
// units each) in the partition, which is charged one more, for its merge, where it
// has more than one.  More (r, c) than CUs would take turns.  Measured, partition /
// direct, 8 KV heads of 128, pages from HBM, * the route taken:
//   bf16  16 requests of 200 tokens 14.0 / 9.3* us, 4 of 500 10.6* / 10.4, 16 of 500
//         16.5 / 12.0*, 4 of 750 11.5* / 14.3, 4 of 1000 15.6* / 15.3, 16 of 2000
//         28.9* / 31.3, 32 of 2000 44.3 / 40.2*, 1 of 2000 12.3* / 24.0
//   E4M3  1 of 250 8.4 / 7.0*, 4 of 500 9.7 / 8.2*, 4 of 750 10.3 / 10.2*, 1 of 1000
//         9.8* / 10.8, 16 of 1000 14.8 / 11.9*, 16 of 2000 19.1* / 19.2
// (Partitions of one step but more workgroups than CUs take longer than this counts:
// 8 of 500, bf16, 14.5* / 10.6; 8 of 1000, E4M3, 13.0* / 10.9.)
constexpr int kDecDirectWaves = 8;
inline bool decode_direct(const int32_t* ctx, int32_t n, int hkv, int32_t split_tokens,
                          const MachineShape& m, const DecodeShape& ds) {
  if (split_tokens > 0 || (int64_t)n * hkv > std::max(1, m.cus)) return false;
  int32_t most = 0;
  for (int32_t r = 0; r < n; ++r) most = std::max(most, ctx[r]);
  const int64_t direct = ((most + 31) / 32 + kDecDirectWaves - 1) / kDecDirectWaves;
  const int64_t total = decode_total_units(ctx, n, hkv, ds.seg);
  const int64_t nwg = decode_nwg(decode_total_units(ctx, n, hkv), 0, m, ds.quarter_wgs);
  const int64_t split = (total + 4 * nwg - 1) / (4 * nwg);  // (a partition workgroup has 4 waves)
  return direct <= split + (split > 1 ? 1 : 0);
}

// Workspace of the decode: partial slots, at most one per (workgroup, (r, c))
// boundary, indexed workgroup + (r * Hkv + c); [slots][g][d] fp32 partial
// outputs, then [slots][g][2] (m, l), each 256-byte aligned.
struct DecodeLayout {
  int64_t nwg, slots;
  size_t part_o_off, part_ml_off, total;
};

inline DecodeLayout decode_layout(int g, int hkv, int d, const int32_t* ctx, int32_t n,
                                  int32_t split_tokens, const MachineShape& m,
                                  const DecodeShape& ds = DecodeShape{}) {
  DecodeLayout L{};
  // (the count of workgroups, and so the workspace, is that of bf16 pools)
  L.nwg = decode_nwg(decode_total_units(ctx, n, hkv), split_tokens, m, ds.quarter_wgs);
  L.slots = L.nwg + (int64_t)n * hkv;
  L.part_o_off = 0;
  L.part_ml_off = align256((size_t)L.slots * g * d * sizeof(float));
  L.total = L.part_ml_off + align256((size_t)L.slots * g * 2 * sizeof(float));
  return L;
}

// The workgroup whose slice holds work unit x (the kernels use the same search).
inline int64_t dec_slice_of(int64_t x, int64_t total, int64_t nwg) {
  int64_t b = x * nwg / total;
  while (b + 1 < nwg && dec_slice_begin(b + 1, total, nwg) <= x) ++b;
  while (b > 0 && dec_slice_begin(b, total, nwg) > x) --b;
  return b;
}

// Does any (r, c) span two slices (then the merge kernel runs)?
inline bool decode_needs_merge(const int32_t* ctx, int32_t n, int hkv, int64_t total,
                               int64_t nwg, int seg = kDecSegCost) {
  int64_t base = 0;
  for (int32_t r = 0; r < n; ++r) {
    const int64_t np = (ctx[r] + 31) / 32, span = seg + np;
    for (int c = 0; c < hkv; ++c) {
      const int64_t first = base + c * span + seg;  // unit of the first pair
      if (dec_slice_of(first, total, nwg) != dec_slice_of(first + np - 1, total, nwg))
        return true;
    }
    base += span * hkv;
  }
  return false;
}

// The (r, c) whose pairs span several slices (the ones the merge kernel
// combines), listed for the merge kernel's arguments: item = r * Hkv + c
// | b0 << 14 | (b1 - b0) << 24, with b0 and b1 the slices of its first and
// last pair, in (r, c) order.  Returns the count, or -1 when the list would
// not fit that packing (more than 2^14 (r, c), 2^10 workgroups, a span of
// more than 255 slices) or more than max items (the caller then merges with
// the kernel that finds its pairs itself).
constexpr int kMergeRcBits = 14, kMergeB0Bits = 10;

inline int decode_merge_list(const int32_t* ctx, int32_t n, int hkv, int64_t total, int64_t nwg,
                             uint32_t* items, int max, int seg = kDecSegCost) {
  if ((int64_t)n * hkv > (1 << kMergeRcBits) || nwg > (1 << kMergeB0Bits)) return -1;
  int cnt = 0;
  int64_t base = 0;
  for (int32_t r = 0; r < n; ++r) {
    const int64_t np = (ctx[r] + 31) / 32, span = seg + np;
    for (int c = 0; c < hkv; ++c) {
      const int64_t first = base + c * span + seg;  // unit of the first pair
      const int64_t b0 = dec_slice_of(first, total, nwg), b1 = dec_slice_of(first + np - 1, total, nwg);
      if (b0 == b1) continue;
      if (cnt == max || b1 - b0 > 255) return -1;
      items[cnt++] = (uint32_t)((int64_t)r * hkv + c) | (uint32_t)b0 << kMergeRcBits |
                     (uint32_t)(b1 - b0) << (kMergeRcBits + kMergeB0Bits);
    }
    base += span * hkv;
  }
  return cnt;
}

// ---- prefill work order ----------------------------------------------------
// n_items items dealt to the XCDs in contiguous slices of per_xcd items; the
// hardware dispatcher sends workgroup b to XCD b % xcds, so workgroup b takes
// item (b % xcds) * per_xcd + b / xcds (none when past the list).
constexpr int pf_per_xcd(int n_items, int xcds) { return (n_items + xcds - 1) / xcds; }
constexpr int pf_xcd_item(int b, int xcds, int per_xcd) {
  return (b % xcds) * per_xcd + b / xcds;
}
constexpr bool pf_xcd_valid(int b, int xcds, int per_xcd, int n_items) {
  return b / xcds < per_xcd && pf_xcd_item(b, xcds, per_xcd) < n_items;
}

// x / d by a multiplication, exact for x * d < 2^32 (the planner checks).
struct FastDiv {
  uint32_t d, m;
};
constexpr FastDiv fast_div(uint32_t d) { return {d, d > 1 ? (uint32_t)(((uint64_t)1 << 32) / d + 1) : 0}; }
constexpr int fast_quot(int x, const FastDiv& f) {
  return f.d > 1 ? (int)(((uint64_t)(uint32_t)x * f.m) >> 32) : x;
}

// The XCD-aware order (at most kPfMaxOrdered requests): a list of entries,
// each a run of q tiles of one request, heaviest entry first; every entry's
// items are dealt over all XCDs, so each XCD works through the same entries in
// the same order and the XCDs finish together whatever the lengths.  (Against
// one contiguous slice of a (KV head, request, q tile) list per XCD, where a
// slice restarted with the long requests at every head and, with fewer heads
// than XCDs, one XCD held the long requests and the next the short ones: 16
// chunks of 512 over mixed prefixes, 32/32 heads, 424 -> 369 us; 8 short
// prompts, 28/4 heads, 39 -> 34 us; 16 long prompts, 32/32 heads, 1.70 -> 1.67
// ms.)  Workgroup b is place b / xcds of XCD b % xcds; entry k takes the
// places [e[k - 1].incl, e[k].incl) of every XCD.
//   hkv a multiple of xcds: an XCD takes whole heads, its items in the order
//     (q tile descending, KV head, query head);
//   xcds a multiple of hkv: `share` XCDs take one head's (q tile descending,
//     query head) list alternately;
//   otherwise: contiguous slices of the (KV head, q tile descending, query
//     head) list.
constexpr int kPfMaxOrdered = 64;
struct PfEntry {        // 32 bytes, read by one lane of the kernel
  int incl;             // places per XCD up to and with this entry
  int req, seq0, len, prefix;  // the request, its first row, rows, cached tokens
  int tile0, nt;        // lowest q tile of the run, q tiles
  int rot;              // XCD that takes the first item (where items do not divide evenly)
};
struct PfOrder {
  int n;                // entries
  int sliced;           // the third way above
  int xcds, hkv, g;
  FastDiv by_xcds, by_share, by_width;  // width: query heads an XCD takes of one q tile
  PfEntry e[kPfMaxOrdered];
};

// Places an entry of nt q tiles takes on each XCD.
constexpr int pf_entry_places(int nt, int g, int hkv, int xcds) {
  return xcds % hkv == 0 ? pf_per_xcd(nt * g, xcds / hkv) : pf_per_xcd(nt * g * hkv, xcds);
}

// Item at place `local` of an entry (rot, nt) on XCD x: q tile counted from
// the last of the run, and query head; false when there is none.
constexpr bool pf_entry_item(const PfOrder& o, int rot, int nt, int x, int local, int& back, int& h) {
  if (!o.sliced) {
    const int share = (int)o.by_share.d, width = (int)o.by_width.d;
    const int xs = fast_quot(x, o.by_share), y = x - xs * share + share - rot;
    const int i = local * share + (y >= share ? y - share : y);
    back = fast_quot(i, o.by_width);
    h = xs * width + i - back * width;
    return back < nt;
  }
  const int per = pf_entry_places(nt, o.g, o.hkv, o.xcds), b = local * o.xcds + (x + o.xcds - rot) % o.xcds;
  if (!pf_xcd_valid(b, o.xcds, per, nt * o.g * o.hkv)) return false;
  const int i = pf_xcd_item(b, o.xcds, per), head = i / (nt * o.g), idx = i % (nt * o.g);
  back = idx / o.g;
  h = head * o.g + idx % o.g;
  return true;
}

// The rot of the entry after one of nt q tiles with `rot`.
constexpr int pf_entry_next_rot(int rot, int nt, int g, int hkv, int xcds) {
  if (xcds % hkv == 0) return (int)(((int64_t)rot + (int64_t)nt * g) % (xcds / hkv));
  if (hkv % xcds == 0) return 0;
  const int per = pf_entry_places(nt, g, hkv, xcds);
  return (rot + (nt * g * hkv + per - 1) / per) % xcds;
}

// Key splits of the paged prefill: the requested count (at most kPfMaxSplits),
// or automatically, when the call has at most one work item per CU, about
// (resident slots) / items splits (at most kPfAutoSplits), each split of the
// longest item keeping at least 8 key tiles that every row sees.  Each split
// adds T * Hq * d * 8 bytes of fp32 partials written and read back, which costs
// more than it gains once the items fill the CUs.
constexpr int kPfMaxSplits = 16;
constexpr int kPfAutoSplits = 8;
constexpr int kPfTileRows = 128;  // query rows per work item
constexpr int kPfTileKeys = 64;   // keys per tile

// Builds the order for chunk lengths cu_host and cached prefixes prefix_host
// (null: none); nreq <= kPfMaxOrdered.  An entry is a whole request, longest
// keys first: the q tiles that read one head's K/V then run together under one
// L2.  When the K/V bytes one XCD reads fit its L2 and the call has at most
// kPfMaxOrdered (request, q tile) pairs, every pair is an entry of its own,
// heaviest first (the list a longest-first dispatch wants), if split_requests:
// the fused step does not (its decode slices fill the slots that light items
// free early; mixed step 224 us with whole requests, 228 us split).
constexpr int64_t kPfL2Bytes = 4 << 20;

inline void pf_build_order(PfOrder& o, const int32_t* cu_host, const int32_t* prefix_host,
                           int32_t nreq, int hq, int hkv, int64_t kv_token_bytes, int xcds,
                           bool split_requests = true) {
  const int g = hq / hkv;
  const int heads_per_xcd = (hkv + xcds - 1) / xcds;
  o.n = 0;
  o.sliced = hkv % xcds != 0 && xcds % hkv != 0;
  o.xcds = xcds;
  o.hkv = hkv;
  o.g = g;
  o.by_xcds = fast_div((uint32_t)xcds);
  o.by_share = fast_div((uint32_t)(xcds % hkv == 0 ? xcds / hkv : 1));
  o.by_width = fast_div((uint32_t)(heads_per_xcd * g));
  auto len = [&](int r) { return cu_host[r + 1] - cu_host[r]; };
  auto prefix = [&](int r) { return prefix_host ? prefix_host[r] : 0; };
  auto tiles = [&](int r) { return (len(r) + kPfTileRows - 1) / kPfTileRows; };
  int64_t pairs = 0, keys = 0;
  for (int32_t r = 0; r < nreq; ++r) {
    pairs += tiles(r);
    if (len(r) > 0) keys += (int64_t)len(r) + prefix(r);
  }
  const bool split = split_requests && pairs <= kPfMaxOrdered &&
                     keys * heads_per_xcd * kv_token_bytes <= kPfL2Bytes;
  int64_t weight[kPfMaxOrdered];  // keys the entry's last row sees
  auto add = [&](int r, int t0, int nt, int64_t w) {
    int i = o.n++;
    for (; i > 0 && weight[i - 1] < w; --i) {  // stable insertion, heaviest first
      weight[i] = weight[i - 1];
      o.e[i] = o.e[i - 1];
    }
    weight[i] = w;
    o.e[i] = PfEntry{0, r, cu_host[r], len(r), prefix(r), t0, nt, 0};
  };
  for (int32_t r = 0; r < nreq; ++r) {
    if (tiles(r) == 0) continue;
    if (!split) {
      add(r, 0, tiles(r), (int64_t)prefix(r) + len(r));
    } else {
      for (int t = 0; t < tiles(r); ++t)
        add(r, t, 1, (int64_t)prefix(r) + std::min(len(r), (t + 1) * kPfTileRows));
    }
  }
  int sum = 0, rot = 0;
  for (int k = 0; k < o.n; ++k) {
    o.e[k].incl = sum += pf_entry_places(o.e[k].nt, g, hkv, xcds);
    o.e[k].rot = rot;
    rot = pf_entry_next_rot(rot, o.e[k].nt, g, hkv, xcds);
  }
}

// Places per XCD of the whole order.
inline int pf_order_places(const PfOrder& o) { return o.n > 0 ? o.e[o.n - 1].incl : 0; }

// Do the order's divisions by multiplication hold for it with nsplit key splits?
inline bool pf_order_fits(const PfOrder& o, int nsplit) {
  const int64_t places = (int64_t)pf_order_places(o) * nsplit, top = (int64_t)1 << 32;
  return places * o.xcds * std::max(o.xcds, nsplit) < top &&
         (places + 1) * o.by_share.d * o.by_width.d < top;
}

inline int prefill_paged_splits(int hq, bool splittable, const int32_t* cu_host,
                                const int32_t* prefix_host, int32_t nreq, int32_t num_splits,
                                const MachineShape& m) {
  if (!splittable) return 1;
  if (num_splits > 0) return std::min(num_splits, kPfMaxSplits);
  const int64_t slots = (int64_t)kWgPerCu * std::max(1, m.cus);
  int64_t items = 0, max_full = 0;
  for (int32_t r = 0; r < nreq; ++r) {
    const int64_t len = cu_host[r + 1] - cu_host[r];
    const int64_t tiles = (len + kPfTileRows - 1) / kPfTileRows;
    items += tiles * hq;
    if (tiles > 0)
      max_full = std::max<int64_t>(max_full,
                                   (prefix_host[r] + (tiles - 1) * kPfTileRows) / kPfTileKeys);
  }
  if (items == 0 || items > slots / 2) return 1;
  int64_t n = slots / items;
  n = std::min<int64_t>(n, 1 + max_full / 8);
  return (int)std::max<int64_t>(1, std::min<int64_t>(n, kPfAutoSplits));
}

inline size_t prefill_paged_ws_bytes(int hq, int d, int64_t T, int nsplit) {
  if (nsplit <= 1) return 0;
  const size_t rows = (size_t)nsplit * T * hq;
  return align256(rows * d * sizeof(float)) + align256(rows * 2 * sizeof(float));
}

}  // namespace dopd
