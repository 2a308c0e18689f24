// Paged KV writers: scatter fresh token-major K/V rows into the page pools.
//   k_pool[page][Hkv][16][d]  (token-major page),  v_pool[page][Hkv][d][16]  (dim-major page)
// Bit copies (bf16, fp32), or E4M3 pools: each bf16 element x of KV head h
// becomes the code of sat(x * fp32(1 / scale[h])) (product in fp32, rounded to
// nearest even; codes rounded to nearest even).  Slots of a page outside the
// written range are never touched.
//
// Two mappings.  The page writer gives a wave K or V of one page of 16 / CW KV
// heads (CW chunks of a row per pass: one head, or two bf16 heads at d = 64; of the
// E4M3 codes of an unpack two, at d = 64 four) and issues all of its 16-byte loads at
// once; a lane holds 4 tokens of 8 (bf16) or 4 (fp32) dims of V, so the transposition
// to dim rows is done in registers four tokens at a time and only gathers rows in LDS,
// privately per wave (no workgroup barrier).  Slots of a page that is written in part
// leave in the widest aligned stores that fit.  The append writer gives a wave 64
// 16-byte chunks of one token's K or V: with one or two tokens per request every page
// is partial and V is written element by element either way, and what counts is the
// chain of loads that finds the request and its page, and the cache lines that the
// elements of V touch.
//
// HBM-bound at size: E4M3 writes of 16 prompts (318 MB, 8 heads, d 128) 74 ->
// 62 us (5.1 TB/s), bf16 writes of 16 prompts at 32 heads 262 -> 231 us
// against one workgroup per (page, head) that transposed element by element
// through LDS; the E4M3 append of 256 requests, 8 heads, 9.8 -> 3.9 us.  Small
// calls are bound by one wave's work on one page, hence K and V in waves of their
// own and the wide stores: 5 prompts of 9-40 tokens, 8 heads, one wave for both and
// element by element 4.6 us (E4M3 5.6, fp32 5.1; 8 chunks of 32 tokens 4.5, 5.3,
// 5.2), now 3.7 (3.5, 4.2; 3.5, 3.5, 4.6), the workgroup per (page, head) 3.4 (3.6,
// 3.8; 3.5, 3.5, 4.0).
#pragma once
#include <type_traits>

#include "common.hpp"
#include "../plan.hpp"

namespace dopd {

constexpr int kKvwWaves = 4;  // waves of a page-writer workgroup: K's and V's of consecutive heads of one page

// Calls of at most this many new tokens per request on average take the append
// writer (256 requests, d 128, kernel time append / pages: one token each, 8 heads
// bf16 4.7 / 6.7 us, E4M3 3.9 / 6.4, 32 heads 10.4 / 13.0; two, 6.6 / 7.5, E4M3
// 5.1 / 7.1, 32 heads 12.8 / 14.3; four the pages win).  The host knows only the
// sum; one long request among single tokens is no slower for it (255 of one token
// and one of 257: 5.8 / 6.8, 32 heads 13.3 / 13.4), and with thousands of requests
// it is faster by the search for a token's request (4095 empty ones and one of
// 8192: 31 / 186, 32 heads 90 / 710).
constexpr int kKvwAppendMean = 2;

// Waves of an append workgroup, a K wave and a V wave: V's stores are most of the
// work, so workgroups of V waves alone fill some CUs while others idle (32 heads,
// 4095 empty requests and one of 8192 tokens, E4M3: workgroups of four K or four V
// waves 92 us, of two and two 67, of one and one 64; one token of 32 bf16 heads
// 3.2, 2.8, 2.6).
constexpr int kKvaWaves = 2;

// TI: element type of the fresh rows, TO: of the pools (uint16_t, uint32_t, or
// uint16_t -> uint8_t for E4M3 pools).
template <typename TI, typename TO, int D>
struct PageWrite {
  static constexpr bool kE4m3 = sizeof(TO) == 1 && sizeof(TI) == 2;
  static_assert(kE4m3 || sizeof(TI) == sizeof(TO), "a copy, or bf16 to E4M3");
  static constexpr int EPC = 16 / (int)sizeof(TI);  // elements of a 16-byte chunk of a row
  static constexpr int CPR = D / EPC;               // chunks of a row
  static constexpr int CW = CPR < 16 ? CPR : 16;    // chunks of a row per pass
  static constexpr int NP = CPR / CW;               // passes
  static constexpr int HW = 16 / CW;                // heads of a wave
  static constexpr int RB = kPage * (int)sizeof(TO);  // bytes of a dim row of a V page
  // V rows in LDS, one row of padding after every EPC rows: the 64 lanes'
  // pieces of four tokens fall into distinct banks.
  static constexpr int ROWS = D + D / EPC;
  static constexpr int kLdsBytes = HW * ROWS * RB;  // of one wave
  using Out = std::conditional_t<kE4m3, u32x2, u32x4>;  // a chunk as the pools hold it

  static __device__ __forceinline__ Out convert(u32x4 x, float inv) {
    if constexpr (kE4m3) {
      Out o;
#pragma unroll
      for (int w = 0; w < 2; ++w)
        o[w] = e4m3x4_from_f32(bf16_bits_to_f32(x[2 * w] & 0xffffu) * inv,
                               bf16_bits_to_f32(x[2 * w] >> 16) * inv,
                               bf16_bits_to_f32(x[2 * w + 1] & 0xffffu) * inv,
                               bf16_bits_to_f32(x[2 * w + 1] >> 16) * inv);
      return o;
    } else {
      return x;
    }
  }
};

// A 16-byte chunk of rows that need not be aligned to more than an element.
typedef uint32_t u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ u32x4 load_chunk(const uint8_t* p) { return *reinterpret_cast<const u32x4_a1*>(p); }
__device__ __forceinline__ u32x4 load_chunk(const uint16_t* p) { return *reinterpret_cast<const u32x4_a2*>(p); }
__device__ __forceinline__ u32x4 load_chunk(const uint32_t* p) { return *reinterpret_cast<const u32x4_a4*>(p); }

template <int N>
using Slots = std::integral_constant<int, N>;

// N slots of each of a lane's PL pieces of SPP slots, at slot `at`; none where
// !on, and none wider than a piece.
template <typename TO, int N, int SPP, int PL>
struct SlotStores {
  static constexpr int B = N * (int)sizeof(TO);
  using Word = std::conditional_t<B == 1, uint8_t, std::conditional_t<B == 2, uint16_t,
               std::conditional_t<B == 4, uint32_t, std::conditional_t<B == 8, u32x2, u32x4>>>>;
  bool on;
  int at;
  Word x[PL];
  // Takes N slots at lo, if `take`, and moves lo past them.
  template <class PieceFn>
  __device__ __forceinline__ SlotStores(bool take, int& lo, PieceFn piece) : on(N <= SPP && take) {
    if constexpr (N <= SPP) {
      at = on ? lo : 0;
      lo += on ? N : 0;
#pragma unroll
      for (int k = 0; k < PL; ++k) x[k] = *reinterpret_cast<const Word*>(piece(k) + at * sizeof(TO));
    }
  }
  __device__ __forceinline__ void store(TO* d, int k) const {
    if constexpr (N <= SPP) *reinterpret_cast<Word*>(d + at) = x[k];
  }
};

// Rows [s0, s1) of one page, K's or V's, for the HW heads from h0 (those below
// hkv): src points at KV head 0 of the row that goes to slot s0; rows are
// row_elems apart, heads head_elems.  dst: the page in the pool, KV head 0.  With
// pack (the handoff block's row of slot 0, KV head 0; head h follows pack_head
// elements later) the rows are written there too.  s: the wave's kLdsBytes of
// LDS (V's only), 16-byte aligned.  Every lane of the wave takes part.
template <typename TI, typename TO, int D, bool PACK, bool IS_V>
__device__ __forceinline__ void write_page_rows(const TI* src, int64_t row_elems, int64_t head_elems, int h0,
                                                int hkv, int s0, int s1, TO* dst, const float* scale, TO* pack,
                                                int64_t pack_head, bool pack_aligned, uint8_t* s) {
  using W = PageWrite<TI, TO, D>;
  using Out = typename W::Out;
  constexpr int EPC = W::EPC, CW = W::CW, NP = W::NP, HW = W::HW, RB = W::RB;
  const int l = lane_id();
  const int c = l % CW, tq = l / CW % 4, sub = l / (4 * CW);
  const int h = h0 + sub;
  const bool on = h < hkv;
  const int64_t col = min(h, hkv - 1) * head_elems + EPC * c;
  // K: chunk u is token 4u + tq (whole rows in a row); V: token 4tq + u (four
  // tokens of a dim in one lane).  Tokens outside [s0, s1) read the nearest
  // one inside, so that no load waits behind a branch.
  auto token = [&](int u) { return IS_V ? 4 * tq + u : 4 * u + tq; };
  u32x4 x[NP][4];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      x[p][u] = load_chunk(src + (min(max(token(u), s0), s1 - 1) - s0) * row_elems + col + EPC * CW * p);
  float inv = 1.f;
  if constexpr (W::kE4m3) inv = 1.0f / scale[on ? h : h0];
  // Streaming stores here and below: the rows are not read again soon, and they
  // leave the caches now instead of being written back while the decode that
  // follows streams the pools.
  auto row_out = [&](TO* d, bool aligned, Out y) {
    if (aligned) {
      __builtin_nontemporal_store(y, reinterpret_cast<Out*>(d));
    } else {
      const TO* e = reinterpret_cast<const TO*>(&y);
#pragma unroll
      for (int i = 0; i < EPC; ++i) d[i] = e[i];
    }
  };
  const bool full = s0 == 0 && s1 == kPage;
  // Rows out (K's to the page, and either to the pack): whole pages of heads that
  // are all there store without a test, so that no load sinks behind one.
  Out v[NP][4];
  auto rows_out = [&](auto whole) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = token(u), col_out = t * D + EPC * (c + CW * p);
        v[p][u] = W::convert(x[p][u], inv);
        if (!(whole || (on && t >= s0 && t < s1))) continue;
        if constexpr (!IS_V) row_out(dst + (int64_t)h * (kPage * D) + col_out, true, v[p][u]);
        if constexpr (PACK) {
          if (pack) row_out(pack + h * pack_head + col_out, pack_aligned, v[p][u]);
        }
      }
  };
  if (full && h0 + HW <= hkv) rows_out(std::true_type{});
  else rows_out(std::false_type{});
  if constexpr (!IS_V) return;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    // Dim i of the chunk: its four tokens side by side, into row e of the head.
    uint8_t* piece = s + (sub * W::ROWS + (c + CW * p) * (EPC + 1)) * RB + tq * (RB / 4);
    if constexpr (sizeof(TO) == 4) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(piece + i * RB) = u32x4{v[p][0][i], v[p][1][i], v[p][2][i], v[p][3][i]};
    } else if constexpr (sizeof(TO) == 2) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t sel = i % 2 ? 0x07060302u : 0x05040100u;
        *reinterpret_cast<u32x2*>(piece + i * RB) =
            u32x2{__builtin_amdgcn_perm(v[p][1][i / 2], v[p][0][i / 2], sel),
                  __builtin_amdgcn_perm(v[p][3][i / 2], v[p][2][i / 2], sel)};
      }
    } else {
#pragma unroll
      for (int w = 0; w < EPC / 4; ++w) {
        const uint32_t a = __builtin_amdgcn_perm(v[p][1][w], v[p][0][w], 0x05010400u);  // t0 t1 of dims 0, 1
        const uint32_t b = __builtin_amdgcn_perm(v[p][1][w], v[p][0][w], 0x07030602u);  // of dims 2, 3
        const uint32_t d = __builtin_amdgcn_perm(v[p][3][w], v[p][2][w], 0x05010400u);
        const uint32_t e = __builtin_amdgcn_perm(v[p][3][w], v[p][2][w], 0x07030602u);
        uint32_t* r = reinterpret_cast<uint32_t*>(piece + 4 * w * RB);
        r[0] = __builtin_amdgcn_perm(d, a, 0x05040100u);
        r[RB / 4] = __builtin_amdgcn_perm(d, a, 0x07060302u);
        r[2 * RB / 4] = __builtin_amdgcn_perm(e, b, 0x05040100u);
        r[3 * RB / 4] = __builtin_amdgcn_perm(e, b, 0x07060302u);
      }
    }
  }
  // The LDS rows are this wave's alone (in order within the wave).
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int PPR = RB / 16;       // 16-byte pieces of a dim row
  constexpr int PIECES = D * PPR;    // of a head
  constexpr int SPP = 16 / (int)sizeof(TO);  // slots of a piece
  constexpr int PL = HW * PIECES / 64;  // pieces of a lane
  const int run = l % PPR;
  auto head_of = [&](int k) { return (l + 64 * k) / PIECES; };
  auto row_of = [&](int k) { return (l + 64 * k) % PIECES / PPR; };
  auto piece = [&](int k) {
    const int e = row_of(k);
    return s + (head_of(k) * W::ROWS + e + e / EPC) * RB + 16 * run;
  };
  auto at = [&](int k) { return dst + (int64_t)(h0 + head_of(k)) * (kPage * D) + row_of(k) * kPage + run * SPP; };
  if (full) {
#pragma unroll
    for (int k = 0; k < PL; ++k)
      if (h0 + head_of(k) < hkv)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(piece(k)), reinterpret_cast<u32x4*>(at(k)));
  } else {
    // Slots [lo, hi) of this lane's pieces, in the widest aligned stores that hold
    // no other slot: the run up to an aligned slot, then down from the widest.
    // Each half reads LDS for all of its stores before the first of them.
    int lo = max(s0 - run * SPP, 0);
    const int hi = min(s1 - run * SPP, SPP);
    auto up = [&](auto n) { return SlotStores<TO, n, SPP, PL>{(lo & n) != 0 && lo + n <= hi, lo, piece}; };
    auto down = [&](auto n) { return SlotStores<TO, n, SPP, PL>{lo + n <= hi, lo, piece}; };
    auto put = [&](const auto& y) {
      if (y.on) {
#pragma unroll
        for (int k = 0; k < PL; ++k)
          if (h0 + head_of(k) < hkv) y.store(at(k), k);
      }
    };
    if (s0 != 0) {
      const auto a = up(Slots<1>{});
      const auto b = up(Slots<2>{});
      const auto c4 = up(Slots<4>{});
      const auto d = up(Slots<8>{});
      put(a), put(b), put(c4), put(d);
    }
    const auto a = down(Slots<16>{});
    const auto b = down(Slots<8>{});
    const auto c4 = down(Slots<4>{});
    const auto d = down(Slots<2>{});
    const auto e = down(Slots<1>{});
    put(a), put(b), put(c4), put(d), put(e);
  }
}

template <typename TI, typename TO>
struct KvWriteArgs {
  const TI* k_new;            // [T][Hkv][D]
  const TI* v_new;
  const float* k_scale;       // [Hkv], E4M3 pools only
  const float* v_scale;
  TO* k_pool;
  TO* v_pool;
  const int32_t* page_table;  // [nreq][pt_stride]
  const int32_t* cu_new;      // [nreq + 1]
  const int32_t* start_pos;   // [nreq]
  int pt_stride, nreq, hkv, total_new;
  int head_groups;            // workgroups of a page (page writer) or of a token (append writer)
};

// Page writer: workgroup b takes waves kKvwWaves * (b % head_groups) .. of the
// (b / head_groups)-th touched page; wave i of a page writes K (even) or V (odd)
// of heads i / 2 * HW ..
template <typename TI, typename TO, int D>
__global__ __launch_bounds__(64 * kKvwWaves) void kv_write_kernel(KvWriteArgs<TI, TO> a) {
  using W = PageWrite<TI, TO, D>;
  __shared__ __attribute__((aligned(16))) uint8_t s[kKvwWaves / 2][W::kLdsBytes];  // of the V waves
  // Touched logical pages of request r: those holding positions [start, start + n).
  int cu_l = 0, n_l = 0, st_l = 0;  // this lane's request
  auto touched = [&](int rr) {
    cu_l = a.cu_new[rr];
    n_l = a.cu_new[rr + 1] - cu_l;
    st_l = a.start_pos[rr];
    asm volatile("" : "+v"(st_l));  // (loaded beside cu_new, not after the test)
    return n_l > 0 ? (st_l + n_l - 1) / kPage - st_l / kPage + 1 : 0;
  };
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int b = grid_block(blockIdx.x, blockIdx.y);
  const int wi = b % a.head_groups * kKvwWaves + w;  // wave of the page
  const int h0 = (wi >> 1) * W::HW;
  if (h0 >= a.hkv) return;
  int r, local;
  if (!find_owner(b / a.head_groups, a.nreq, touched, r, local)) return;
  const int row0 = __builtin_amdgcn_readlane(cu_l, r % 64), n = __builtin_amdgcn_readlane(n_l, r % 64);
  const int start = __builtin_amdgcn_readlane(st_l, r % 64);
  const int lp = start / kPage + local;                 // logical page
  const int p_lo = max(start, lp * kPage);              // first position written in this page
  const int p_hi = min(start + n, lp * kPage + kPage);  // one past the last
  const int64_t page = a.page_table[(int64_t)r * a.pt_stride + lp];
  const int64_t row_elems = (int64_t)a.hkv * D;
  const int64_t src = ((int64_t)row0 + (p_lo - start)) * row_elems;
  const int64_t page_elems = (int64_t)a.hkv * (kPage * D);
  if (wi & 1)
    write_page_rows<TI, TO, D, false, true>(a.v_new + src, row_elems, D, h0, a.hkv, p_lo - lp * kPage,
                                            p_hi - lp * kPage, a.v_pool + page * page_elems, a.v_scale,
                                            (TO*)nullptr, 0, false, s[w >> 1]);
  else
    write_page_rows<TI, TO, D, false, false>(a.k_new + src, row_elems, D, h0, a.hkv, p_lo - lp * kPage,
                                             p_hi - lp * kPage, a.k_pool + page * page_elems, a.k_scale,
                                             (TO*)nullptr, 0, false, nullptr);
}

// The request whose rows hold token t: the last r with cu[r] <= t, found by
// whole-wave steps (two trips to memory up to 4096 requests).
__device__ __forceinline__ int find_token_owner(const int32_t* cu, int nreq, int t) {
  const int l = lane_id();
  int lo = 0, n = nreq;  // cu[lo] <= t < cu[lo + n]
  while (n > 1) {
    const int step = (n + 63) / 64;
    const bool in = l * step < n;
    const int v = in ? cu[lo + l * step] : 0;
    const int j = __popcll(__ballot(in && v <= t)) - 1;
    lo += j * step;
    n = min(step, n - j * step);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Append writer: the waves of a token take 64 16-byte chunks of its K row (even
// waves) or its V row (odd ones) each; workgroup b holds kKvaWaves waves of token
// b / head_groups, counted from the first request's first.
template <typename TI, typename TO, int D>
__global__ __launch_bounds__(64 * kKvaWaves) void kv_append_kernel(KvWriteArgs<TI, TO> a) {
  using W = PageWrite<TI, TO, D>;
  using Out = typename W::Out;
  constexpr int EPC = W::EPC;
  __shared__ __attribute__((aligned(16))) TO s[kKvaWaves][64 * EPC];
  const int l = lane_id(), wl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int b = grid_block(blockIdx.x, blockIdx.y);
  int t = b / a.head_groups;
  if (t >= a.total_new) return;  // uniform
  const int w = b % a.head_groups * kKvaWaves + wl;
  const int half = a.hkv * W::CPR;  // chunks of a row
  const bool is_v = w & 1;
  const int c0 = 64 * (w >> 1), i = c0 + l;
  if (c0 >= half) return;
  const int h = i / W::CPR, c = i % W::CPR;
  const bool on = i < half;
  u32x4 x = {0, 0, 0, 0};
  float scale = 1.f;
  auto row = [&] {
    x = *reinterpret_cast<const u32x4*>((is_v ? a.v_new : a.k_new) + ((int64_t)t * a.hkv + h) * D + EPC * c);
  };
  if (on) {
    row();  // beside the lengths: nearly every call's rows start at 0
    if constexpr (W::kE4m3) scale = is_v ? a.v_scale[h] : a.k_scale[h];
  }
  const int first = a.cu_new[0];
  t += first;
  if (t >= a.cu_new[a.nreq]) return;  // uniform
  if (first != 0 && on) row();
  const int r = find_token_owner(a.cu_new, a.nreq, t);
  const int pos = a.start_pos[r] + (t - a.cu_new[r]);
  const int64_t page = a.page_table[(int64_t)r * a.pt_stride + pos / kPage];
  const Out y = W::convert(x, W::kE4m3 ? 1.0f / scale : 1.f);
  const int slot = pos % kPage;
  if (!is_v) {
    if (on)
      __builtin_nontemporal_store(y, reinterpret_cast<Out*>(a.k_pool + (page * a.hkv + h) * (kPage * D) +
                                                            slot * D + EPC * c));
    return;
  }
  // V elements lie a page row apart: through this wave's LDS, so that the lanes
  // of a store take neighbouring dims (a quarter to an eighth of the cache lines
  // of a store by which each lane writes its own chunk).
  *reinterpret_cast<Out*>(s[wl] + EPC * l) = y;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  TO* d = a.v_pool + (page * a.hkv * D + c0 * EPC + l) * kPage + slot;
#pragma unroll
  for (int u = 0; u < EPC; ++u)
    if (c0 * EPC + 64 * u < a.hkv * D) d[64 * kPage * u] = s[wl][64 * u + l];  // (a row is whole 64s)
}

}  // namespace dopd
