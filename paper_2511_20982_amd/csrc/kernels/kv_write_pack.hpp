// Paged KV write of fresh prompts that also emits their handoff buffer.
//
// A prefill-completed request's cache is exactly the K/V rows its prefill
// just produced, so the handoff buffer ((K/V, head, token, dim) order, one
// layer) can be written from the same fresh rows the paged write reads,
// instead of gathering the pages back from the pool afterwards: every K/V byte
// is read once and written twice (pool page and handoff buffer), in one
// launch.  The page writer's mapping (a wave takes K or V of a (page, KV head)), start
// position 0 for every request (fresh prompts).  Slots of a request's last
// page past its length are never touched.
#pragma once
#include "kv_write.hpp"

namespace dopd {

struct WritePackArgs {
  const uint16_t* k_new;      // [T][Hkv][D] bf16
  const uint16_t* v_new;      // [T][Hkv][D]
  void* k_pool;               // [P][Hkv][16][D] bf16, or E4M3 codes
  void* v_pool;               // [P][Hkv][D][16]
  const int32_t* page_table;  // [nreq][pt_stride] (rows of these requests)
  int pt_stride;
  const int32_t* cu;          // [nreq + 1] rows of each request in k_new / v_new
  int nreq, hkv;
  int head_groups;            // workgroups of a page
  void* out;                  // handoff buffer (pool elements), or null (paged write only)
  const int64_t* out_off;     // [nreq] element offset of each request's block
  const float* k_scale;       // [Hkv], E4M3 pools only
  const float* v_scale;       // [Hkv]
};

// Workgroup b: heads of group b % head_groups of logical page b / head_groups of
// the concatenated page lists, K and V in waves of their own (a page's waves of K
// come first), or BOTH one after the other in a wave.  The fused step takes the
// latter: its writer workgroups hold slots the prefill waits for, and twice as many
// of them cost more than their shorter life gives (mixed step 220.5 against 216.9
// us, E4M3 142.7 against 138.5).  K and V of the same heads side by side would store
// to handoff rows and pages that are a power of two apart when a prompt's length is:
// 8 prompts of 512, d 64, 8 / 16 heads 6.3 / 9.8 us against 4.8 / 7.8 (BOTH 5.1 /
// 7.4, but one prompt of 20 tokens 4.4 against 3.4).  s: this wave's
// PageWrite<...>::kLdsBytes of LDS.
template <typename TO, int D, bool BOTH>
__device__ __forceinline__ void kv_write_pack_workgroup(const WritePackArgs& a, int b, uint8_t* s) {
  using W = PageWrite<uint16_t, TO, D>;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nk = (a.hkv + W::HW - 1) / W::HW;        // waves of a page's K
  const int wi = b % a.head_groups * kKvwWaves + w;  // wave of the page: K's, then V's (or both)
  if (wi >= (BOTH ? nk : 2 * nk)) return;
  const bool is_v = wi >= nk;
  const int h0 = (is_v ? wi - nk : wi) * W::HW;
  int cu_l = 0, n_l = 0;  // this lane's request
  auto pages = [&](int rr) {
    cu_l = a.cu[rr];
    n_l = a.cu[rr + 1] - cu_l;
    return (n_l + kPage - 1) / kPage;
  };
  int r, lp;
  if (!find_owner(b / a.head_groups, a.nreq, pages, r, lp)) return;
  const int row0 = __builtin_amdgcn_readlane(cu_l, r % 64), n = __builtin_amdgcn_readlane(n_l, r % 64);
  const int s1 = min(kPage, n - lp * kPage);  // live slots [0, s1) of this page
  const int64_t page = a.page_table[(int64_t)r * a.pt_stride + lp];
  const int64_t row_elems = (int64_t)a.hkv * D;
  const int64_t src = ((int64_t)row0 + lp * kPage) * row_elems;
  TO* pk = nullptr;
  TO* pv = nullptr;
  bool aligned = false;
  if (a.out) {
    const int64_t base = a.out_off[r];
    pk = static_cast<TO*>(a.out) + base + (int64_t)lp * kPage * D;
    pv = pk + (int64_t)a.hkv * n * D;
    // the rest of a chunk's offset is a multiple of its size
    aligned = (reinterpret_cast<uintptr_t>(pk) & (sizeof(typename W::Out) - 1)) == 0;
  }
  const int64_t page_elems = (int64_t)a.hkv * (kPage * D);
  if (BOTH || !is_v)
    write_page_rows<uint16_t, TO, D, true, false>(a.k_new + src, row_elems, D, h0, a.hkv, 0, s1,
                                                  static_cast<TO*>(a.k_pool) + page * page_elems, a.k_scale, pk,
                                                  (int64_t)n * D, aligned, s);
  if (BOTH || is_v)
    write_page_rows<uint16_t, TO, D, true, true>(a.v_new + src, row_elems, D, h0, a.hkv, 0, s1,
                                                 static_cast<TO*>(a.v_pool) + page * page_elems, a.v_scale, pv,
                                                 (int64_t)n * D, aligned, s);
}

template <int D>
__global__ __launch_bounds__(64 * kKvwWaves) void kv_write_pack_kernel(WritePackArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t s[kKvwWaves][PageWrite<uint16_t, uint16_t, D>::kLdsBytes];
  kv_write_pack_workgroup<uint16_t, D, false>(a, (int)blockIdx.x, s[threadIdx.x >> 6]);
}

}  // namespace dopd
