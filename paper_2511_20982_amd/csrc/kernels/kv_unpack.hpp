// Handoff unpack on the receiving instance: scatters a packed
// (layer, K/V, head, token, dim) buffer into the local page pools, the inverse
// of kv_pack.  Slots past the request's length are never touched.
//
// bf16 and fp32 pools: one workgroup per (page, handoff, layer*2*Hkv + kv*Hkv +
// head); K rows are copied as they are, V rows are transposed to the dim-major
// page block through LDS.  E4M3 pools: the page writer's mapping, a wave for the
// K or V of one (handoff, layer, page) and HW heads, which turns V four tokens at
// a time in registers (16 one-byte LDS reads a V run are what it saves).
// HBM-bound at size.  Measured, workgroup per block / wave per page, 8 requests of
// 300-900 tokens, 20 layers, buffer from HBM: E4M3 8 heads of 128 112 / 79 us, 32
// heads 434 / 309, 8 heads of 64 100 / 41; bf16 of d 128 4 heads 67 / 78, 8 heads
// 135 / 155, 32 heads 577 / 609; fp32 8 heads of 128 273 / 317, of 64 134 / 156.
// (bf16 of d 64, 104 / 78 and 32 heads 405 / 309, would gain from the second.)
#pragma once
#include "kv_pack.hpp"
#include "kv_write.hpp"

namespace dopd {

// STREAM: streaming loads, for buffers of more than kHandoffStreamBytes.
template <typename T, int D, bool STREAM>
__global__ __launch_bounds__(256) void kv_unpack_kernel(
    const T* __restrict__ in, const int64_t* __restrict__ in_off, const int32_t* __restrict__ req_ids,
    const int32_t* __restrict__ seq_lens, T* __restrict__ k_pool, T* __restrict__ v_pool,
    int num_pages, const int32_t* __restrict__ page_table, int pt_stride, int hkv) {
  constexpr int kEl = 16 / sizeof(T);
  constexpr int CPR = D / kEl;   // 16-byte chunks per token row
  constexpr int TP = D + kEl;    // padded LDS row (elements)
  __shared__ __attribute__((aligned(16))) T s_v[kPage * TP];
  const int pg = blockIdx.x, n = blockIdx.y, z = blockIdx.z, tid = threadIdx.x;
  const int len = seq_lens[n];
  if (pg * kPage >= len) return;  // uniform for the workgroup
  const int layer = z / (2 * hkv);
  const int kv = (z / hkv) % 2;
  const int h = z % hkv;
  const int r = req_ids[n];
  const int64_t page = page_table[(int64_t)r * pt_stride + pg];
  const int nvalid = min(kPage, len - pg * kPage);
  const int64_t lpage = (int64_t)layer * num_pages + page;
  const T* src = in + in_off[n] + ((((int64_t)layer * 2 + kv) * hkv + h) * len + (int64_t)pg * kPage) * D;
  const bool aligned = ((reinterpret_cast<uintptr_t>(src) & 15) == 0);
  auto chunk = [&](int i) {
    const u32x4* p = reinterpret_cast<const u32x4*>(src) + i;
    return STREAM ? __builtin_nontemporal_load(p) : *p;
  };

  if (kv == 0) {
    T* dst = k_pool + (lpage * hkv + h) * kPage * D;
    if (aligned) {
      // streaming stores (here and below): the pages leave the caches now,
      // not as write-back during the kernels that follow
      for (int i = tid; i < nvalid * CPR; i += 256)
        __builtin_nontemporal_store(chunk(i), reinterpret_cast<u32x4*>(dst) + i);
    } else {
      for (int i = tid; i < nvalid * D; i += 256) dst[i] = src[i];
    }
    return;
  }
  // V: token rows into LDS, then dim rows of the page's slots.
  if (aligned) {
    for (int i = tid; i < nvalid * CPR; i += 256) {
      const int t = i / CPR, c = i % CPR;
      *reinterpret_cast<u32x4*>(&s_v[t * TP + c * kEl]) = chunk(i);
    }
  } else {
    for (int i = tid; i < nvalid * D; i += 256) s_v[(i / D) * TP + i % D] = src[i];
  }
  __syncthreads();
  T* vdst = v_pool + (lpage * hkv + h) * D * kPage;
  constexpr int RUNS = kPage / kEl;  // 16-byte runs per dim row
  for (int i = tid; i < D * RUNS; i += 256) {
    const int e = i / RUNS, run = i % RUNS;
    T* drow = vdst + e * kPage + run * kEl;
    if (nvalid == kPage) {
      u32x4 x;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if constexpr (sizeof(T) == 2) {
          const int s = run * kEl + 2 * w;
          x[w] = (uint32_t)s_v[s * TP + e] | ((uint32_t)s_v[(s + 1) * TP + e] << 16);
        } else {
          x[w] = s_v[(run * kEl + w) * TP + e];
        }
      }
      __builtin_nontemporal_store(x, reinterpret_cast<u32x4*>(drow));
    } else {
      for (int k = 0; k < kEl; ++k) {
        const int s = run * kEl + k;
        if (s < nvalid) drow[k] = s_v[s * TP + e];
      }
    }
  }
}

struct UnpackPagesArgs {
  const uint8_t* in;
  const int64_t* in_off;      // [nhand] element offset of each handoff's block
  const int32_t* req_ids;     // [nhand] page-table rows
  const int32_t* seq_lens;    // [nhand]
  uint8_t* k_pool;            // [layers][P][Hkv][16][D]
  uint8_t* v_pool;            // [layers][P][Hkv][D][16]
  const int32_t* page_table;
  int num_pages, pt_stride, hkv, nhand, layers;
  int head_groups;            // workgroups of a page of one layer
};

// Workgroup b: heads of group b % head_groups of the (b / head_groups)-th
// (handoff, layer, page), pages fastest.
template <int D>
__global__ __launch_bounds__(64 * kKvwWaves) void kv_unpack_pages_kernel(UnpackPagesArgs a) {
  using T = uint8_t;
  using W = PageWrite<T, T, D>;
  __shared__ __attribute__((aligned(16))) uint8_t s[kKvwWaves / 2][W::kLdsBytes];  // of the V waves
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int b = grid_block(blockIdx.x, blockIdx.y);
  const int wi = b % a.head_groups * kKvwWaves + w;  // wave of the page: K's, V's, ..
  const int h0 = (wi >> 1) * W::HW;
  if (h0 >= a.hkv) return;
  int len_l = 0, req_l = 0;  // this lane's handoff
  auto items = [&](int x) {
    len_l = a.seq_lens[x];
    req_l = a.req_ids[x];
    return a.layers * ((len_l + kPage - 1) / kPage);
  };
  int n, local;
  if (!find_owner(b / a.head_groups, a.nhand, items, n, local)) return;
  const int len = __builtin_amdgcn_readlane(len_l, n % 64), r = __builtin_amdgcn_readlane(req_l, n % 64);
  const int np = (len + kPage - 1) / kPage, layer = local / np, pg = local % np;
  const int64_t page = (int64_t)layer * a.num_pages + a.page_table[(int64_t)r * a.pt_stride + pg];
  const int64_t half = (int64_t)a.hkv * len * D;  // elements of a layer's K or V
  const T* k_src = a.in + a.in_off[n] + layer * 2 * half + (int64_t)pg * kPage * D;
  const int64_t row_elems = D, head_elems = (int64_t)len * D, page_elems = (int64_t)a.hkv * (kPage * D);
  const int s1 = min(kPage, len - pg * kPage);
  if (wi & 1)
    write_page_rows<T, T, D, false, true>(k_src + half, row_elems, head_elems, h0, a.hkv, 0, s1,
                                          a.v_pool + page * page_elems, nullptr, (T*)nullptr, 0, false, s[w >> 1]);
  else
    write_page_rows<T, T, D, false, false>(k_src, row_elems, head_elems, h0, a.hkv, 0, s1,
                                           a.k_pool + page * page_elems, nullptr, (T*)nullptr, 0, false, nullptr);
}

}  // namespace dopd
