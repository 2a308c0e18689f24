// fp32 attention (prefill, chunk prefill and decode): fp32 operands, products
// and sums throughout, on the fp32 matrix instruction.
//
// The query rows of one request that read one KV head form columns: column ci
// is chunk row ci / g, query head c * g + ci % g (a decode step is a chunk of
// one row), and sees cached positions 0 .. prefix + ci / g.  A workgroup takes
// 16 columns; its W waves take the 16-key tiles w, w + W, ... and merge through
// LDS.  Per tile and wave
//   S^T[16 keys][16 cols] = K[16][d] . Q^T[d][16]     d / 4 v_mfma_f32_16x16x4_f32
//   O^T[d][16 cols]      += V^T[d][16] . P^T[16][16]  (d / 16) x 4 of them
// A contraction index may be permuted when both operands agree: a lane reads a
// run of d / 4 elements of one K row, and the S^T accumulator (keys 4 (l / 16)
// + 0..3) is the P^T operand as it stands.  The next tile's loads are in flight
// while a tile is computed.
//
// Bound by latency at small sizes: the columns share each K/V load and the
// waves share the keys, so a 120-key row is two tiles deep (one wave per (row,
// head) that visited key after key took 0.3 - 0.45 us a key).  Six prompts of
// 60-120 tokens, 8/2 heads, d 64: prefill 43 -> 7.8 us, their decode 43 -> 6.5;
// of 500-1000 tokens, 64/8 heads, d 128: 7.4 -> 0.86 ms and 530 -> 36 us.  Up to
// about 5 tokens that wave was faster (3.5-4.2 us; here 5-6: a tile's products
// and a longer program).
//
// Rounding: a score's products are added eight at a time and then pair by pair
// (one chain of d / 2, as two accumulators over all of d make it, left outputs at
// d 128 a third further from 64 bits than sums over a wave's lanes: six prompts
// of 8-16 tokens 1.12e-7 against 0.80e-7, now 0.77e-7; of 60-120 tokens 1.71e-7
// against 1.44e-7, now 1.13e-7), and the division by the row sum rounds once.
//
// Keys past a column's limit are masked by select in S^T, and V of positions
// past the request's last key is replaced by 0.  A tile some columns see and
// others do not whose V holds a NaN or an infinity is added key by key with
// selects, so that no column takes 0 * inf from a key it does not see.
#pragma once
#include "common.hpp"
#include "../plan.hpp"

namespace dopd {

// Elements of the caller's fp32 arrays are aligned to 4 bytes only.
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4 load_f32x4(const float* p) { return *reinterpret_cast<const f32x4_a4*>(p); }

__device__ __forceinline__ void load_to(float* d, const float* p) {
  const f32x4 x = load_f32x4(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = x[i];
}

struct AttnF32Args {
  const float* q;             // [T][Hq][D]
  const float* k;             // fresh rows [T][Hkv][D], or the pool [P][Hkv][16][D]
  const float* v;             // fresh rows [T][Hkv][D], or the pool [P][Hkv][D][16]
  const int32_t* page_table;  // pools only: [nreq][pt_stride]
  // Chunk rows of request r: [cu[r], cu[r + 1]); null: one row each, row r.
  const int32_t* cu;
  // Keys before the chunk: prefix[r] (null: 0).  One row each: ctx[r] - 1.
  const int32_t* prefix;
  const int32_t* ctx;
  float* out;                 // [T][Hq][D]
  float* lse;                 // [T][Hq] or null
  int pt_stride, nreq, hq, hkv;
  float scale;
};

// x / y for several x: 1 / y in two parts, so that the quotient is rounded about
// once (x * (1 / y) is rounded twice).
struct F32Quot {
  float inv, low;
  __device__ __forceinline__ explicit F32Quot(float y) : inv(1.f / y), low(fmaf(-inv, y, 1.f) * inv) {}
  __device__ __forceinline__ float operator()(float x) const {
    return fabsf(x) < INFINITY ? fmaf(x, inv, x * low) : x * inv;
  }
};

constexpr int kF32Cols = 16;  // columns of a workgroup
constexpr int kF32Keys = 16;  // keys of a tile (one page)

// Waves of a workgroup: eight at d = 64; four at d = 128, whose two buffered
// tiles leave a wave no fewer than 256 registers.  Either way two waves share a
// SIMD, so that calls of more workgroups than CUs run at once (d 128 at one wave:
// 6 prompts of 8-16 tokens, 64/8 heads, 14.7 us against 9.6; of 500-1000 tokens
// 1240 against 855).  The tiles are scalars, not vectors: as vectors, whose
// registers have to lie side by side, 22-34 of them were spilled.
template <int D>
constexpr int f32_waves() { return D == 64 ? 8 : 4; }

template <int D, bool PAGED, int W = f32_waves<D>()>
__global__ __launch_bounds__(64 * W, 8 / W) void attn_f32_kernel(AttnF32Args a) {
  constexpr int KR = D / 4;     // elements of a K row one lane holds
  constexpr int NT = D / 16;    // O^T tiles of 16 dims
  constexpr int OP = D + 4;     // padded row of the merge buffer
  __shared__ float s_o[W][kF32Cols][OP];
  __shared__ float s_m[W][kF32Cols], s_l[W][kF32Cols];
  const int l = lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int hq = a.hq, hkv = a.hkv, g = hq / hkv;

  // Block: (request, column tile, KV head), the last column tiles (the most
  // keys) of a request first.
  auto tiles_of = [&](int rows) { return (rows * g + kF32Cols - 1) / kF32Cols; };
  int row_l = 0, n_l = 0, pre_l = 0;  // this lane's request
  auto items = [&](int x) {
    row_l = a.cu ? a.cu[x] : x;
    n_l = a.cu ? a.cu[x + 1] - row_l : 1;
    pre_l = a.ctx ? a.ctx[x] - 1 : (a.prefix ? a.prefix[x] : 0);
    return tiles_of(n_l) * hkv;
  };
  int r, local;
  if (!find_owner(grid_block(blockIdx.x, blockIdx.y), a.nreq, items, r, local)) return;  // uniform
  const int L = __builtin_amdgcn_readlane(n_l, r % 64), row0 = __builtin_amdgcn_readlane(row_l, r % 64);
  const int P = __builtin_amdgcn_readlane(pre_l, r % 64);
  const int c = local % hkv;
  const int ncols = L * g;
  const int col0 = (tiles_of(L) - 1 - local / hkv) * kF32Cols;
  const int cl = l & 15, qg = l >> 4;
  const int ci = min(col0 + cl, ncols - 1);  // (columns past the end repeat the last; not stored)
  const int limit = P + ci / g;              // last key this lane's column sees
  const int first_limit = P + col0 / g;      // last key every column sees
  const int nkeys = P + (min(col0 + kF32Cols, ncols) - 1) / g + 1;
  const int ntiles = (nkeys + kF32Keys - 1) / kF32Keys;
  // One tile: wave 0 stores its result, with no merge (9.6 -> 6.8 us on the 6
  // prompts of 8-16 tokens above).
  if (ntiles == 1 && w > 0) return;

  // Q^T operand of step i: Q[col][KR qg + i].
  float qv[KR];
  {
    const float* qp = a.q + ((int64_t)(row0 + ci / g) * hq + c * g + ci % g) * D + KR * qg;
#pragma unroll
    for (int i = 0; i < KR; i += 4) load_to(qv + i, qp + i);
  }

  // Dim of O^T tile n, row x: fresh V rows are read NT dims at a time, pool
  // rows (dim-major) a dim at a time.
  auto dim_of = [](int n, int x) { return PAGED ? 16 * n + x : NT * x + n; };
  const int32_t* pt = PAGED ? a.page_table + (int64_t)r * a.pt_stride : nullptr;
  struct Tile {
    float k[KR];     // K[key l % 16][KR qg + 0 ..]
    float v[NT][4];  // v[n][j] = V[key 4 qg + j][dim_of(n, l % 16)]
  };
  // Positions past the last key read the last one (fresh) or their page slot,
  // which may hold anything (pools).
  auto load = [&](Tile& t, int kt) {
    if constexpr (PAGED) {
      const int64_t blk = ((int64_t)pt[kt] * hkv + c) * (kPage * D);
      const float* kp = a.k + blk + cl * D + KR * qg;
#pragma unroll
      for (int i = 0; i < KR; i += 4) load_to(t.k + i, kp + i);
      const float* vp = a.v + blk + 4 * qg;
#pragma unroll
      for (int n = 0; n < NT; ++n) load_to(t.v[n], vp + dim_of(n, cl) * kPage);
    } else {
      const int key = min(kt * kF32Keys + cl, nkeys - 1);
      const float* kp = a.k + ((int64_t)(row0 + key) * hkv + c) * D + KR * qg;
#pragma unroll
      for (int i = 0; i < KR; i += 4) load_to(t.k + i, kp + i);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kj = min(kt * kF32Keys + 4 * qg + j, nkeys - 1);
        const float* vp = a.v + ((int64_t)(row0 + kj) * hkv + c) * D + NT * cl;
#pragma unroll
        for (int n = 0; n < NT; n += 4) {
          const f32x4 x = load_f32x4(vp + n);
#pragma unroll
          for (int i = 0; i < 4; ++i) t.v[n + i][j] = x[i];
        }
      }
    }
  };

  f32x4 o[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;  // of this lane's column; lsum of its own keys only

  auto compute = [&](Tile& t, int kt) {
    f32x4 sum[KR / 2];  // of eight products each, then added pair by pair
#pragma unroll
    for (int i = 0; i < KR / 2; ++i) {
      sum[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[2 * i], qv[2 * i], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      sum[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[2 * i + 1], qv[2 * i + 1], sum[i], 0, 0, 0);
#pragma unroll
      for (int b = 1; (i + 1) % (2 * b) == 0; b *= 2) sum[i + 1 - 2 * b] += sum[i + 1 - b];
    }
    const int key0 = kt * kF32Keys + 4 * qg;  // this lane's keys key0 .. key0 + 3
    f32x4 s = sum[0] * a.scale;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (key0 + j > limit) s[j] = -INFINITY;
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx);
    const float base = m_new == -INFINITY ? 0.f : m_new;  // (no visible key so far: p = 0)
    const float alpha = expf(m - base);
    f32x4 p;
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = expf(s[j] - base);
    lsum = lsum * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
    m = m_new;
#pragma unroll
    for (int n = 0; n < NT; ++n) o[n] *= alpha;
    bool odd = false;
    if (kt * kF32Keys + kF32Keys - 1 > first_limit) {  // uniform: some column does not see all keys
      bool bad = false;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (key0 + j >= nkeys) t.v[n][j] = 0.f;
          bad |= !(fabsf(t.v[n][j]) < INFINITY);
        }
      odd = __ballot(bad) != 0;
    }
    if (!odd) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < NT; ++n)
          o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.v[n][j], p[j], o[n], 0, 0, 0);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        for (int src = 0; src < 4; ++src) {  // key 4 src + j of the tile
          const float pk = __shfl(p[j], 16 * src + cl, 64);
          const bool seen = kt * kF32Keys + 4 * src + j <= limit;
#pragma unroll
          for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int x = 0; x < 4; ++x) {  // V[key][dim_of(n, 4 qg + x)] is lane 16 src + 4 qg + x's
              const float vk = __shfl(t.v[n][j], 16 * src + 4 * qg + x, 64);
              o[n][x] = seen ? o[n][x] + pk * vk : o[n][x];
            }
        }
    }
  };

  if (w < ntiles) {
    Tile t0, t1;
    load(t0, w);
    for (int kt = w; kt < ntiles; kt += 2 * W) {
      if (kt + W < ntiles) load(t1, kt + W);
      compute(t0, kt);
      if (kt + W >= ntiles) break;
      if (kt + 2 * W < ntiles) load(t0, kt + 2 * W);
      compute(t1, kt + W);
    }
  }
  lsum += __shfl_xor(lsum, 16, 64);
  lsum += __shfl_xor(lsum, 32, 64);
  // The lane anew: held over the loop it costs registers the tiles need.
  int le;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(le));
  const int ce = le & 15, qe = le >> 4;
  if (ntiles == 1) {
    const int cx = col0 + ce;
    if (cx >= ncols) return;
    lsum += m - m;  // (no finite score: NaN, as the merge below has it)
    const F32Quot quot(lsum);
    const int64_t row = (int64_t)(row0 + cx / g) * hq + c * g + cx % g;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) a.out[row * D + dim_of(n, 4 * qe + j)] = quot(o[n][j]);
    if (a.lse && qe == 0) a.lse[row] = m + logf(lsum);
    return;
  }
  if (qe == 0) {
    s_m[w][ce] = m;
    s_l[w][ce] = lsum;
  }
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int j = 0; j < 4; ++j) s_o[w][ce][dim_of(n, 4 * qe + j)] = o[n][j];
  __syncthreads();
  const int live = min(kF32Cols, ncols - col0);
  for (int i = 64 * w + le; i < live * D; i += 64 * W) {
    const int x = i / D, e = i % D, cx = col0 + x;
    float M = s_m[0][x];
#pragma unroll
    for (int u = 1; u < W; ++u) M = fmaxf(M, s_m[u][x]);
    float sum = 0.f, acc = 0.f;
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const float f = expf(s_m[u][x] - M);  // a wave that saw no key of the column: 0
      sum += f * s_l[u][x];
      acc += f * s_o[u][x][e];
    }
    const int64_t row = (int64_t)(row0 + cx / g) * hq + c * g + cx % g;
    a.out[row * D + e] = F32Quot(sum)(acc);
    if (a.lse && e == 0) a.lse[row] = M + logf(sum);
  }
}

}  // namespace dopd
