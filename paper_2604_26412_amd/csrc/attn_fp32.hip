// Draft attention for float32 inputs on the float32 matrix instruction
// v_mfma_f32_16x16x4_f32: every product and sum is a float32 one, as on the
// vector ALU, at 4 x its rate and without its cross-lane score reductions.
//
// One workgroup of 8 waves serves RT 16-row query tiles of one (sequence, KV
// head, split).  Each wave takes every eighth 16-key block of the split with
// its own online-softmax state, and the eight states are merged through LDS at
// the end, in wave order.
//
// Operands need no LDS.  The reduction index of a product may be permuted as
// long as both operands agree, so a lane's four channels per load are adjacent:
//   S^T = K Q^T  lane (i = lane % 16, g = lane / 16) holds channels
//                16 u + 4 g + e of key / query row i (u = 0..7, e = 0..3): eight
//                16-byte loads of one row, RoPE partners (u, u + 4) in one lane.
//   O^T = V^T P^T  accumulator register v of S^T is key 4 g + v of row i, which
//                is already the second product's operand; V lanes hold channels
//                4 i + 64 t + e of key 4 g + v (t = 0, 1): 256-byte segments.
// The next block's keys are loaded once this block's scores are formed, its
// values once this block's values are used.
//
// What bounds it: 64 products of 32 clocks a block and row tile, against 16 KB
// of K/V: the matrix rate from 32 rows on, the stream below, and for small calls
// the chain of dependent loads (length, page id, keys) and of a wave's blocks.
// Against the vector-ALU kernel that served these inputs before (it reduces each
// score over 16 lanes and walks the page table for every key and row), whole
// calls of 8 KV heads: 1 x 256 keys, 16 rows 64 -> 16 us; 4 x 2048 keys, 16 rows
// 112 -> 21 us (2.8 TB/s); 16 x 4096 keys, 32 rows 2082 -> 119 us (4.5 TB/s);
// 4 x 4096 keys, 128 rows 1792 -> 102 us (84 TFLOP/s of 150).
#include "kvshot_common.h"

namespace kvshot {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLn2 = 0.693147180559945309f;
constexpr int kWaves = 8;
constexpr int kKeys = 16;    // keys per block: never more than a page, so a block has one page id

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Table entries of one row's channels 16 u + 4 g + e (u < 4), and the rotation by them.
__device__ __forceinline__ void load_cs(const float2* row, int g, f32x4 (&cs)[8]) {
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int i = 0; i < 2; ++i) cs[2 * u + i] = *(const f32x4*)(row + 16 * u + 4 * g + 2 * i);
}
__device__ __forceinline__ void rotate(f32x4 (&x)[8], const f32x4 (&cs)[8]) {
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = cs[2 * u + e / 2][2 * (e & 1)], s = cs[2 * u + e / 2][2 * (e & 1) + 1];
      const float lo = x[u][e], hi = x[u + 4][e];
      x[u][e] = lo * c - hi * s;
      x[u + 4][e] = hi * c + lo * s;
    }
}

template <int RT>
__global__ __launch_bounds__(64 * kWaves) void attn_fp32_kernel(AttnParams p) {
  __shared__ float sh_o[kWaves][RT * 16][kHeadDim];
  __shared__ float2 sh_ml[kWaves][RT * 16];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15;   // query row of the tile (key row for K, channel group for V)
  const int g = lane >> 4;

  // (row group, split) fastest: the workgroups that read one prefix run on one XCD
  int id = xcd_remap((int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x),
                     (int)(gridDim.x * gridDim.y * gridDim.z));
  const int rg = id % p.row_groups;
  id /= p.row_groups;
  const int split = id % p.splits;
  id /= p.splits;
  const int h = id % p.hkv, b = id / p.hkv;

  // query rows first: their loads wait for nothing
  f32x4 qx[RT][8];
  int row_j[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rc = min((rg * RT + rt) * 16 + i16, p.rows - 1);
    row_j[rt] = rc / p.group;
    const int hq = h * p.group + (rc - row_j[rt] * p.group);
    const float* qr = (const float*)p.q + (((int64_t)b * p.nq + row_j[rt]) * p.hq + hq) * kHeadDim + 4 * g;
#pragma unroll
    for (int u = 0; u < 8; ++u) qx[rt][u] = *(const f32x4*)(qr + 16 * u);
  }

  int T = clamp_ctx(p.ctx_lens[b], p.max_pages_per_seq, p.page_shift);
  T = T > p.max_ctx ? p.max_ctx : T;
  int s0 = 0, S = p.tree ? p.n_nodes : p.nq;
  if (!p.tree) {
    s0 = p.step_offsets[b];
    s0 = s0 < 0 ? 0 : (s0 > p.max_draft - p.nq ? p.max_draft - p.nq : s0);
    S = s0 + p.nq;
  }
  const int P = position_base(p, b, T);
  const int key_beg = split * p.blocks_per_split * kBlockKeys;
  const int key_end = min(key_beg + p.blocks_per_split * kBlockKeys, T);
  const int nblk = key_end > key_beg ? (key_end - key_beg + kKeys - 1) / kKeys : 0;
  const bool last = split == p.splits - 1;
  const float* kp = (const float*)p.k_pages;
  const float* vp = (const float*)p.v_pages;
  const int pmask = (1 << p.page_shift) - 1;

  // page ids of this wave's next 64 blocks, one per lane
  int pids = 0;
  auto load_pids = [&](int blk) {
    const int mine = blk + lane * kWaves;
    if (mine < nblk)
      pids = physical_page(p.page_table, b, p.max_pages_per_seq, (key_beg + mine * kKeys) >> p.page_shift,
                           p.num_pages);
  };

  // This wave's blocks: prefix blocks wave, wave + 8, ..., then (last split) draft blocks 7 - wave, ...
  // Rows past the end of either range repeat its last row: their weights are
  // zero, and a zero times whatever an unused slot holds would not be.
  bool draft = false;
  int blk = wave, pid = 0;
  auto to_draft = [&]() {   // after the last prefix block; returns whether a draft block is left
    draft = true;
    blk = kWaves - 1 - wave;
    return last && blk * kKeys < S;
  };
  f32x4 kx[8], vx[4][2];
  auto load_k = [&]() {
    const float* r;
    if (draft) {
      r = (const float*)p.draft_k + draft_offset(b, min(blk * kKeys + i16, S - 1), h, p.max_draft, p.hkv);
    } else {
      const int key = min(key_beg + blk * kKeys + i16, key_end - 1);
      r = kp + kv_offset(pid, h, key & pmask, p.page_stride, p.head_stride, p.slot_stride);
    }
    r += 4 * g;
#pragma unroll
    for (int u = 0; u < 8; ++u) kx[u] = *(const f32x4*)(r + 16 * u);
  };
  auto load_v = [&]() {
    const int64_t stride = draft ? (int64_t)p.hkv * kHeadDim : p.slot_stride;
    const int first = draft ? blk * kKeys : (key_beg + blk * kKeys) & pmask;   // row of the block's first key
    const int left = draft ? S - blk * kKeys : key_end - (key_beg + blk * kKeys);
    const float* base = draft ? (const float*)p.draft_v + draft_offset(b, 0, h, p.max_draft, p.hkv)
                              : vp + kv_offset(pid, h, 0, p.page_stride, p.head_stride, p.slot_stride);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* r = base + (first + min(4 * g + v, left - 1)) * stride + 4 * i16;
      vx[v][0] = *(const f32x4*)r;
      vx[v][1] = *(const f32x4*)(r + 64);
    }
  };
  bool more = blk < nblk;
  if (more) {
    load_pids(blk);
  } else {
    more = to_draft();
  }

  uint64_t anc_mine = 0;
  int depth_mine = 0;
  if (p.tree) anc_mine = tree_ancestry_wave(p.parents + (int64_t)b * p.n_nodes, p.n_nodes, lane, &depth_mine);
  auto clamp_pos = [&](int pos) { return pos >= p.max_position ? p.max_position - 1 : pos; };

  // table rows of the queries' positions, and the draft keys each row may see
  f32x4 cs[RT][8];   // (cos, sin) pairs of channels 16 u + 4 g + (0, 1) and + (2, 3)
  uint64_t sees[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    int qpos = P + s0 + row_j[rt];
    if (p.tree) {
      const int node = query_node(p, b, row_j[rt]);
      const uint32_t lo = __shfl((uint32_t)anc_mine, node), hi = __shfl((uint32_t)(anc_mine >> 32), node);
      sees[rt] = ((uint64_t)hi << 32) | lo;
      qpos = P + __shfl(depth_mine, node);
    } else {
      sees[rt] = ~0ull >> (63 - (s0 + row_j[rt]));   // s0 + j <= max_draft - 1 <= 63
    }
    load_cs(p.rope + (int64_t)clamp_pos(qpos) * kHalfDim, g, cs[rt]);
  }
  if (more) {
    if (!draft) pid = __builtin_amdgcn_readlane(pids, 0);
    load_k();
    load_v();
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    rotate(qx[rt], cs[rt]);
#pragma unroll
    for (int u = 0; u < 8; ++u) qx[rt][u] *= p.qscale;
  }

  float m[RT], l[RT];
  f32x4 o[RT][8];   // o[rt][4 t + e][v]: channel 4 (4 g + v) + 64 t + e of row i16
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m[rt] = -INFINITY;
    l[rt] = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) o[rt][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  // Scores of the keys in kx, the new weights and the rescaled state.  Bit v of vis[rt]: this lane's
  // key 4 g + v is visible to its row.
  float pw[RT][4];
  auto scores = [&](const uint32_t (&vis)[RT]) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      f32x4 s[4];   // four short chains: less rounding than one of 32 products
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = mfma4(kx[u][e], qx[rt][u][e], s[e]);
      f32x4 sc = (s[0] + s[1]) + (s[2] + s[3]);
      float mb = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sc[v] = (vis[rt] >> v) & 1u ? sc[v] : -INFINITY;
        mb = fmaxf(mb, sc[v]);
      }
      mb = fmaxf(mb, __shfl_xor(mb, 16));
      mb = fmaxf(mb, __shfl_xor(mb, 32));
      const float mn = fmaxf(m[rt], mb);
      const float mu = mn == -INFINITY ? 0.0f : mn;
      const float alpha = exp2f(m[rt] - mu);
      m[rt] = mn;
      float ls = 0.0f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        pw[rt][v] = exp2f(sc[v] - mu);
        ls += pw[rt][v];
      }
      l[rt] = l[rt] * alpha + ls;   // this lane group's keys; the groups are summed at the end
#pragma unroll
      for (int c = 0; c < 8; ++c) o[rt][c] *= alpha;
    }
  };
  auto accumulate = [&]() {
    // A key of weight zero contributes nothing, also where its value is not
    // finite; in a product it would.  Such values are taken out of the operand
    // and added row by row where their weight is not zero, from a copy of the
    // block in this wave's part of the merge buffer.
    float chk = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) chk = __builtin_fmaf(vx[v][t][e], 0.0f, chk);
    if (__builtin_expect(__ballot(chk != 0.0f) != 0, 0)) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          *(f32x4*)&sh_o[wave][4 * g + v][4 * i16 + 64 * t] = vx[v][t];
#pragma unroll
          for (int e = 0; e < 4; ++e) vx[v][t][e] = vx[v][t][e] * 0.0f != 0.0f ? 0.0f : vx[v][t][e];
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
      for (int key = 0; key < kKeys; ++key) {
        float pk[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const float a = (key & 1) ? pw[rt][1] : pw[rt][0], c = (key & 1) ? pw[rt][3] : pw[rt][2];
          pk[rt] = __shfl((key & 2) ? c : a, 16 * (key >> 2) + i16);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const f32x4 val = *(const f32x4*)&sh_o[wave][key][16 * g + 4 * w + 64 * t];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int rt = 0; rt < RT; ++rt)
                if (val[e] * 0.0f != 0.0f && pk[rt] != 0.0f) o[rt][4 * t + e][w] += pk[rt] * val[e];
          }
      }
      __builtin_amdgcn_wave_barrier();   // the next block may reuse the buffer
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) o[rt][4 * t + e] = mfma4(vx[v][t][e], pw[rt][v], o[rt][4 * t + e]);
  };

  for (int n = 1; more; ++n) {
    uint32_t vis[RT];
    if (draft) {
      const int s = min(blk * kKeys + i16, S - 1);
      f32x4 kcs[8];
      load_cs(p.rope + (int64_t)clamp_pos(P + (p.tree ? __shfl(depth_mine, s) : s)) * kHalfDim, g, kcs);
      rotate(kx, kcs);
      const int sk = blk * kKeys + 4 * g;   // <= 60
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) vis[rt] = (uint32_t)(sees[rt] >> sk) & (S - sk >= 4 ? 15u : (1u << max(S - sk, 0)) - 1u);
    } else {
      const int left = key_end - (key_beg + blk * kKeys) - 4 * g;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) vis[rt] = left >= 4 ? 15u : (1u << max(left, 0)) - 1u;
    }
    scores(vis);
    blk += kWaves;
    more = draft ? blk * kKeys < S : blk < nblk;
    if (!more && !draft) {
      more = to_draft();
    } else if (more && !draft) {
      if ((n & 63) == 0) load_pids(blk);
      pid = __builtin_amdgcn_readlane(pids, n & 63);
    }
    if (more) load_k();
    accumulate();
    if (more) load_v();
  }

  // merge the waves: common maximum, then the scaled sums in wave order
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    l[rt] += __shfl_xor(l[rt], 16);
    l[rt] += __shfl_xor(l[rt], 32);
    if (g == 0) sh_ml[wave][rt * 16 + i16] = make_float2(m[rt], l[rt]);
  }
  __syncthreads();
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sh_ml[w][rt * 16 + i16].x);
    const float f = exp2f(m[rt] - (M == -INFINITY ? 0.0f : M));
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = l[rt] != 0.0f ? o[rt][4 * t + e][v] * f : 0.0f;
        *(f32x4*)&sh_o[wave][rt * 16 + i16][16 * g + 4 * v + 64 * t] = x;
      }
  }
  __syncthreads();
  for (int at = threadIdx.x; at < RT * 16 * (kHeadDim / 4); at += 64 * kWaves) {
    const int rl = at / (kHeadDim / 4), ch = (at % (kHeadDim / 4)) * 4;
    const int r = rg * RT * 16 + rl;
    if (r >= p.rows) continue;
    float M = -INFINITY, L = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sh_ml[w][rl].x);
    const float Mu = M == -INFINITY ? 0.0f : M;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float2 ml = sh_ml[w][rl];
      L += ml.y * exp2f(ml.x - Mu);
      acc += *(const f32x4*)&sh_o[w][rl][ch];
    }
    const int j = r / p.group, hq = h * p.group + (r - j * p.group);
    if (p.splits == 1) {
      const float inv = 1.0f / L;
      const int64_t qrow = ((int64_t)b * p.nq + j) * p.hq + hq;
      acc *= inv;
      if (p.out_fp32) {
        *(f32x4*)((float*)p.out + qrow * kHeadDim + ch) = acc;
      } else {
        *(uint2*)((uint16_t*)p.out + qrow * kHeadDim + ch) =
            make_uint2(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]));
      }
      if (p.lse && ch == 0) p.lse[qrow] = (M + log2f(L)) * kLn2;
    } else {
      const int64_t prow = (((int64_t)b * p.hkv + h) * p.rows_pad + r) * p.splits + split;
      *(f32x4*)(p.part_o + prow * kHeadDim + ch) = acc;
      if (ch == 0) p.part_ml[prow] = make_float2(M, L);
    }
  }
}

}  // namespace

int fp32_rows_per_wg(int rows) { return rows <= 16 ? 16 : 32; }

hipError_t launch_attn_fp32(const AttnParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.splits * p.row_groups), (unsigned)p.hkv, (unsigned)p.batch);
  if (fp32_rows_per_wg(p.rows) == 16)
    hipLaunchKernelGGL(attn_fp32_kernel<1>, grid, dim3(64 * kWaves), 0, s, p);
  else
    hipLaunchKernelGGL(attn_fp32_kernel<2>, grid, dim3(64 * kWaves), 0, s, p);
  return hipGetLastError();
}

}  // namespace kvshot
