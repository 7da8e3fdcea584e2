// Tree attention on the vector ALUs, the fp32 path: one workgroup of four
// waves per (sequence, node, kv head) handles the G query heads of that kv
// head, four at a time (one a wave).  Keys are visited in tiles of 64, each
// tile's K and V rows staged in LDS by the whole workgroup with coalesced
// 16-byte loads, so the G heads (and, per pass, the four waves) share one
// read of them.  Scores take one key per lane (a dot product over an LDS row
// padded against bank conflicts); an online (running-max) softmax per head;
// the value accumulation takes one or two head dimensions per lane.
//
// The head size is a template parameter: piece and row indexes are then shifts,
// the score's LDS reads unroll, and 16 keys' value reads are in flight (8 heads
// of 64 dims, prefix 128, 16 nodes: 11.1 us a call with run-time divisions and
// one 4-key group of reads at a time, 7.8 now).
//
// The visible key set of node i is the prefix [0, P_b) plus the tree rows of
// the node's root path (arXiv 2603.01639, section 3.2: the tree attention
// mask shows each candidate its ancestors only).
#include "ltd_device.hpp"
#include "ltd_launch.hpp"
#include "tree_walk.hpp"

namespace ltd {
namespace {

constexpr int kTileKeys = 64;
constexpr int kVecWaves = 4;
constexpr int kVecThreads = kVecWaves * kWave;

// Four consecutive elements of a cache row as floats (16-byte loads when the
// row data is float and 16-byte aligned).
template <typename T, bool kVec>
__device__ __forceinline__ void load4(const T* p, int64_t i, float (&x)[4]) {
  if constexpr (kVec) {
    const float4 v = *reinterpret_cast<const float4*>(p + i);
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = load_f32(p, i + e);
  }
}

template <typename T, bool kVec, int HD>
__global__ void __launch_bounds__(kVecThreads) attn_vector_kernel(
    const T* __restrict__ q, const T* __restrict__ k_cache, const T* __restrict__ v_cache,
    const int32_t* __restrict__ block_table, const int32_t* __restrict__ prefix_len,
    const int32_t* __restrict__ parents, const int32_t* __restrict__ n_nodes, T* __restrict__ out,
    int Nmax, int Hq, int Hkv, int kv_rows, int max_blocks, float scale, const int32_t* status) {
  constexpr int d = HD;
  constexpr int kPieces = kTileKeys * HD / 4 / kVecThreads;  // 16-byte pieces a thread loads
  // K transposed by groups of 4 dims (lane = key reads 16 consecutive bytes,
  // consecutive lanes consecutive 16-byte words); V by rows (lanes = dims)
  __shared__ float4 kt_s[HD / 4][kTileKeys];
  __shared__ __attribute__((aligned(16))) float v_s[kTileKeys * HD];
  __shared__ float4 q_s[kVecWaves][HD / 4];
  __shared__ __attribute__((aligned(16))) float p_s[kVecWaves][kTileKeys];
  __shared__ int path_s[LTD_MAX_NODES];
  __shared__ int path_len_s;

  const int i = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  if (halted(status)) return;
  if (i >= n_nodes[b]) return;  // uniform for the workgroup
  const int G = Hq / Hkv;
  const int P = prefix_len[b];
  const int32_t* par = parents + static_cast<int64_t>(b) * Nmax;
  if (t == 0) path_len_s = root_path(par, i, path_s);  // tree rows node i may see
  __syncthreads();
  const int n_keys = P + path_len_s;
  const int n_tiles = (n_keys + kTileKeys - 1) / kTileKeys;
  constexpr int dq = HD / 4;  // 16-byte pieces of a row

  for (int h0 = 0; h0 < G; h0 += kVecWaves) {
    const int h = h0 + w;             // this wave's head within the group
    const bool head = h < G;
    const int64_t q_off = ((static_cast<int64_t>(b) * Nmax + i) * Hq + g * G + (head ? h : 0)) * d;
    for (int e = lane; e < d; e += kWave)
      reinterpret_cast<float*>(q_s[w])[e] = head ? load_f32(q, q_off + e) * scale : 0.f;
    float m = -INFINITY, l = 0.f;
    float acc0 = 0.f, acc1 = 0.f;  // head dims lane and lane + 64
    // Tile loads go through registers one tile ahead: thread t holds the
    // 16-byte pieces x = t + 256 j of the tile's rows (piece x: row x / dq,
    // dims 4 (x % dq) .. + 3), so the next tile's loads are in flight while
    // the current one is computed.
    float kr4[kPieces][4], vr4[kPieces][4];
    auto fetch = [&](int tile) {
      const int base = tile * kTileKeys;
      const int cnt = min(kTileKeys, n_keys - base);
#pragma unroll
      for (int j = 0; j < kPieces; ++j) {
        const int x = t + j * kVecThreads;
        const int r = x / dq, c = (x % dq) * 4;
        if (r < cnt) {
          const int kt = base + r;
          const int row = kt < P ? kt : P + path_s[kt - P];
          const int64_t off = cache_row(block_table, b, g, row, Hkv, d, kv_rows, max_blocks) + c;
          load4<T, kVec>(k_cache, off, kr4[j]);
          load4<T, kVec>(v_cache, off, vr4[j]);
        }
      }
    };
    if (n_tiles > 0) fetch(0);
    for (int tile = 0; tile < n_tiles; ++tile) {
      const int base = tile * kTileKeys;
      const int cnt = min(kTileKeys, n_keys - base);
      __syncthreads();  // every wave is done with the previous tile (and q_s is written)
      // (rows past the tile's keys are zero: their weights are zero too, and
      // stale LDS could hold NaN)
#pragma unroll
      for (int j = 0; j < kPieces; ++j) {
        const int x = t + j * kVecThreads;
        const int r = x / dq, c = (x % dq) * 4;
        if (r < kTileKeys) {
          const bool in = r < cnt;
          kt_s[c / 4][r] = in ? make_float4(kr4[j][0], kr4[j][1], kr4[j][2], kr4[j][3])
                              : make_float4(0.f, 0.f, 0.f, 0.f);
          *reinterpret_cast<float4*>(v_s + r * HD + c) =
              in ? make_float4(vr4[j][0], vr4[j][1], vr4[j][2], vr4[j][3])
                 : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
      if (tile + 1 < n_tiles) fetch(tile + 1);
      __syncthreads();
      if (!head) continue;
      // score of key `lane`: four independent partial sums over groups of 4 dims
      float s = -INFINITY;
      {
        float d4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int eg = 0; eg < dq; eg += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float4 kv = kt_s[eg + u][lane];
            const float4 qv = q_s[w][eg + u];
            d4[u] += qv.x * kv.x + qv.y * kv.y + qv.z * kv.z + qv.w * kv.w;
          }
        }
        if (lane < cnt) s = (d4[0] + d4[1]) + (d4[2] + d4[3]);
      }
      const float m_new = fmaxf(m, wave_max_dpp(s));
      const float p = lane < cnt ? expf(s - m_new) : 0.f;
      const float alpha = expf(m - m_new);
      l = l * alpha + wave_sum_dpp(p);
      acc0 *= alpha;
      acc1 *= alpha;
      m = m_new;
      p_s[w][lane] = p;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // (weights past cnt are 0, and so are those rows of V; 16 keys' reads are
      // in flight at a time)
      float a0[4] = {0.f, 0.f, 0.f, 0.f}, a1[4] = {0.f, 0.f, 0.f, 0.f};
      const int cnt16 = (cnt + 15) & ~15;
#pragma unroll 4
      for (int u = 0; u < cnt16; u += 4) {
        const float4 p4 = *reinterpret_cast<const float4*>(&p_s[w][u]);
        const float pu[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          a0[k] += pu[k] * v_s[(u + k) * HD + lane];
          if (d > kWave) a1[k] += pu[k] * v_s[(u + k) * HD + lane + kWave];
        }
      }
      acc0 += (a0[0] + a0[1]) + (a0[2] + a0[3]);
      acc1 += (a1[0] + a1[1]) + (a1[2] + a1[3]);
    }
    if (head) {
      const float inv = 1.f / l;
      if (lane < d) store_f32(out, q_off + lane, acc0 * inv);
      if (lane + kWave < d) store_f32(out, q_off + lane + kWave, acc1 * inv);
    }
    __syncthreads();  // q_s and the tiles are reused by the next head group
  }
}

}  // namespace

hipError_t launch_attn_rowwise(const AttnShape& s, const void* q, const void* k_cache,
                               const void* v_cache, const int32_t* block_table,
                               const int32_t* prefix_len, const int32_t* parents,
                               const int32_t* n_nodes, void* out, float scale,
                               const int32_t* status, hipStream_t stream) {
  const dim3 grid(s.Nmax, s.Hkv, s.B);
  const auto launch = [&](auto kern, auto elem) {
    using T = decltype(elem);
    hipLaunchKernelGGL(kern, grid, dim3(kVecThreads), 0, stream, static_cast<const T*>(q),
                       static_cast<const T*>(k_cache), static_cast<const T*>(v_cache), block_table,
                       prefix_len, parents, n_nodes, static_cast<T*>(out), s.Nmax, s.Hq, s.Hkv,
                       s.kv_rows, s.max_blocks, scale, status);
  };
  if (s.dtype == LTD_DTYPE_F32) {
    // 16-byte loads when both caches are 16-byte aligned (every row and piece
    // offset is a multiple of 4 elements)
    const bool vec = (reinterpret_cast<uintptr_t>(k_cache) % 16) == 0 &&
                     (reinterpret_cast<uintptr_t>(v_cache) % 16) == 0;
    if (s.d == 64)
      launch(vec ? attn_vector_kernel<float, true, 64> : attn_vector_kernel<float, false, 64>, float{});
    else
      launch(vec ? attn_vector_kernel<float, true, 128> : attn_vector_kernel<float, false, 128>, float{});
  } else {
    launch(s.d == 64 ? attn_vector_kernel<uint16_t, false, 64> : attn_vector_kernel<uint16_t, false, 128>,
           uint16_t{});
  }
  return hipGetLastError();
}

}  // namespace ltd
