// direct.hip -- gfx950 kernels for trees of any size, read from global memory: the tile kernel
// (pair records, features from an LDS tile) and the fallback (features from global memory too).
#include "perfect_walk.h"
#include "vector_leaves.h"

namespace bridger {

// ======================================================================== DIRECT
// Fallback for any forest: one row per lane, nodes and features read from global memory.
// VK: 0 scalar leaves; 4 or 8 (K <= VK) or 64 vector leaves (class sums in registers / LDS).
// PAIR: pair records (layout in internal.h), else the 16-byte ones.
template <bool LEAVES, int VK = 0, bool PAIR = false>
__global__ __launch_bounds__(256) void direct_kernel(LaunchArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr bool VK_REG = VK == 4 || VK == 8;  // vector leaves, class sums in registers
  constexpr int VR = VK_REG ? VK : 4;
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool row_ok = row < a.n_rows;
  const int64_t rr = row_ok ? row : 0;
  const float *xr = a.X + rr * (int64_t)a.F;
  const int T = a.n_trees;
  double *acc_lds = reinterpret_cast<double *>(smem) + threadIdx.x;
  const int slot_stride = blockDim.x;
  ClassAcc ca;
  ca.k = 0;
  ca.acc = class_init(a, 0, true);
  ca.next_b = a.class_begin[1];
  double vacc[VR];
  if (VK_REG) vec_init_reg(a, vacc, true);
  if (VK == 64) vec_init(a, acc_lds, slot_stride, true);
  auto feature = [&](int f) { return a.pre_kind ? preprocess(a, f, rr, xr[f]) : xr[f]; };
  for (int t = 0; t < T; ++t) {
    int64_t n = a.tree_start[t];  // record of the leaf
    uint32_t word;                // its value, or (PAIR, vector leaves) its row of class values
    if constexpr (PAIR) {
      const uint2 *recs = reinterpret_cast<const uint2 *>(a.nodes) + n;
      uint32_t i = 0;
      uint2 rc = recs[0];
      while (!(rc.y & kPairLeaf)) {
        i += (rc.y >> kPairRelShift) + (feature((int)(rc.y & 1023u)) <= __uint_as_float(rc.x) ? 0u : 1u);
        rc = recs[i];
      }
      n += i;
      word = rc.x;
    } else {
      const int4 *recs = reinterpret_cast<const int4 *>(a.nodes);
      int4 rc = recs[n];
      while (rc.y >= 0) {
        n = (feature(rc.y) <= __int_as_float(rc.x)) ? rc.z : rc.w;
        rc = recs[n];
      }
      word = (uint32_t)rc.x;
    }
    if (LEAVES) {
      if (row_ok) a.out_leaf[row * (int64_t)T + a.tree_order[t]] = a.leaf_map[n];
    } else if (VK) {
      const int64_t leaf[1] = {PAIR ? (int64_t)word : n};
      if (VK_REG) vec_add_reg(a, vacc, leaf);
      else vec_add(a, acc_lds, slot_stride, leaf);
    } else {
      class_advance(a, ca, t, acc_lds, slot_stride, true);
      ca.acc += (double)__uint_as_float(word);
    }
  }
  if (LEAVES) return;
  if (VK_REG) {
    vec_store_reg(a, vacc, acc_lds, slot_stride);
  } else if (!VK) {
    class_flush_all(a, ca, acc_lds, slot_stride, true);
  }
  if (row_ok) finalize_store(a, reinterpret_cast<double *>(smem) + threadIdx.x, slot_stride, row);
}

// =================================================================== DIRECT tile
// Trees too large for the RAGGED layouts (fully grown ones: tens of thousands of nodes, 20 and
// more levels).  A walk is a chain of dependent loads, most of them past L2's 4 MB, so what counts
// is how many are in flight and how many lines they touch:
//   * G waves share a 64-row tile (one lane group each) and split every batch of G * U trees, U a
//     wave at a time, all lanes of a wave on the same U trees;
//   * 8-byte pair records (layout in internal.h), two sibling records adjacent, the last levels of
//     a tree gathered by subtrees of at most 32 records, so they cost a lane one or two lines.
// The sums stay those of one lane adding its trees in ascending order: the waves leave their
// leaves in LDS and after the batch's barrier one wave adds the batch to the class sums, tree by
// tree (vector leaves: one wave per four classes), while the others walk the next batch.
// 64 trees grown on 20,000 rows, 51,630 x 90 rows: 655 us with one row and one tree per lane (three
// waves a CU, 16-byte records, features from global memory); this kernel: 156 us.
template <bool LEAVES, bool VEC>
__global__ __launch_bounds__(1024) void direct_tile_kernel(LaunchArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int U = kDirectBatch;
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.groups, T = a.n_trees, K = a.K;
  const int64_t row = (int64_t)blockIdx.x * 64 + lane;
  const bool row_ok = row < a.n_rows;
  const uint32_t lane_off = 4u * (uint32_t)lane;
  double *acc = reinterpret_cast<double *>(smem + a.lds_acc_off) + lane;  // class k at 64 k
  uint32_t *vals = reinterpret_cast<uint32_t *>(smem + a.lds_top_off) + lane;

  load_tile_all<4, false>(smem, a, lane, row, row_ok, g, G);
  if (!LEAVES)
    for (int k = g; k < K; k += G) acc[64 * k] = class_init(a, k, true);
  __syncthreads();

  const int per = G * U, batches = (T + per - 1) / per;
  for (int b = 0; b < batches; ++b) {
    const int q = b * per + g * U;
    uint32_t *out = vals + (size_t)(b & 1) * per * 64;
    if (q < T) {
      const uint2 *recs[U];
      uint2 rec[U];
      uint32_t idx[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // slots past the last tree walk it again
        const int t = q + u < T ? q + u : T - 1;
        recs[u] = reinterpret_cast<const uint2 *>(a.nodes) + (uint32_t)a.tree_start[t];
        idx[u] = 0u;
        rec[u] = recs[u][0];
      }
      for (int level = 0; level <= 64; ++level) {  // validated trees are at most 64 deep
        uint32_t xv[U];
        bool any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          xv[u] = gather_x<false, 4>(smem, ((rec[u].y & 1023u) << 8) | lane_off);
          any = any || !(rec[u].y & kPairLeaf);
        }
        if (!__any(any)) break;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!(rec[u].y & kPairLeaf)) {
            const bool right = !(__uint_as_float(xv[u]) <= __uint_as_float(rec[u].x));
            idx[u] += (rec[u].y >> kPairRelShift) + (right ? 1u : 0u);
            rec[u] = recs[u][idx[u]];
          }
        }
      }
      if (LEAVES) {
        int32_t id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int t = q + u < T ? q + u : T - 1;
          id[u] = a.leaf_map[(uint32_t)a.tree_start[t] + idx[u]];
        }
        if (row_ok && q + U <= T) {
          store_leaf_ids(a, row, q, id);
        } else if (row_ok) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int32_t id1[1] = {id[u]};
            if (q + u < T) store_leaf_ids(a, row, q + u, id1);
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) out[(g * U + u) * 64] = rec[u].x;
      }
    }
    if (LEAVES) continue;
    __syncthreads();  // the batch's leaves are in LDS; the previous batch is added
    const int n = T - b * per < per ? T - b * per : per;
    if (VEC) {
      const int groups = vec_stride(K) >> 2;
      const float4 *rows = reinterpret_cast<const float4 *>(a.leaf_vec);
      for (int kg = g; kg < groups; kg += G) {
        double s[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = 4 * kg + c < K ? acc[64 * (4 * kg + c)] : 0.0;
#pragma unroll 4
        for (int i = 0; i < n; ++i) {
          const float4 w = rows[(size_t)out[i * 64] * groups + kg];
          s[0] += (double)w.x;
          s[1] += (double)w.y;
          s[2] += (double)w.z;
          s[3] += (double)w.w;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (4 * kg + c < K) acc[64 * (4 * kg + c)] = s[c];
      }
    } else if (g == b % G) {  // the classes' trees are contiguous
      int k = 0, i = 0;
      while (i < n) {
        while (b * per + i >= a.class_begin[k + 1]) ++k;
        const int end = a.class_begin[k + 1] - b * per < n ? a.class_begin[k + 1] - b * per : n;
        double s = acc[64 * k];
#pragma unroll 4
        for (; i < end; ++i) s += (double)__uint_as_float(out[i * 64]);
        acc[64 * k] = s;
      }
    }
  }
  if (LEAVES) return;
  __syncthreads();
  if (g == 0 && row_ok) finalize_store(a, acc, 64, row);
}

// ---------------------------------------------------------------------- launchers
int launch_direct_tile(const LaunchArgs &a, int waves, int64_t n_wg, int lds_bytes, void *stream) {
  const int threads = 64 * waves;
  if (a.out_leaf)
    return launch_common(direct_tile_kernel<true, false>, threads, n_wg, lds_bytes, stream, a);
  if (a.vec)
    return launch_common(direct_tile_kernel<false, true>, threads, n_wg, lds_bytes, stream, a);
  return launch_common(direct_tile_kernel<false, false>, threads, n_wg, lds_bytes, stream, a);
}

template <bool PAIR>
static int launch_direct_p(const LaunchArgs &a, int64_t n_wg, void *stream) {
  const int lds = a.out_leaf ? 0 : 256 * 8 * a.K;
  if (a.out_leaf) return launch_common(direct_kernel<true, 0, PAIR>, 256, n_wg, lds, stream, a);
  if (a.vec && a.K <= 4)
    return launch_common(direct_kernel<false, 4, PAIR>, 256, n_wg, lds, stream, a);
  if (a.vec && a.K <= 8)
    return launch_common(direct_kernel<false, 8, PAIR>, 256, n_wg, lds, stream, a);
  if (a.vec) return launch_common(direct_kernel<false, 64, PAIR>, 256, n_wg, lds, stream, a);
  return launch_common(direct_kernel<false, 0, PAIR>, 256, n_wg, lds, stream, a);
}

int launch_direct(const LaunchArgs &a, bool pairs, int64_t n_wg, void *stream) {
  return pairs ? launch_direct_p<true>(a, n_wg, stream) : launch_direct_p<false>(a, n_wg, stream);
}

}  // namespace bridger
