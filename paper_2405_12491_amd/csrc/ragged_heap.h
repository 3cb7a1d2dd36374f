// ragged_heap.h -- the lockstep walk of ragged trees over padded top-level heaps and two-level
// deep blocks (layout in internal.h: RAGGED heaps), templated per number of top levels.
//
// What bounds it: per (wave, tree) the walk issues its node steps on the VALU, and every
// wave-wide block load occupies the texture addresser for at least 16 clocks, about two more per
// cache line it touches.  The steps are therefore kept free of per-slot branches and lane masks:
//   * the first L levels are a complete heap (a leaf above level L is padded with nodes whose
//     two subtrees hold the same leaf), so a step is PERFECT's four instructions a level and no
//     lane can be done before the heap ends;
//   * a deep block holds a node and its two children (16 bytes, two levels a load).  Its
//     feature fields are byte offsets into the row tile in place (the tile starts at LDS 0 and
//     a feature's row spans 64 elements, so a mask and an or make the address; the fields of the
//     children come to the same place by one rotate).  A step of a lane that has reached its
//     leaf computes the same step again with the same result: only the loads are masked.
// Measured on 1000 trees up to depth 12, 4M x 256 rows: 89 VALU and 28 scalar instructions and
// 3.9 wave-wide loads (row tile and copies included) per (wave, tree), one VALU instruction per
// clock and CU, addresser 91% busy, 9.42 ms; the treelet walk it replaced took 114, 92 and 4.0 and
// 14.1 ms.  100 trees of depth 12 over 1M x 28 rows: 0.227 ms (0.362).
#pragma once
#include "perfect_walk.h"
#include "vector_leaves.h"

namespace bridger {

// Load part `part` of `parts` of this lane's row of bins (XB bytes each) into the feature-major
// tile of 16-bit bins (64 rows, feature rows of 128 bytes); 8-bit bins are widened.
template <int XB>
__device__ __forceinline__ void load_row_bins16(const LaunchArgs &a, uint32_t lane_off,
                                                int64_t row, bool row_ok, int part, int parts) {
  auto put = [&](int f, uint32_t v) {
    *(__attribute__((address_space(3))) uint16_t *)(uintptr_t)(lane_off + 128u * (uint32_t)f) =
        (uint16_t)v;
  };
  const int f0 = (a.F * part) / parts, f1 = (a.F * (part + 1)) / parts;
  if (!row_ok) {
    for (int f = f0; f < f1; ++f) put(f, 0u);
    return;
  }
  const uint8_t *xr = reinterpret_cast<const uint8_t *>(a.X) + row * (int64_t)a.F * XB;
  if (a.x_vec4) {
    constexpr int E = 16 / XB;  // bins per 16-byte load
    const uint4 *x4 = reinterpret_cast<const uint4 *>(xr);
    const int n4 = (a.F * XB) >> 4;
    const int i0 = (n4 * part) / parts, i1 = (n4 * (part + 1)) / parts;
    for (int i = i0; i < i1; ++i) {
      const uint4 v = x4[i];
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < E; ++e)
        put(i * E + e, (w[(e * XB) >> 2] >> (8 * ((e * XB) & 3))) & (XB == 2 ? 0xFFFFu : 0xFFu));
    }
  } else {
    for (int f = f0; f < f1; ++f)
      put(f, XB == 2 ? (uint32_t)reinterpret_cast<const uint16_t *>(xr)[f] : (uint32_t)xr[f]);
  }
}

// A lane group is R = 64 / GPW rows (heap_rows); a wave holds GPW groups (1, 2 or 4), the G waves of
// a workgroup share R rows, and the G * GPW groups walk contiguous ranges of the trees, U trees at a
// time.  With one group per wave (MULTI false) all lanes of a wave are on the same trees and the
// tree addresses are wave-uniform; small batches take more groups per wave instead, so that a
// group's chain of batches is shorter (each group then has its own copies of the heaps).  The tile
// has 64 columns whatever R: every lane has its own, a row in several of them, so the gathers meet
// no bank conflicts.
// XB: bytes of an element of X (4; 2 or 1: the tile then holds 16-bit bins).  FIN: fp32 with
// finite thresholds (bins: always).  VK: 0 scalar leaves; 4 or 8 (K <= VK) or 64 vector leaves,
// class sums in registers / LDS (a leaf's word is then its row of leaf_vec).  KS: scalar leaves
// of several classes: -1 class sums in LDS slots, else the sums of the (at most KS) classes that
// a group's trees span in registers until the walk is done; 0: one class.
// C: columns of the tile.  fp32 rows of more than kHeapWideFeatures features take 32, with groups of
// 32 or 16 rows: the halves of a wave then read the same columns.
template <int L, int U, bool LEAVES, int XB, bool FIN, int VK, int KS, bool MULTI, int C>
__global__ __launch_bounds__(1024) void ragged_heap_kernel(LaunchArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int XL = XB == 4 ? 4 : 2;              // bytes of an element of the tile
  constexpr uint32_t kShift = XL * C == 256 ? 8u : 7u;  // log2 of a feature's row of the tile
  static_assert(XL * C == 128 || XL * C == 256, "a feature's row is 128 or 256 bytes");
  static_assert(C == 64 || (C == 32 && XB == 4 && MULTI), "32 columns: fp32 rows, several groups");
  constexpr uint32_t kField = 1023u << kShift;     // a feature field in place: its row's offset
  constexpr uint32_t kLeaf = 1024u << kShift;      // a rotated child's leaf flag
  constexpr uint32_t TB = 8u << L;                 // bytes of one tree's heap
  constexpr bool VK_REG = VK == 4 || VK == 8;
  constexpr int VR = VK_REG ? VK : 4;
  static_assert((U * TB) % 1024 == 0, "a batch is whole 1 KB copies");
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int T = a.n_trees;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = MULTI ? a.heap_rows : 64, GPW = MULTI ? 64 / R : 1;
  const int GT = a.groups;                         // lane groups of the workgroup
  const int gi = MULTI ? lane / R : 0;             // this lane's group within the wave
  const int g = wave * GPW + gi;
  const int64_t row = (int64_t)blockIdx.x * R + (MULTI ? (lane & (R - 1)) : lane);
  const bool row_ok = row < a.n_rows;
  const uint32_t lane_off = tile_row_off<XL>(lane & (C - 1));
  const uint32_t wbuf = (uint32_t)a.lds_top_off + (uint32_t)(wave * GPW) * (U * TB);
  const uint32_t buf = wbuf + (uint32_t)gi * (U * TB);
  const int ga = (int)(((int64_t)T * g) / GT), gb = (int)(((int64_t)T * (g + 1)) / GT);
  const int NB = MULTI ? ((T + GT - 1) / GT + U - 1) / U : (gb - ga + U - 1) / U;  // batches

  // the heaps of batch j of the wave's groups into their buffers (U empty heaps follow the last)
  auto copy_tops = [&](int j) {
    for (int i = 0; i < GPW; ++i) {
      const int q = min((int)(((int64_t)T * (wave * GPW + i)) / GT) + j * U, T);
#pragma unroll
      for (uint32_t k = 0; k < U * TB / 1024; ++k)
        __builtin_amdgcn_global_load_lds(
            (const void *)(reinterpret_cast<const uint8_t *>(a.tops) + (size_t)q * TB + k * 1024 +
                           (size_t)lane * 16),
            (__attribute__((address_space(3))) void *)((lds_byte *)smem + wbuf +
                                                       (uint32_t)i * (U * TB) + k * 1024),
            16, 0, 0);
    }
  };
  const int waves = (int)(blockDim.x >> 6);
  // the tile's part of this lane: column col, part `part` of `parts` of its features
  const int col = lane & (C - 1);
  const int part = C == 32 ? 2 * wave + (lane >> 5) : wave, parts = C == 32 ? 2 * waves : waves;
  auto load_tile = [&](auto nan_tag) {
    constexpr bool NAN_TO_INF = decltype(nan_tag)::value;
    if constexpr (MULTI) load_tile_any<4, NAN_TO_INF>(smem, a, col, row, row_ok, part, parts);
    else load_tile_all<4, NAN_TO_INF>(smem, a, lane, row, row_ok, wave, waves);
  };
  if constexpr (XB != 4) {
    if (NB > 0) copy_tops(0);
    load_row_bins16<XB>(a, lane_off, row, row_ok, wave, waves);
  } else if (a.tile_norm) {
    // Normalizer: the rows as they are, each column's norm (one lane adds its squares in feature
    // order, as the row-norm pass does; a float's square is exact in double), then the division.
    // That pass, its scratch and their allocation cost a small batch 25 us.  The norms pass
    // through the first copy buffer.
    a.pre_kind = 0;
    load_tile(std::false_type{});
    __syncthreads();
    double *norm = reinterpret_cast<double *>(smem + a.lds_top_off) + col;
    if (wave == 0) {
      double s = 0.0;
#pragma unroll 8
      for (int f = 0; f < a.F; ++f) {
        const double x = (double)lds_f32(smem, (uint32_t)f * (4u * C) + lane_off);
        s = s + x * x;
      }
      *norm = s == 0.0 ? 1.0 : __builtin_sqrt(s);
    }
    __syncthreads();
    const double rn = *norm;
    __syncthreads();
    if (NB > 0) copy_tops(0);
    const int f1 = (a.F * (part + 1)) / parts;
    for (int f = (a.F * part) / parts; f < f1; ++f) {
      __attribute__((address_space(3))) float *x =
          (__attribute__((address_space(3))) float *)(uintptr_t)((uint32_t)f * (4u * C) + lane_off);
      const float v = (float)((double)*x / rn);
      *x = FIN && v != v ? __builtin_inff() : v;
    }
  } else {
    if (NB > 0) copy_tops(0);
    load_tile(std::integral_constant<bool, FIN>{});
  }
  __syncthreads();

  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.nodes, (short)0, (int)a.nodes_bytes, kBufferRsrcWord3);
  const bool flat = a.flat != 0;  // no tree is deeper than L: a leaf word per slot, no blocks

  double *acc_lds = reinterpret_cast<double *>(smem + a.lds_acc_off) + tid;
  const int slot_stride = (int)blockDim.x;
  int k0 = 0;  // KS > 0: the class of the group's first tree
  if (KS > 0)
    while (k0 + 1 < a.K && ga >= a.class_begin[k0 + 1]) ++k0;
  ClassAcc ca;
  ca.k = k0;
  ca.acc = LEAVES ? 0.0 : class_init(a, k0, g == 0);
  ca.next_b = KS != 0 ? a.class_begin[k0 + 1] : 0x7fffffff;
  double vacc[VR];
  if (VK_REG) vec_init_reg(a, vacc, g == 0);
  if (VK == 64) vec_init(a, acc_lds, slot_stride, g == 0);
  double cs[KS > 0 ? KS : 1];
#pragma unroll
  for (int j = 0; j < (KS > 0 ? KS : 1); ++j) cs[j] = 0.0;
  auto advance_reg = [&](int t) {  // as in perfect_global_kernel: finished sums shift through cs
    while (t >= ca.next_b) {
#pragma unroll
      for (int j = KS - 1; j > 0; --j) cs[j] = cs[j - 1];
      cs[0] = ca.acc;
      ca.k += 1;
      ca.acc = class_init(a, ca.k, g == 0);
      ca.next_b = a.class_begin[ca.k + 1];
    }
  };

  for (int j = 0; j < NB; ++j) {
    const int q = ga + j * U;
    const int nvalid = gb - q < U ? gb - q : U;  // (MULTI: per lane, and 0 or less past its trees)
    wait_stage();  // this batch's heaps have landed
    uint32_t m[U], base[U], res[U], oi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t first = lds_u64(smem, buf + u * TB).x;
      base[u] = MULTI ? first : (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
      m[u] = 1u;
    }
#pragma unroll
    for (int d = 0; d < L; ++d) {
      uint2 rec[U];
      uint32_t xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) rec[u] = lds_u64(smem, (m[u] << 3) + buf + u * TB);
#pragma unroll
      for (int u = 0; u < U; ++u) xv[u] = gather_x<FIN, XL>(smem, rec[u].y | lane_off);
#pragma unroll
      for (int u = 0; u < U; ++u) m[u] = step_slot<FIN, XL>(m[u], rec[u].x, xv[u]);
    }
    // the heaps are read: the next batch's can land while the deep blocks are walked
    if (j + 1 < NB) copy_tops(j + 1);
    if (flat) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t s = base[u] + m[u] - (1u << L);
        res[u] = LEAVES ? 0u : __builtin_amdgcn_raw_buffer_load_b32(rsrc, s * 4u, 0, 0);
        oi[u] = s;
      }
    } else {
      u32x4 blk[U];
      bool live[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        live[u] = true;
        blk[u] = u32x4{0u, 0u, 0u, 0u};
        res[u] = oi[u] = 0u;
      }
      // slot m of block level lv (2^L 4^lv <= m < 2^(L+1) 4^lv) is block base + m + off
      uint32_t off = 0u - (1u << L), width = 1u << L;
      for (int lv = 0; lv < 32; ++lv) {  // trees are at most 64 levels deep
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (live[u])
            blk[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (m[u] + (base[u] + off)) * 16u, 0, 0);
        uint32_t x1[U], x2[U], m2[U], wc[U], b1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x1[u] = gather_x<FIN, XL>(smem, (blk[u].w & kField) | lane_off);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool r = XB == 4 ? !(__uint_as_float(x1[u]) <= __uint_as_float(blk[u].x))
                                 : x1[u] > blk[u].x;
          wc[u] = r ? blk[u].z : blk[u].y;
          m2[u] = __builtin_amdgcn_alignbit(blk[u].w, blk[u].w, r ? 21u : 10u);
          b1[u] = r ? 1u : 0u;
          x2[u] = gather_x<FIN, XL>(smem, (m2[u] & kField) | lane_off);
        }
        bool any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool r = XB == 4 ? !(__uint_as_float(x2[u]) <= __uint_as_float(wc[u]))
                                 : x2[u] > wc[u];
          if (LEAVES) oi[u] = live[u] ? 2u * (m[u] + (base[u] + off)) + b1[u] : oi[u];
          res[u] = wc[u];
          live[u] = (m2[u] & kLeaf) == 0u;
          m[u] = 4u * m[u] + 2u * b1[u] + (r ? 1u : 0u);
          any = any || live[u];
        }
        if (!__any(any)) break;
        off -= 2u * width;
        width *= 4u;
      }
    }
    // trees q .. q + nvalid - 1 in order
    if (LEAVES) {
      if (row_ok) {
        int32_t id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) id[u] = a.leaf_map[oi[u]];
        if (nvalid == U) {
          store_leaf_ids(a, row, q, id);
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int32_t id1[1] = {id[u]};
            if (u < nvalid) store_leaf_ids(a, row, q + u, id1);
          }
        }
      }
    } else if (VK != 0) {
      // 5..8 classes: one tree's row at a time (four in flight took 86 registers and 3% longer for
      // 300k x 28 rows, 100 trees, 7 classes, which take 130 us)
      constexpr int VN = VK == 8 ? 1 : U;
      if (nvalid == U) {
#pragma unroll
        for (int v = 0; v < U; v += VN) {
          int64_t leaf[VN];
#pragma unroll
          for (int u = 0; u < VN; ++u) leaf[u] = res[v + u];
          if (VK_REG) vec_add_reg(a, vacc, leaf);
          else vec_add(a, acc_lds, slot_stride, leaf);
          if (VN < U) __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (u < nvalid) {
            const int64_t leaf[1] = {res[u]};
            if (VK_REG) vec_add_reg(a, vacc, leaf);
            else vec_add(a, acc_lds, slot_stride, leaf);
          }
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u < nvalid) {
          if (KS > 0) advance_reg(q + u);
          else if (KS < 0) class_advance(a, ca, q + u, acc_lds, slot_stride, g == 0);
          ca.acc += (double)__uint_as_float(res[u]);
        }
      }
    }
  }
  if (LEAVES) return;
  // Class sums: one class, or sums in registers, go over the tile and the copies (every wave is
  // done with them after the barrier; no copy is in flight after the last batch).
  wait_stage();
  if (VK == 0 && KS >= 0) __syncthreads();
  if (VK_REG) __syncthreads();
  if constexpr (VK_REG) {
    vec_store_reg(a, vacc, acc_lds, slot_stride);
  } else if constexpr (VK == 0 && KS < 0) {
    class_flush_all(a, ca, acc_lds, slot_stride, g == 0);
  } else if constexpr (VK == 0 && KS > 0) {
    for (int c = 0; c < a.K; ++c) {
      const int d = ca.k - c;  // class c's sum: ca.acc (d = 0) or cs[d - 1] (k0 <= c < ca.k)
      double v = d == 0 ? ca.acc : class_init(a, c, g == 0);
#pragma unroll
      for (int j = 0; j < KS; ++j)
        if (c >= k0 && d == j + 1) v = cs[j];
      acc_lds[c * slot_stride] = v;
    }
  } else if constexpr (VK == 0) {
    acc_lds[0] = ca.acc;
  }
  __syncthreads();
  groups_finalize_store(a, reinterpret_cast<double *>(smem + a.lds_acc_off), R, GT, slot_stride,
                        tid, row, row_ok);
}

// ---------------------------------------------------------------------- launchers
template <int L, int U, int XB, bool FIN, bool MULTI, int C>
static int launch_heap_luxfm(const LaunchArgs &a, int threads, int64_t n_wg, int lds_bytes,
                            void *stream) {
#define BRIDGER_HEAP(LEAVES, VK, KS) \
  launch_common(ragged_heap_kernel<L, U, LEAVES, XB, FIN, VK, KS, MULTI, C>, threads, n_wg, lds_bytes, stream, a)
  if (a.out_leaf) return BRIDGER_HEAP(true, 0, 0);
  if (a.vec && a.K <= 4) return BRIDGER_HEAP(false, 4, 0);
  if (a.vec && a.K <= 8) return BRIDGER_HEAP(false, 8, 0);
  if (a.vec) return BRIDGER_HEAP(false, 64, 0);
  if (a.K == 1) return BRIDGER_HEAP(false, 0, 0);
  if (a.acc_alias) return BRIDGER_HEAP(false, 0, kHeapClassRegs);
  return BRIDGER_HEAP(false, 0, -1);
#undef BRIDGER_HEAP
}

template <int L, int U, int XB, bool FIN>
static int launch_heap_luxf(const LaunchArgs &a, int threads, int64_t n_wg, int lds_bytes,
                            void *stream) {
  if constexpr (XB == 4)
    if (a.rows_per_wg == 32)
      return launch_heap_luxfm<L, U, XB, FIN, true, 32>(a, threads, n_wg, lds_bytes, stream);
  return a.heap_rows < 64 ? launch_heap_luxfm<L, U, XB, FIN, true, 64>(a, threads, n_wg, lds_bytes, stream)
                          : launch_heap_luxfm<L, U, XB, FIN, false, 64>(a, threads, n_wg, lds_bytes, stream);
}

template <int L, int U>
static int launch_heap_lu(const LaunchArgs &a, int waves, int64_t n_wg, int lds_bytes,
                          void *stream) {
  const int threads = 64 * waves;
  if (a.x_bytes == 2) return launch_heap_luxf<L, U, 2, true>(a, threads, n_wg, lds_bytes, stream);
  if (a.x_bytes == 1) return launch_heap_luxf<L, U, 1, true>(a, threads, n_wg, lds_bytes, stream);
  return a.finite_thresholds ? launch_heap_luxf<L, U, 4, true>(a, threads, n_wg, lds_bytes, stream)
                             : launch_heap_luxf<L, U, 4, false>(a, threads, n_wg, lds_bytes, stream);
}

}  // namespace bridger
