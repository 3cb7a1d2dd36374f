// bin.hip -- exact feature quantization ("data type rewriting", Table 2): each fp32 feature
// value becomes its bin, the number of the forest's distinct thresholds on that feature that
// are strictly below it.  For a threshold t of rank k among them, x <= t iff bin(x) <= k
// (-0.0 and +0.0 are one threshold; a NaN feature gets the table's size, above every rank,
// so it goes right at every split as the fp32 compare sends it).
//
// A value is looked up in two steps (layout in internal.h: bin tables): a uniform grid over the
// feature's thresholds, one cell per threshold (or per 2 to 16), gives the number of thresholds in lower cells, and
// a search over power-of-two steps counts those of its own cell, as many steps as the fullest cell
// of the run of features needs (3 or 4 where thresholds are drawn from the data, against 10 to 12
// for the whole table).  A cell is the truncated product fl(fl(x - lo) * scale), which never
// decreases with x, so thresholds in lower cells are below x and those in higher ones are not.
//
// What bounds it: the LDS gathers and the instructions around them, no longer the chain of a
// whole binary search.  A thread keeps one column, four features where rows and bins are
// aligned for it, so the features' parameters stay in registers, the loads and stores of a
// wave are consecutive, and no index is divided.
// Measured against the binary search over whole tables (32-feature groups, one element a lane):
// 1M x 28 rows, 910 thresholds a feature, 121 -> 40 us, 4,553 265 -> 180, 12,000 (a column a thread) 735 ->
// 280; 100k x 784, 66 (8-bit bins): 343 -> 146 us; 4M x 256, 2,750 (32 runs of 8 features, whose partial
// lines are what is left): 8.6 -> 4.1 ms.
#include "kernel_common.h"

namespace bridger {

constexpr int kBinThreads = 1024;

// LDS: the run's part of the image is staged and searched there; else it is searched in place.
template <int XB, int V, bool LDS>
__global__ __launch_bounds__(kBinThreads) void bin_kernel(LaunchArgs a, BinTables bt,
                                                          int64_t rows_per_block) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  constexpr int kIlp = V == 4 ? 2 : 4;  // rows in flight per thread
  const int tid = threadIdx.x;
  const BinRun run = bt.runs[blockIdx.x % (uint32_t)bt.n_runs];
  const int64_t r0 = (int64_t)(blockIdx.x / (uint32_t)bt.n_runs) * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < a.n_rows ? r0 + rows_per_block : a.n_rows;
  const bool staged = LDS && run.staged;
  if (staged) {
    const uint4 *src = reinterpret_cast<const uint4 *>(bt.image + run.word0);
    for (int i = tid; i < (run.words >> 2); i += kBinThreads) {
      const uint4 v = src[i];
      *(__attribute__((address_space(3))) uint64_t *)(uintptr_t)(16 * i) = v.x | (uint64_t)v.y << 32;
      *(__attribute__((address_space(3))) uint64_t *)(uintptr_t)(16 * i + 8) = v.z | (uint64_t)v.w << 32;
    }
    __syncthreads();
  }
  const int units = (run.f1 - run.f0 + V - 1) / V;   // columns of the run
  const int rpi = (int)blockDim.x / units;           // rows per pass of the workgroup
  const int rr = tid / units, f = run.f0 + (tid - rr * units) * V;
  if (rr >= rpi) return;
  float lo[V], scale[V], top[V];
  uint32_t start[V], tab[V];  // byte offsets into the run's image
  int n[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const BinFeature p = bt.features[f + v];
    lo[v] = p.lo;
    scale[v] = p.scale;
    top[v] = p.top;
    n[v] = p.n;
    start[v] = 2u * (uint32_t)(p.start - 2 * run.word0);
    tab[v] = 4u * (uint32_t)(p.tab - run.word0);
  }
  const int steps = __builtin_amdgcn_readfirstlane(run.steps);
  const uint8_t *img = reinterpret_cast<const uint8_t *>(bt.image + run.word0);

  auto rows = [&](auto lds_tag) {
    constexpr bool IN_LDS = decltype(lds_tag)::value;
    auto below = [&](uint32_t at, float x) {  // the table's element at byte `at`
      return (IN_LDS ? lds_f32(smem, at) : *reinterpret_cast<const float *>(img + at)) < x;
    };
    for (int64_t row = r0 + rr; row < r1; row += (int64_t)rpi * kIlp) {
      float x[kIlp][V];
#pragma unroll
      for (int i = 0; i < kIlp; ++i) {
        const int64_t r = row + (int64_t)i * rpi;
        const float *p = a.X + (r < r1 ? r : row) * (int64_t)a.F + f;
        if constexpr (V == 4) {
          const float4 q = *reinterpret_cast<const float4 *>(p);
          x[i][0] = q.x;
          x[i][1] = q.y;
          x[i][2] = q.z;
          x[i][3] = q.w;
        } else {
          x[i][0] = *p;
        }
      }
      if (a.pre_kind) {
#pragma unroll
        for (int i = 0; i < kIlp; ++i) {
          const int64_t r = row + (int64_t)i * rpi;
#pragma unroll
          for (int v = 0; v < V; ++v) x[i][v] = preprocess(a, f + v, r < r1 ? r : row, x[i][v]);
        }
      }
      uint32_t at[kIlp][V];  // byte offset of the element the count stands at
#pragma unroll
      for (int i = 0; i < kIlp; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float c = fminf(fmaxf((x[i][v] - lo[v]) * scale[v], 0.0f), top[v]);
          const uint32_t s = start[v] + 2u * (uint32_t)c;
          at[i][v] = tab[v] + 4u * (IN_LDS ? lds_u16(smem, s)
                                           : (uint32_t)*reinterpret_cast<const uint16_t *>(img + s));
        }
      // an element past the cell is not below x, and +inf elements follow the table: 8 of them
      // for the last steps, one that the larger steps are clamped to
      for (int st = steps; st >= 16; st >>= 1) {
#pragma unroll
        for (int i = 0; i < kIlp; ++i)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const uint32_t e = min(at[i][v] + 4u * (uint32_t)(st - 1), tab[v] + 4u * (uint32_t)n[v]);
            at[i][v] += below(e, x[i][v]) ? 4u * (uint32_t)st : 0u;
          }
      }
      auto step = [&](auto st_tag) {
        constexpr uint32_t ST = decltype(st_tag)::value;
#pragma unroll
        for (int i = 0; i < kIlp; ++i)
#pragma unroll
          for (int v = 0; v < V; ++v)
            at[i][v] += below(at[i][v] + 4u * (ST - 1), x[i][v]) ? 4u * ST : 0u;
      };
      if (steps >= 8) step(std::integral_constant<uint32_t, 8>{});
      if (steps >= 4) step(std::integral_constant<uint32_t, 4>{});
      if (steps >= 2) step(std::integral_constant<uint32_t, 2>{});
      if (steps >= 1) step(std::integral_constant<uint32_t, 1>{});
#pragma unroll
      for (int i = 0; i < kIlp; ++i) {
        const int64_t r = row + (int64_t)i * rpi;
        if (r >= r1) break;
        uint32_t b[V];
#pragma unroll
        for (int v = 0; v < V; ++v)
          b[v] = x[i][v] == x[i][v] ? (at[i][v] - tab[v]) >> 2 : (uint32_t)n[v];
        uint8_t *q = reinterpret_cast<uint8_t *>(a.xq) + (r * (int64_t)a.F + f) * XB;
        if constexpr (V == 4 && XB == 2)
          *reinterpret_cast<uint2 *>(q) = make_uint2(b[0] | b[1] << 16, b[2] | b[3] << 16);
        else if constexpr (V == 4)
          *reinterpret_cast<uint32_t *>(q) = b[0] | b[1] << 8 | b[2] << 16 | b[3] << 24;
        else if constexpr (XB == 2)
          *reinterpret_cast<uint16_t *>(q) = (uint16_t)b[0];
        else
          *q = (uint8_t)b[0];
      }
    }
  };
  if (staged) rows(std::true_type{});
  else rows(std::false_type{});
}

template <int XB, int V>
static int launch_bin_xv(const LaunchArgs &a, const BinTables &bt, bool lds, int threads,
                         int64_t blocks, int64_t rows, void *stream) {
  const auto k = lds ? bin_kernel<XB, V, true> : bin_kernel<XB, V, false>;
  const int bytes = lds ? bt.lds_bytes : 0;
  const int e = ensure_lds_limit((const void *)k, bytes);
  if (e != 0) return e;
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), bytes, (hipStream_t)stream, a, bt,
                     rows);
  return (int)hipGetLastError();
}

int launch_bin(const LaunchArgs &a, const BinTables &bt, bool lds, bool v4, void *stream) {
  int threads = kBinThreads;
  int64_t blocks, rows;
  if (lds) {
    // Whole rounds of resident workgroups: every workgroup has the same work, so a last round with
    // few of them costs as much as a full one.  Few rounds, since each stages its tables.
    const int64_t slots = (int64_t)256 * (bt.lds_bytes <= kLdsBytesPerCU / 2 ? 2 : 1);
    int64_t per_run = 1;
    double best = 0.0;
    for (int k = 1; k <= 4; ++k) {
      const int64_t p = std::max<int64_t>(1, k * slots / bt.n_runs), wg = p * bt.n_runs;
      const double used = (double)wg / (double)((wg + slots - 1) / slots * slots);
      if (used > best + 0.03) {
        best = used;
        per_run = p;
      }
    }
    rows = std::max<int64_t>(64, (a.n_rows + per_run - 1) / per_run);
  } else {
    // tables in L2: a thread per column and four or two rows, in workgroups that a row fits
    if (!v4 ? bt.max_features <= 256 : bt.max_features <= 1024) threads = 256;
    const int64_t units = v4 ? (bt.max_features + 3) / 4 : bt.max_features;
    const int64_t pass = threads / units * (v4 ? 2 : 4);
    // at most 2^20 workgroups
    const int64_t passes = (a.n_rows * bt.n_runs + pass * (int64_t(1) << 20) - 1) / (pass * (int64_t(1) << 20));
    rows = pass * std::max<int64_t>(1, passes);
  }
  blocks = (a.n_rows + rows - 1) / rows * bt.n_runs;
  if (a.x_bytes == 2)
    return v4 ? launch_bin_xv<2, 4>(a, bt, lds, threads, blocks, rows, stream)
              : launch_bin_xv<2, 1>(a, bt, lds, threads, blocks, rows, stream);
  if (a.x_bytes == 1)
    return v4 ? launch_bin_xv<1, 4>(a, bt, lds, threads, blocks, rows, stream)
              : launch_bin_xv<1, 1>(a, bt, lds, threads, blocks, rows, stream);
  return (int)hipErrorInvalidValue;
}

}  // namespace bridger
