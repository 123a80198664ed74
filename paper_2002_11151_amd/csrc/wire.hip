// All-paths analytical wire model (Sec. IV-D: more paths than the shortest one): kernels and their launch.
#include "xbar_common.h"

using namespace xbar_detail;

namespace {

// ---------------------------------------------------------------------------------------------
// wire model with all first-order paths (Sec. IV-D: more paths than the shortest one)
//   a_ij = sum_j' G_ij' (r_source + (min(j,j') + 1) r_row)      drops on the row wire
//   b_ij = sum_i' G_i'j ((R - max(i,i')) r_col + r_sense)       rises on the column wire
//   G_ni = G / (1 + a + b),   plane = (G_ni+ - G_ni-) / dG
// Both sums split into a prefix and a suffix part, so one scan along the row and one along the column replace
// the O(R + C) sum per device.  Scratch: A[S_w][2][K][N] (double); the row kernel writes a into A, the column
// kernel adds b and leaves the plane value in the slot of array 0 (with one converter per array: each
// array's value in its own slot).
// ---------------------------------------------------------------------------------------------
struct WireArgs {
  const float* W;
  double* A;         // [S_w][2][K][N]
  int K, N, R, C, S_w, slice_bits, tiles_c;
  uint32_t flags;
  double g_min, dg, inv_dg, var_sigma, r_row, r_col, r_source, r_sense, qw, q_per_w;
  float w_max;
  uint64_t seed, step;
  const unsigned long long* step_add;   // optional device counter added to step
};

// Conductances of the device pair (slice s) of weight (k, n) before the wire model.
__device__ __forceinline__ void wire_device_pair(const WireArgs& a, NormalStream& rng, int k, int n, int s, double g[2]) {
  const int q = quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w);
  const int digit = (int)(((uint32_t)::abs(q) >> (a.slice_bits * s)) & ((1u << a.slice_bits) - 1));
  g[0] = a.g_min + (q > 0 ? digit * a.dg : 0.0);
  g[1] = a.g_min + (q < 0 ? digit * a.dg : 0.0);
  if (a.flags & XBAR_NI_VARIATION) {
    double z[2];
    rng.pair((((uint64_t)k * (uint64_t)a.N + (uint64_t)n) * (uint64_t)a.S_w + (uint64_t)s) * 2, z[0], z[1]);
    g[0] *= 1.0 + a.var_sigma * z[0];
    g[1] *= 1.0 + a.var_sigma * z[1];
  }
}

// grid (tiles x groups of 8 tile rows, S_w); a wave scans one tile row at a time (both arrays): the devices, computed
// once in a short loop (with variation they are most of the work), through LDS, then lane l holds the ceil(C / 64)
// consecutive columns that start at l ceil(C / 64).
__global__ __launch_bounds__(256) void wire_rows_kernel(WireArgs a) {
  __shared__ double2 line[4][256];                 // [wave][column]: the two arrays
  const int groups = (a.R + 7) >> 3;
  const int tile = blockIdx.x / groups, group = blockIdx.x - tile * groups;
  const int tr = tile / a.tiles_c, tc = tile - tr * a.tiles_c;
  const int s = blockIdx.y;
  const int k0 = tr * a.R, n0 = tc * a.C;
  const int rows = min(a.R, a.K - k0), cols = min(a.C, a.N - n0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int cpl = (a.C + 63) >> 6;
  const size_t pol_stride = (size_t)a.K * a.N;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
#pragma unroll 1
  for (int i = group * 8 + wave; i < min(rows, group * 8 + 8); i += 4) {
#pragma unroll 1
    for (int u = 0; u < cpl; ++u) {
      const int j = u * 64 + lane;
      double g[2] = {0.0, 0.0};
      if (j < cols) wire_device_pair(a, rng, k0 + i, n0 + j, s, g);
      line[wave][j] = make_double2(g[0], g[1]);
    }
    wave_exchange();
    double l0[4][2], l1[4][2];                     // inclusive prefixes inside the lane
    double run0[2] = {0.0, 0.0}, run1[2] = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= cpl) break;
      const int j = lane * cpl + u;
      const double2 v = line[wave][j];
      const double g[2] = {v.x, v.y};
#pragma unroll
      for (int pol = 0; pol < 2; ++pol) {
        run0[pol] += g[pol];                       // sum_{j' <= j} G
        run1[pol] += (double)(j + 1) * g[pol];     // sum_{j' <= j} (j' + 1) G
        l0[u][pol] = run0[pol];
        l1[u][pol] = run1[pol];
      }
    }
    double before0[2], before1[2], total[2];       // sums over the lanes to the left, and the row total
#pragma unroll
    for (int pol = 0; pol < 2; ++pol) {
      const double inc0 = wave_inclusive_scan(run0[pol], lane);
      const double inc1 = wave_inclusive_scan(run1[pol], lane);
      before0[pol] = inc0 - run0[pol];
      before1[pol] = inc1 - run1[pol];
      total[pol] = __shfl(inc0, 63, 64);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u >= cpl) break;
      const int j = lane * cpl + u;
      if (j < cols) {
        const size_t at = ((size_t)(2 * s) * a.K + k0 + i) * a.N + n0 + j;
#pragma unroll
        for (int pol = 0; pol < 2; ++pol) {
          const double p0 = before0[pol] + l0[u][pol], p1 = before1[pol] + l1[u][pol];
          a.A[at + pol * pol_stride] = a.r_source * total[pol] + a.r_row * (p1 + (double)(j + 1) * (total[pol] - p0));
        }
      }
    }
    wave_exchange();                               // the next row is written over this one
  }
}

// grid (tiles x strips of CB columns, S_w); thread = (segment of the tile rows, column).  The devices of a thread's few
// rows are computed once and kept in LDS; the segments' sums are exchanged, and a second walk knows, at every row, the
// sums over all devices above and below and finishes the plane value.  1024 threads with 4 rows each (128-row tiles):
// a layer has few tiles, so this pass is bound by the length of a thread's chain (a quarter of the rows per
// thread and every device computed twice took 54 us on a 333 x 91 layer).
template <int CB>
__global__ __launch_bounds__(1024) void wire_cols_kernel(WireArgs a) {
  constexpr int SEG = 1024 / CB;
  extern __shared__ double wire_lds[];
  double* tot = wire_lds;                          // [sum of G | sum of (R - i) G][array][SEG][CB]
  double2* dev = reinterpret_cast<double2*>(wire_lds + 4 * 1024);   // [row of the segment][1024]
  const int strips = (a.C + CB - 1) / CB;
  const int tile = blockIdx.x / strips, strip = blockIdx.x - tile * strips;
  const int tr = tile / a.tiles_c, tc = tile - tr * a.tiles_c;
  const int s = blockIdx.y;
  const int k0 = tr * a.R, n0 = tc * a.C;
  const int rows = min(a.R, a.K - k0), cols = min(a.C, a.N - n0);
  const int seg = threadIdx.x / CB, lane = threadIdx.x % CB;
  const int j = strip * CB + lane;
  const int per = (a.R + SEG - 1) / SEG;           // rows of a segment
  const int i_begin = seg * per, count = j < cols ? max(0, min(rows, i_begin + per) - i_begin) : 0;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
  double t0[2] = {0.0, 0.0}, t1[2] = {0.0, 0.0};
#pragma unroll 1
  for (int u = 0; u < count; ++u) {
    double g[2];
    wire_device_pair(a, rng, k0 + i_begin + u, n0 + j, s, g);
    dev[u * 1024 + threadIdx.x] = make_double2(g[0], g[1]);
#pragma unroll
    for (int pol = 0; pol < 2; ++pol) {
      t0[pol] += g[pol];
      t1[pol] += (double)(a.R - i_begin - u) * g[pol];
    }
  }
#pragma unroll
  for (int pol = 0; pol < 2; ++pol) {
    tot[(pol * SEG + seg) * CB + lane] = t0[pol];
    tot[((2 + pol) * SEG + seg) * CB + lane] = t1[pol];
  }
  __syncthreads();
  double above[2] = {0.0, 0.0}, below[2] = {0.0, 0.0}, total[2] = {0.0, 0.0};
#pragma unroll 8
  for (int g = 0; g < SEG; ++g)
#pragma unroll
    for (int pol = 0; pol < 2; ++pol) {
      const double x0 = tot[(pol * SEG + g) * CB + lane], x1 = tot[((2 + pol) * SEG + g) * CB + lane];
      total[pol] += x0;
      above[pol] += g < seg ? x0 : 0.0;            // sum_{i' <= i} G, starts at the segments above
      below[pol] += g >= seg ? x1 : 0.0;           // sum_{i' > i} (R - i') G, starts with this and later segments
    }
  const size_t pol_stride = (size_t)a.K * a.N;
#pragma unroll 4
  for (int u = 0; u < count; ++u) {
    const int i = i_begin + u;
    const size_t at = ((size_t)(2 * s) * a.K + k0 + i) * a.N + n0 + j;
    const double wa[2] = {a.A[at], a.A[at + pol_stride]};
    const double2 v = dev[u * 1024 + threadIdx.x];
    const double g[2] = {v.x, v.y};
    double e[2];
#pragma unroll
    for (int pol = 0; pol < 2; ++pol) {
      above[pol] += g[pol];
      below[pol] -= (double)(a.R - i) * g[pol];
      const double b = a.r_col * ((double)(a.R - i) * above[pol] + below[pol]) + a.r_sense * total[pol];
      e[pol] = g[pol] / (1.0 + wa[pol] + b);
    }
    if (a.flags & XBAR_ADC_PER_ARRAY) {            // each array is read on its own
      a.A[at] = e[0] * a.inv_dg;
      a.A[at + pol_stride] = e[1] * a.inv_dg;
    } else {
      a.A[at] = (e[0] - e[1]) * a.inv_dg;
    }
  }
}

template <int CB>
int launch_wire_cols(const WireArgs& w, unsigned tiles, hipStream_t st) {
  const int per = cdiv(w.R, 1024 / CB);
  const size_t lds = (size_t)1024 * (32 + 16 * per);
  const void* k = reinterpret_cast<const void*>(&wire_cols_kernel<CB>);
  if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return XBAR_EHIP;
  hipLaunchKernelGGL(wire_cols_kernel<CB>, dim3(tiles * (unsigned)cdiv(w.C, CB), (unsigned)w.S_w), dim3(1024), lds, st, w);
  return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
}

}  // namespace

namespace xbar_detail {

int launch_wire_model(const xbar_config* cfg, const float* W, int K, int N, float w_max, uint64_t step, double* wire_u,
                      hipStream_t st) {
  const Derived d = derive(cfg);
  WireArgs w;
  w.W = W; w.A = wire_u;
  w.K = K; w.N = N; w.R = cfg->xbar_rows; w.C = cfg->xbar_cols; w.S_w = d.S_w;
  w.slice_bits = cfg->slice_bits;
  w.qw = (double)((1u << cfg->weight_bits) - 1);
  w.q_per_w = w.qw / (double)w_max;
  w.tiles_c = cdiv(N, cfg->xbar_cols);
  w.flags = cfg->flags;
  w.g_min = 1.0 / (double)cfg->r_max;
  w.dg = (1.0 / (double)cfg->r_min - w.g_min) / (double)((1 << cfg->slice_bits) - 1);
  w.inv_dg = 1.0 / w.dg;
  w.var_sigma = (double)cfg->var_sigma;
  w.r_row = (double)cfg->r_row; w.r_col = (double)cfg->r_col;
  w.r_source = (double)cfg->r_source; w.r_sense = (double)cfg->r_sense;
  w.w_max = w_max; w.seed = cfg->seed; w.step = step; w.step_add = current_step_source();
  const unsigned tiles = (unsigned)(cdiv(K, cfg->xbar_rows) * w.tiles_c);
  hipLaunchKernelGGL(wire_rows_kernel, dim3(tiles * (unsigned)cdiv(cfg->xbar_rows, 8), (unsigned)d.S_w), dim3(256), 0, st, w);
  if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  // 32 columns per block up to 128 rows, 16 beyond: at most four rows per thread, whose devices take 64 KiB of LDS beside 32 of
  // sums, so one block of sixteen waves has a compute unit to itself
  return cfg->xbar_rows <= 128 ? launch_wire_cols<32>(w, tiles, st) : launch_wire_cols<16>(w, tiles, st);
}

}  // namespace xbar_detail
