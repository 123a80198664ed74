// Digital peripheral operations of a crossbar-based network (Sec. IV-B: ReLU, batch normalisation and
// pooling are computed in the digital domain and are not touched by the crossbar non-idealities), plus
// the loss and the plain SGD step of the digital parameters, so that a whole training step runs on the
// GPU.  Activations are NHWC float tensors; sums that decide statistics are accumulated in double
// precision in a fixed order (deterministic).  All of it is HBM-bound elementwise or reduction work.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "xbar.h"

namespace {

inline bool aligned16(const void* p) { return p != nullptr && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }
constexpr int kStatRows = 512;    // rows per block of the per-channel reductions

// Elementwise passes: bound by HBM (large tensors: up to 4.6 TB/s) or by the launch (small ones).  A thread takes one quad, or four
// where that still leaves eight blocks per compute unit: their loads are in flight together.  The last thread takes the odd elements.
struct ReluFwd {
  static constexpr int kInputs = 1;
  __device__ static float of(float a, float, float) { return a > 0.0f ? a : 0.0f; }
};
struct ReluBwd {       // a: the forward output, b: the error
  static constexpr int kInputs = 2;
  __device__ static float of(float a, float b, float) { return a > 0.0f ? b : 0.0f; }
};
struct Add {
  static constexpr int kInputs = 2;
  __device__ static float of(float a, float b, float) { return a + b; }
};
struct AddReluBwd {    // a: the forward output, b + c: the error
  static constexpr int kInputs = 3;
  __device__ static float of(float a, float b, float c) { return a > 0.0f ? b + c : 0.0f; }
};

template <class OP, int QUADS>
__global__ __launch_bounds__(256) void flat_kernel(const float* a, const float* b, const float* c, float* y, size_t n) {
  const size_t n4 = n >> 2, q0 = (size_t)blockIdx.x * (256 * QUADS) + threadIdx.x;
  float4 va[QUADS], vb[QUADS], vc[QUADS];
#pragma unroll
  for (int u = 0; u < QUADS; ++u) {
    const size_t q = q0 + 256 * u;
    va[u] = vb[u] = vc[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (q < n4) {
      va[u] = reinterpret_cast<const float4*>(a)[q];
      if (OP::kInputs > 1) vb[u] = reinterpret_cast<const float4*>(b)[q];
      if (OP::kInputs > 2) vc[u] = reinterpret_cast<const float4*>(c)[q];
    }
  }
#pragma unroll
  for (int u = 0; u < QUADS; ++u) {
    const size_t q = q0 + 256 * u;
    if (q < n4)
      reinterpret_cast<float4*>(y)[q] = make_float4(OP::of(va[u].x, vb[u].x, vc[u].x), OP::of(va[u].y, vb[u].y, vc[u].y),
                                                    OP::of(va[u].z, vb[u].z, vc[u].z), OP::of(va[u].w, vb[u].w, vc[u].w));
    if (q == n4)
      for (size_t i = n4 * 4; i < n; ++i)
        y[i] = OP::of(a[i], OP::kInputs > 1 ? b[i] : 0.0f, OP::kInputs > 2 ? c[i] : 0.0f);
  }
}

template <class OP>
void launch_flat(const float* a, const float* b, const float* c, float* y, size_t n, hipStream_t st) {
  const size_t quads = (n + 3) >> 2;
  if (quads >= (size_t)4 * 256 * 2048)
    hipLaunchKernelGGL((flat_kernel<OP, 4>), dim3((unsigned)((quads + 1023) / 1024)), dim3(256), 0, st, a, b, c, y, n);
  else
    hipLaunchKernelGGL((flat_kernel<OP, 1>), dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, a, b, c, y, n);
}

// Logistic function; the exponential is taken in double precision so that the float result is the
// correctly rounded one in all but rare cases.
__global__ __launch_bounds__(256) void sigmoid_fwd_kernel(const float* x, float* y, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = (float)(1.0 / (1.0 + ::exp(-(double)x[i])));
}

__global__ __launch_bounds__(256) void sigmoid_bwd_kernel(const float* y, const float* dy, float* dx, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    const double s = (double)y[i];
    dx[i] = (float)((double)dy[i] * s * (1.0 - s));
  }
}

__device__ __forceinline__ float sgd_step(float p, float g, float lr) { return p - lr * g; }

__global__ __launch_bounds__(256) void sgd_kernel(float* p, const float* g, size_t n, float lr) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = sgd_step(p[i], g[i], lr);
}

// VEC consecutive floats of memory (one, or four from a 16-byte boundary).
template <int VEC>
__device__ __forceinline__ void load_vec(const float* p, float (&v)[VEC]) {
  if constexpr (VEC == 4) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  } else {
    v[0] = *p;
  }
}
template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&v)[VEC]) {
  if constexpr (VEC == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  else *p = v[0];
}

// A channel's normalisation.  `of` is the forward output: the backward pass of normalisation and ReLU in one evaluates it again and
// must find the same sign, so it is written without room for the compiler to contract it in two ways.
struct Norm {
  double gamma, beta, mean, invstd;
  __device__ __forceinline__ double xhat(float x) const { return ((double)x - mean) * invstd; }
  __device__ __forceinline__ float of(float x) const { return (float)__builtin_fma(gamma, xhat(x), beta); }
};
// Channels c .. of the parameters; gamma and beta (null: not needed) one every `stride` floats.
template <int VEC>
__device__ __forceinline__ void load_norm(Norm (&n)[VEC], const float* gamma, const float* beta, int stride, const float* mean,
                                          const float* invstd, int c) {
  float g[VEC], b[VEC], mu[VEC], is[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) g[e] = b[e] = 0.0f;
  if (stride == 1) {
    if (gamma) load_vec<VEC>(gamma + c, g);
    if (beta) load_vec<VEC>(beta + c, b);
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      g[e] = gamma[(size_t)(c + e) * stride];
      if (beta) b[e] = beta[(size_t)(c + e) * stride];
    }
  }
  load_vec<VEC>(mean + c, mu);
  load_vec<VEC>(invstd + c, is);
#pragma unroll
  for (int e = 0; e < VEC; ++e) n[e] = Norm{(double)g[e], (double)b[e], (double)mu[e], (double)is[e]};
}

// Per-channel sums over a block of rows: part[chunk][channel][2] = (sum x, sum x^2), or with BWD (sum dy, sum dy xhat); RELU: of
// the errors where the normalised value was positive.  A thread takes VEC neighbouring channels (four 16 bytes wide, where the rows
// allow it), LANES threads a strip of channels, 256 / LANES groups of threads the rows; HBM-bound where rows are many, else a
// block's chain of loads and sums.  us, against one channel per thread and a sum of all groups by one thread: 8192 x 64 forward
// 11.6 -> 4.4, backward 14.1 -> 6.2; all 53 forward layers of a ResNet-50 at batch 64 867 -> 700, the backward ones 1715 -> 1554
// with the ReLU's passes in them.
template <bool BWD, bool RELU, int VEC, int LANES>
__global__ __launch_bounds__(256) void bn_partial_kernel(const float* x, const float* dy, const float* gamma, const float* beta,
                                                         const float* mean, const float* invstd, double* part, size_t rows, int C) {
  constexpr int G = 256 / LANES, CT = VEC * LANES, VALUES = 2 * CT, SHARES = 256 / VALUES;
  __shared__ double red[2][G][CT];
  __shared__ double shares[SHARES][VALUES];
  const int lane = threadIdx.x % LANES, grp = threadIdx.x / LANES;
  const int c = blockIdx.y * CT + VEC * lane;
  const size_t r0 = (size_t)blockIdx.x * kStatRows;
  const size_t r1 = r0 + kStatRows < rows ? r0 + kStatRows : rows;
  double s0[VEC], s1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s0[e] = s1[e] = 0.0;
  if (c < C) {
    Norm nm[VEC];
    if (BWD) load_norm<VEC>(nm, RELU ? gamma : nullptr, RELU ? beta : nullptr, 1, mean, invstd, c);
#pragma unroll 4
    for (size_t r = r0 + grp; r < r1; r += G) {
      float v[VEC], d[VEC];
      load_vec<VEC>(x + r * C + c, v);
      if (BWD) load_vec<VEC>(dy + r * C + c, d);
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if (BWD) {
          const double g = !RELU || nm[e].of(v[e]) > 0.0f ? (double)d[e] : 0.0;
          s0[e] += g;                       // sum dy
          s1[e] += g * nm[e].xhat(v[e]);    // sum dy xhat
        } else {
          s0[e] += (double)v[e];
          s1[e] += (double)v[e] * (double)v[e];
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    red[0][grp][VEC * lane + e] = s0[e];
    red[1][grp][VEC * lane + e] = s1[e];
  }
  __syncthreads();
  const int value = threadIdx.x % VALUES, share = threadIdx.x / VALUES;     // every sum in a fixed order
  double t = 0.0;
#pragma unroll
  for (int g = share; g < G; g += SHARES) t += red[value / CT][g][value % CT];
  shares[share][value] = t;
  __syncthreads();
  const int cv = blockIdx.y * CT + value % CT;
  if (threadIdx.x < VALUES && cv < C) {
    t = 0.0;
#pragma unroll
    for (int k = 0; k < SHARES; ++k) t += shares[k][value];
    part[((size_t)blockIdx.x * C + cv) * 2 + value / CT] = t;
  }
}

// One wave per channel adds the chunk sums: lane l takes chunks l, l + 64, ..., then a fixed
// butterfly over the lanes.
__device__ __forceinline__ void bn_chunk_sums(const double* part, int chunks, int C, int c, double& s0, double& s1) {
  const int lane = threadIdx.x & 63;
  s0 = s1 = 0.0;
  for (int k = lane; k < chunks; k += 64) {
    s0 += part[((size_t)k * C + c) * 2];
    s1 += part[((size_t)k * C + c) * 2 + 1];
  }
#pragma unroll
  for (int d = 32; d; d >>= 1) {
    s0 += __shfl_xor(s0, d, 64);
    s1 += __shfl_xor(s1, d, 64);
  }
}

__global__ __launch_bounds__(256) void bn_finalize_fwd_kernel(const double* part, int chunks, int C, size_t rows,
                                                              float eps, float* mean, float* invstd) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= C) return;                                 // whole waves leave together
  double s0, s1;
  bn_chunk_sums(part, chunks, C, c, s0, s1);
  if ((threadIdx.x & 63) != 0) return;
  const double mu = s0 / (double)rows;
  double var = s1 / (double)rows - mu * mu;        // biased variance of the batch
  if (var < 0.0) var = 0.0;
  mean[c] = (float)mu;
  invstd[c] = (float)(1.0 / ::sqrt(var + (double)eps));
}

// With `step` also the SGD step of the channel's parameters: what they were, which the last kernel needs, takes the place of the
// channel's first partial sums (this wave alone has read them).
__global__ __launch_bounds__(256) void bn_finalize_bwd_kernel(double* part, int chunks, int C, float* dgamma, float* dbeta,
                                                              float* gamma, float* beta, int step, float lr) {
  const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= C) return;
  double s0, s1;
  bn_chunk_sums(part, chunks, C, c, s0, s1);
  if ((threadIdx.x & 63) != 0) return;
  dbeta[c] = (float)s0;
  dgamma[c] = (float)s1;
  if (step) {
    const float g = gamma[c], b = beta[c];
    float* old = reinterpret_cast<float*>(part + (size_t)c * 2);
    old[0] = g;
    old[1] = b;
    gamma[c] = sgd_step(g, (float)s1, lr);
    beta[c] = sgd_step(b, (float)s0, lr);
  }
}

// Which elements a thread of the normalisation's last kernels has: VEC channels of ROWS rows.  Rows of quads: `lanes` (a power of two)
// threads side by side along the channels.  Other rows: threads side by side through the rows as they lie in memory, a fixed
// number of whole rows apart from one of a thread's elements to the next (lanes of powers of two leave half of the threads of 257
// channels without one: 50176 x 257, forward and backward 42.1 -> 37.1, 58.6 -> 51.4 us).
template <int VEC, int ROWS>
struct RowSpan {
  int c;
  size_t r0, step;
  __device__ __forceinline__ RowSpan(int lanes_log2, size_t rows, int C) {
    if constexpr (VEC == 1) {
      const uint32_t t = blockIdx.x * 256u + threadIdx.x, row = t / (uint32_t)C;
      step = (rows + ROWS - 1) / ROWS;
      r0 = row;
      c = row < step ? (int)(t - row * (uint32_t)C) : C;         // C: none
    } else {
      const int lanes = 1 << lanes_log2;
      step = 256 >> lanes_log2;
      c = VEC * ((int)blockIdx.y * lanes + ((int)threadIdx.x & (lanes - 1)));
      r0 = (size_t)blockIdx.x * ROWS * step + (threadIdx.x >> lanes_log2);
    }
  }
};

// y = normalised x; RELU: its positive part, after `skip` has been added where there is one.  HBM-bound; the channel's parameters
// are read and converted once per thread.  Passes over memory of a layer's forward and backward step with ReLU: 8 instead of 13
// (ResNet-50, batch 64: all digital passes 11.2 -> 6.9 ms; ResNet-20, batch 128: 200 launches of some 4 us -> 110).
template <bool RELU, int VEC, int ROWS>
__global__ __launch_bounds__(256) void bn_apply_fwd_kernel(const float* x, const float* skip, const float* gamma, const float* beta,
                                                           const float* mean, const float* invstd, float* y, size_t rows, int C,
                                                           int lanes_log2) {
  const RowSpan<VEC, ROWS> at(lanes_log2, rows, C);
  if (at.c >= C) return;
  float v[ROWS][VEC], s[ROWS][VEC];
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const size_t r = at.r0 + u * at.step;
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[u][e] = s[u][e] = 0.0f;
    if (r < rows) {
      load_vec<VEC>(x + r * C + at.c, v[u]);
      if (RELU && skip) load_vec<VEC>(skip + r * C + at.c, s[u]);
    }
  }
  Norm nm[VEC];
  load_norm<VEC>(nm, gamma, beta, 1, mean, invstd, at.c);
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const size_t r = at.r0 + u * at.step;
    float o[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      o[e] = nm[e].of(v[u][e]);
      if (RELU && skip) o[e] += s[u][e];
      if (RELU) o[e] = o[e] > 0.0f ? o[e] : 0.0f;
    }
    if (r < rows) store_vec<VEC>(y + r * C + at.c, o);
  }
}

// gamma, beta: one every `stride` floats.
template <bool RELU, int VEC, int ROWS>
__global__ __launch_bounds__(256) void bn_apply_bwd_kernel(const float* x, const float* dy, const float* gamma, const float* beta,
                                                           int stride, const float* mean, const float* invstd, const float* dgamma,
                                                           const float* dbeta, float* dx, size_t rows, int C, int lanes_log2,
                                                           double inv_rows) {
  const RowSpan<VEC, ROWS> at(lanes_log2, rows, C);
  if (at.c >= C) return;
  float v[ROWS][VEC], d[ROWS][VEC];
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const size_t r = at.r0 + u * at.step;
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[u][e] = d[u][e] = 0.0f;
    if (r < rows) {
      load_vec<VEC>(x + r * C + at.c, v[u]);
      load_vec<VEC>(dy + r * C + at.c, d[u]);
    }
  }
  Norm nm[VEC];
  load_norm<VEC>(nm, gamma, RELU ? beta : nullptr, stride, mean, invstd, at.c);
  float dg[VEC], db[VEC];
  load_vec<VEC>(dgamma + at.c, dg);
  load_vec<VEC>(dbeta + at.c, db);
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const size_t r = at.r0 + u * at.step;
    float o[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float g = !RELU || nm[e].of(v[u][e]) > 0.0f ? d[u][e] : 0.0f;
      o[e] = (float)(nm[e].gamma * nm[e].invstd *
                     ((double)g - (double)db[e] * inv_rows - nm[e].xhat(v[u][e]) * (double)dg[e] * inv_rows));
    }
    if (r < rows) store_vec<VEC>(dx + r * C + at.c, o);
  }
}

// The launch of either: one row per thread, or four where that leaves eight blocks per compute unit.
struct ApplyGrid {
  int lanes_log2 = 0, four_rows;
  dim3 grid;
  ApplyGrid(size_t rows, int C, int vec) {
    if (vec == 1) {
      four_rows = rows * (size_t)C / 256 >= 4 * 2048;
      grid = dim3((unsigned)(((four_rows ? (rows + 3) / 4 : rows) * (size_t)C + 255) / 256));
      return;
    }
    const int across = C / vec;
    while (lanes_log2 < 8 && (1 << lanes_log2) < across) ++lanes_log2;
    const size_t step = 256 >> lanes_log2, strips = (size_t)(across + (1 << lanes_log2) - 1) >> lanes_log2;
    const size_t blocks = (rows + step - 1) / step;
    four_rows = blocks * strips >= 4 * 2048;
    grid = dim3((unsigned)(four_rows ? (blocks + 3) / 4 : blocks), (unsigned)strips);
  }
};

// GROUPS threads share the positions of an output, 256 / GROUPS outputs side by side, AHEAD loads of a thread in flight.  us, 1 / 4 /
// 16 threads an output: 8192 outputs of 64 positions 4.6 / 3.2 / 3.0, of 784 28 / 9.1 / 9.7; 32768 of 49 4.3 / 3.3 / 4.1; 65536 of 49
// 4.3 / 3.7 / 5.5, of 9 3.0 / 3.2 / 4.5; 131072 of 49 4.5 / 4.6 / 12, of 16 3.3 / 3.9 / 6.7; 524288 of 49 17 / 17 / 39; any of up to four
// positions 1.  (A thread each for 16 channels of a sample, 16 threads a channel, whatever the sizes: the 64 x 49 x 2048 of a ResNet-50 at
// batch 64 12.1, with a thread an output and one load at a time 8.2, now 4.5; 2097152 of one position 61, 6.0, 7.3.)
constexpr size_t kPoolBlocks = 1 << 20;     // of one launch; beyond that a block takes several

template <int GROUPS, int AHEAD>
__global__ __launch_bounds__(256) void avgpool_fwd_kernel(const float* x, float* y, size_t outputs, int positions, int C) {
  constexpr int LANES = 256 / GROUPS;
  __shared__ double red[GROUPS][LANES];
  const int lane = threadIdx.x % LANES, grp = threadIdx.x / LANES;
  for (size_t o0 = (size_t)blockIdx.x * LANES; o0 < outputs; o0 += (size_t)gridDim.x * LANES) {
    const size_t o = o0 + lane;
    double s = 0.0;
    if (o < outputs) {
      const size_t b = outputs >> 32 ? o / (size_t)C : (uint32_t)o / (uint32_t)C, c = o - b * C;
      const float* from = x + b * positions * C + c;
#pragma unroll AHEAD
      for (int p = grp; p < positions; p += GROUPS) s += (double)from[(size_t)p * C];
    }
    if constexpr (GROUPS > 1) {
      red[grp][lane] = s;
      __syncthreads();
      s = 0.0;
#pragma unroll
      for (int g = 0; g < GROUPS; ++g) s += red[g][lane];        // fixed order
    }
    if (grp == 0 && o < outputs) y[o] = (float)(s / (double)positions);
    if constexpr (GROUPS > 1) __syncthreads();
  }
}

template <int GROUPS, int AHEAD>
void launch_avgpool(const float* x, float* y, size_t outputs, int positions, int C, hipStream_t st) {
  const size_t blocks = (outputs + 256 / GROUPS - 1) / (256 / GROUPS);
  hipLaunchKernelGGL((avgpool_fwd_kernel<GROUPS, AHEAD>), dim3((unsigned)(blocks < kPoolBlocks ? blocks : kPoolBlocks)), dim3(256), 0, st, x, y,
                     outputs, positions, C);
}

__global__ __launch_bounds__(256) void avgpool_bwd_kernel(const float* dy, float* dx, int batch, int positions, int C) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)batch * positions * C) return;
  const int c = (int)(i % C);
  const size_t b = i / ((size_t)positions * C);
  dx[i] = dy[b * C + c] / (float)positions;
}

struct PoolGeom {
  int B, H, W, C, k, stride, pad, OH, OW;
};

// Place of thread i in a [b][h][w][channels / VEC] tensor.
struct PoolAt {
  int b, h, w, c;
  __device__ __forceinline__ PoolAt(uint32_t i, int H, int W, int vecs, int vec) {
    c = vec * (int)(i % (uint32_t)vecs);
    i /= (uint32_t)vecs;
    w = (int)(i % (uint32_t)W);
    i /= (uint32_t)W;
    h = (int)(i % (uint32_t)H);
    b = (int)(i / (uint32_t)H);
  }
};

// VEC neighbouring channels per thread: four where the rows are quads (16-byte loads, a quarter of the index arithmetic).
// 64 x 112 x 112 x 64, windows of 3: forward 157 -> 70 us, backward 361 -> 97.
template <int VEC>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const float* x, float* y, int32_t* arg, PoolGeom g, uint32_t threads) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= threads) return;
  const PoolAt at(i, g.OH, g.OW, g.C / VEC, VEC);
  float best[VEC];
  int32_t best_at[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    best[e] = -INFINITY;
    best_at[e] = -1;
  }
  const int ih0 = at.h * g.stride - g.pad, iw0 = at.w * g.stride - g.pad;
  const int ih1 = min(ih0 + g.k, g.H), iw1 = min(iw0 + g.k, g.W);
  const float* image = x + (size_t)at.b * g.H * g.W * g.C + at.c;
  for (int ih = max(ih0, 0); ih < ih1; ++ih)
    for (int iw = max(iw0, 0); iw < iw1; ++iw) {
      const int32_t pos = ih * g.W + iw;                     // position inside the image; first maximum wins
      float v[VEC];
      load_vec<VEC>(image + (size_t)pos * g.C, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (v[e] > best[e]) { best[e] = v[e]; best_at[e] = pos; }
    }
  const size_t o = (((size_t)at.b * g.OH + at.h) * g.OW + at.w) * g.C + at.c;
  store_vec<VEC>(y + o, best);
  if constexpr (VEC == 4) *reinterpret_cast<int4*>(arg + o) = make_int4(best_at[0], best_at[1], best_at[2], best_at[3]);
  else arg[o] = best_at[0];
}

// Gather form of the backward pass: an input pixel adds the errors of the windows that chose it, the last window first.
template <int VEC>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const float* dy, const int32_t* arg, float* dx, PoolGeom g, uint32_t threads) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= threads) return;
  const PoolAt at(i, g.H, g.W, g.C / VEC, VEC);
  const int32_t me = at.h * g.W + at.w;
  float s[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s[e] = 0.0f;
  const int y0 = at.h + g.pad, x0 = at.w + g.pad;            // windows oh: oh stride <= y0 < oh stride + k
  const int oh1 = min(y0 / g.stride, g.OH - 1), ow1 = min(x0 / g.stride, g.OW - 1);
  const int oh0 = y0 < g.k ? 0 : (y0 - g.k) / g.stride + 1, ow0 = x0 < g.k ? 0 : (x0 - g.k) / g.stride + 1;
  for (int oh = oh1; oh >= oh0; --oh)
    for (int ow = ow1; ow >= ow0; --ow) {
      const size_t o = (((size_t)at.b * g.OH + oh) * g.OW + ow) * g.C + at.c;
      float d[VEC];
      load_vec<VEC>(dy + o, d);
      int32_t chosen[VEC];
      if constexpr (VEC == 4) {
        const int4 q = *reinterpret_cast<const int4*>(arg + o);
        chosen[0] = q.x; chosen[1] = q.y; chosen[2] = q.z; chosen[3] = q.w;
      } else {
        chosen[0] = arg[o];
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (chosen[e] == me) s[e] += d[e];
    }
  store_vec<VEC>(dx + (((size_t)at.b * g.H + at.h) * g.W + at.w) * g.C + at.c, s);
}

// One wave per sample: loss = log(sum exp(z - max)) - (z_label - max), dlogits = scale (softmax - onehot).
__global__ __launch_bounds__(64) void softmax_xent_kernel(const float* logits, const int32_t* labels, float* loss,
                                                          float* dlogits, int classes, float scale) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const float* z = logits + (size_t)b * classes;
  float mx = -INFINITY;
  for (int j = lane; j < classes; j += 64) mx = fmaxf(mx, z[j]);
  for (int d = 32; d; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
  double s = 0.0;
  for (int j = lane; j < classes; j += 64) s += ::exp((double)z[j] - (double)mx);
  for (int d = 32; d; d >>= 1) s += __shfl_xor(s, d, 64);
  const int label = labels[b];
  const bool known = label >= 0 && label < classes;          // an unknown label gives a NaN loss, no target
  if (lane == 0) loss[b] = known ? (float)(::log(s) - ((double)z[label] - (double)mx)) : NAN;
  for (int j = lane; j < classes; j += 64) {
    const double pj = ::exp((double)z[j] - (double)mx) / s;
    dlogits[(size_t)b * classes + j] = (float)((double)scale * (pj - (j == label ? 1.0 : 0.0)));
  }
}

// Parameter-free residual shortcut across a stage boundary: spatial subsampling by `stride` and zero
// padding of the new channels, half before and half behind the old ones.
struct ShortcutGeom {
  int B, H, W, C, stride, OH, OW, OC, lo;
};

__global__ __launch_bounds__(256) void shortcut_fwd_kernel(const float* x, float* y, ShortcutGeom g) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)g.B * g.OH * g.OW * g.OC) return;
  const int oc = (int)(i % g.OC);
  size_t u = i / g.OC;
  const int ow = (int)(u % g.OW);
  u /= g.OW;
  const int oh = (int)(u % g.OH), b = (int)(u / g.OH);
  const int c = oc - g.lo;
  y[i] = (c >= 0 && c < g.C) ? x[(((size_t)b * g.H + oh * g.stride) * g.W + ow * g.stride) * g.C + c] : 0.0f;
}

__global__ __launch_bounds__(256) void shortcut_bwd_kernel(const float* dy, float* dx, ShortcutGeom g) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (size_t)g.B * g.H * g.W * g.C) return;
  const int c = (int)(i % g.C);
  size_t u = i / g.C;
  const int iw = (int)(u % g.W);
  u /= g.W;
  const int ih = (int)(u % g.H), b = (int)(u / g.H);
  const bool kept = ih % g.stride == 0 && iw % g.stride == 0 && ih / g.stride < g.OH && iw / g.stride < g.OW;
  dx[i] = kept ? dy[(((size_t)b * g.OH + ih / g.stride) * g.OW + iw / g.stride) * g.OC + c + g.lo] : 0.0f;
}

// max |x|: per-block maxima, then one block over them.  |x| is compared as an unsigned integer (the
// order of non-negative floats); a NaN input gives a NaN-patterned result.
__global__ __launch_bounds__(256) void absmax_kernel(const float* x, size_t n, uint32_t* part) {
  __shared__ uint32_t red[4];
  uint32_t m = 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const uint32_t v = __float_as_uint(x[i]) & 0x7FFFFFFFu;
    m = v > m ? v : m;
  }
  for (int d = 32; d; d >>= 1) {
    const uint32_t o = (uint32_t)__shfl_xor((int)m, d, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) m = red[w] > m ? red[w] : m;
    part[blockIdx.x] = m;
  }
}

// Strips of 64 channels (whole 256-byte pieces of a row) where they make 160 blocks or more, else of 16: blocks enough outweigh that
// another block takes the other half of a 128-byte line.  us, whole calls, strips of 16 / of 64, forward, backward: 12544 x 256 (100
// blocks of 64) 14.4 / 14.3, 20.0 / 25.1, 2000 x 2048 (128) 17.3 / 15.9, 25.0 / 27.5; 12544 x 512 (200) 22.6 / 20.0, 35.3 / 33.3, 50000 x 130
// (294) 27.2 / 29.3, 42.5 / 34.9, 12544 x 1024 (400) 36.6 / 30.0, 58.8 / 44.9, 50176 x 257 (490) 51.7 / 42.1, 82.4 / 58.6.
template <bool BWD, bool RELU>
void launch_bn_partial(const float* x, const float* dy, const float* gamma, const float* beta, const float* mean, const float* invstd,
                       double* part, size_t rows, int channels, int chunks, hipStream_t st) {
  const int wide = (channels + 63) / 64;
  const bool narrow = channels <= 32 || (long long)chunks * wide < 160;
  const dim3 grid((unsigned)chunks, (unsigned)(narrow ? (channels + 15) / 16 : wide));
  void (*k)(const float*, const float*, const float*, const float*, const float*, const float*, double*, size_t, int);
  if ((channels & 3) == 0) k = narrow ? bn_partial_kernel<BWD, RELU, 4, 4> : bn_partial_kernel<BWD, RELU, 4, 16>;
  else k = narrow ? bn_partial_kernel<BWD, RELU, 1, 16> : bn_partial_kernel<BWD, RELU, 1, 64>;
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, x, dy, gamma, beta, mean, invstd, part, rows, channels);
}

inline int launched() { return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP; }

}  // namespace

extern "C" {

int xbar_relu_fwd(const float* x, float* y, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(y)) return XBAR_EALIGN;
  launch_flat<ReluFwd>(x, nullptr, nullptr, y, n, reinterpret_cast<hipStream_t>(hip_stream));
  return launched();
}

int xbar_relu_bwd(const float* y, const float* dy, float* dx, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(y) || !aligned16(dy) || !aligned16(dx)) return XBAR_EALIGN;
  launch_flat<ReluBwd>(y, dy, nullptr, dx, n, reinterpret_cast<hipStream_t>(hip_stream));
  return launched();
}

int xbar_sigmoid_fwd(const float* x, float* y, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(y)) return XBAR_EALIGN;
  hipLaunchKernelGGL(sigmoid_fwd_kernel, dim3(blocks_for(n)), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream), x, y, n);
  return launched();
}

int xbar_sigmoid_bwd(const float* y, const float* dy, float* dx, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(y) || !aligned16(dy) || !aligned16(dx)) return XBAR_EALIGN;
  hipLaunchKernelGGL(sigmoid_bwd_kernel, dim3(blocks_for(n)), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream), y, dy,
                     dx, n);
  return launched();
}

int xbar_add(const float* a, const float* b, float* y, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(a) || !aligned16(b) || !aligned16(y)) return XBAR_EALIGN;
  launch_flat<Add>(a, b, nullptr, y, n, reinterpret_cast<hipStream_t>(hip_stream));
  return launched();
}

int xbar_add_relu_bwd(const float* y, const float* a, const float* b, float* dx, size_t n, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(y) || !aligned16(a) || !aligned16(b) || !aligned16(dx)) return XBAR_EALIGN;
  launch_flat<AddReluBwd>(y, a, b, dx, n, reinterpret_cast<hipStream_t>(hip_stream));
  return launched();
}

int xbar_sgd(float* p, const float* g, size_t n, float lr, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(p) || !aligned16(g)) return XBAR_EALIGN;
  if (!std::isfinite(lr)) return XBAR_EINVAL;
  hipLaunchKernelGGL(sgd_kernel, dim3(blocks_for(n)), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream), p, g, n, lr);
  return launched();
}

size_t xbar_bn_workspace_bytes(size_t rows, int channels) {
  if (rows == 0 || channels <= 0) return 0;
  const size_t chunks = (rows + kStatRows - 1) / kStatRows;
  return align256(chunks * (size_t)channels * 2 * sizeof(double));
}

static int bn_fwd(const float* x, const float* gamma, const float* beta, const float* skip, bool relu, float* y, float* mean,
                  float* invstd, size_t rows, int channels, float eps, void* ws, size_t ws_bytes, hipStream_t st) {
  if (rows == 0 || channels <= 0 || rows > ((size_t)1 << 31)) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(gamma) || !aligned16(beta) || !aligned16(y) || !aligned16(mean) || !aligned16(invstd) ||
      !aligned16(ws) || (skip && !aligned16(skip)))
    return XBAR_EALIGN;
  if (!(eps >= 0.0f) || !std::isfinite(eps)) return XBAR_EINVAL;
  if (ws_bytes < xbar_bn_workspace_bytes(rows, channels)) return XBAR_EWORKSPACE;
  const int chunks = (int)((rows + kStatRows - 1) / kStatRows);
  double* part = reinterpret_cast<double*>(ws);
  launch_bn_partial<false, false>(x, nullptr, nullptr, nullptr, nullptr, nullptr, part, rows, channels, chunks, st);
  if (launched()) return XBAR_EHIP;
  hipLaunchKernelGGL(bn_finalize_fwd_kernel, dim3((unsigned)((channels + 3) / 4)), dim3(256), 0, st, part, chunks, channels,
                     rows, eps, mean, invstd);
  if (launched()) return XBAR_EHIP;
  const ApplyGrid at(rows, channels, (channels & 3) == 0 ? 4 : 1);
  void (*k)(const float*, const float*, const float*, const float*, const float*, const float*, float*, size_t, int, int);
  if ((channels & 3) == 0) {
    if (relu) k = at.four_rows ? bn_apply_fwd_kernel<true, 4, 4> : bn_apply_fwd_kernel<true, 4, 1>;
    else k = at.four_rows ? bn_apply_fwd_kernel<false, 4, 4> : bn_apply_fwd_kernel<false, 4, 1>;
  } else {
    if (relu) k = at.four_rows ? bn_apply_fwd_kernel<true, 1, 4> : bn_apply_fwd_kernel<true, 1, 1>;
    else k = at.four_rows ? bn_apply_fwd_kernel<false, 1, 4> : bn_apply_fwd_kernel<false, 1, 1>;
  }
  hipLaunchKernelGGL(k, at.grid, dim3(256), 0, st, x, skip, gamma, beta, mean, invstd, y, rows, channels, at.lanes_log2);
  return launched();
}

static int bn_bwd(const float* x, const float* dy, float* gamma, float* beta, const float* mean, const float* invstd, float* dx,
                  float* dgamma, float* dbeta, size_t rows, int channels, bool relu, bool step, float lr, void* ws, size_t ws_bytes,
                  hipStream_t st) {
  if (rows == 0 || channels <= 0 || rows > ((size_t)1 << 31)) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(dy) || !aligned16(gamma) || !aligned16(mean) || !aligned16(invstd) || !aligned16(dx) ||
      !aligned16(dgamma) || !aligned16(dbeta) || !aligned16(ws))
    return XBAR_EALIGN;
  if (ws_bytes < xbar_bn_workspace_bytes(rows, channels)) return XBAR_EWORKSPACE;
  const int chunks = (int)((rows + kStatRows - 1) / kStatRows);
  double* part = reinterpret_cast<double*>(ws);
  if (relu) launch_bn_partial<true, true>(x, dy, gamma, beta, mean, invstd, part, rows, channels, chunks, st);
  else launch_bn_partial<true, false>(x, dy, gamma, beta, mean, invstd, part, rows, channels, chunks, st);
  if (launched()) return XBAR_EHIP;
  hipLaunchKernelGGL(bn_finalize_bwd_kernel, dim3((unsigned)((channels + 3) / 4)), dim3(256), 0, st, part, chunks, channels,
                     dgamma, dbeta, gamma, beta, (int)step, lr);
  if (launched()) return XBAR_EHIP;
  const float* old = reinterpret_cast<const float*>(part);       // parameters before the step: pairs, four floats apart
  const ApplyGrid at(rows, channels, (channels & 3) == 0 ? 4 : 1);
  void (*k)(const float*, const float*, const float*, const float*, int, const float*, const float*, const float*, const float*,
            float*, size_t, int, int, double);
  if ((channels & 3) == 0) {
    if (relu) k = at.four_rows ? bn_apply_bwd_kernel<true, 4, 4> : bn_apply_bwd_kernel<true, 4, 1>;
    else k = at.four_rows ? bn_apply_bwd_kernel<false, 4, 4> : bn_apply_bwd_kernel<false, 4, 1>;
  } else {
    if (relu) k = at.four_rows ? bn_apply_bwd_kernel<true, 1, 4> : bn_apply_bwd_kernel<true, 1, 1>;
    else k = at.four_rows ? bn_apply_bwd_kernel<false, 1, 4> : bn_apply_bwd_kernel<false, 1, 1>;
  }
  hipLaunchKernelGGL(k, at.grid, dim3(256), 0, st, x, dy, step ? old : gamma, step ? old + 1 : beta, step ? 4 : 1, mean, invstd,
                     dgamma, dbeta, dx, rows, channels, at.lanes_log2, 1.0 / (double)rows);
  return launched();
}

int xbar_bn_fwd(const float* x, const float* gamma, const float* beta, float* y, float* mean, float* invstd, size_t rows,
                int channels, float eps, void* ws, size_t ws_bytes, void* hip_stream) {
  return bn_fwd(x, gamma, beta, nullptr, false, y, mean, invstd, rows, channels, eps, ws, ws_bytes,
                reinterpret_cast<hipStream_t>(hip_stream));
}

int xbar_bn_bwd(const float* x, const float* dy, const float* gamma, const float* mean, const float* invstd, float* dx,
                float* dgamma, float* dbeta, size_t rows, int channels, void* ws, size_t ws_bytes, void* hip_stream) {
  return bn_bwd(x, dy, const_cast<float*>(gamma), nullptr, mean, invstd, dx, dgamma, dbeta, rows, channels, false, false, 0.0f, ws,
                ws_bytes, reinterpret_cast<hipStream_t>(hip_stream));
}

int xbar_bn_relu_fwd(const float* x, const float* gamma, const float* beta, const float* skip, float* y, float* mean, float* invstd,
                     size_t rows, int channels, float eps, void* ws, size_t ws_bytes, void* hip_stream) {
  return bn_fwd(x, gamma, beta, skip, true, y, mean, invstd, rows, channels, eps, ws, ws_bytes,
                reinterpret_cast<hipStream_t>(hip_stream));
}

int xbar_bn_bwd_sgd(const float* x, const float* dy, float* gamma, float* beta, const float* mean, const float* invstd, float* dx,
                    float* dgamma, float* dbeta, size_t rows, int channels, int relu, int update, float lr, void* ws, size_t ws_bytes,
                    void* hip_stream) {
  if (!aligned16(beta)) return XBAR_EALIGN;
  if (update && !std::isfinite(lr)) return XBAR_EINVAL;
  return bn_bwd(x, dy, gamma, beta, mean, invstd, dx, dgamma, dbeta, rows, channels, relu != 0, update != 0, lr, ws, ws_bytes,
                reinterpret_cast<hipStream_t>(hip_stream));
}

int xbar_avgpool_fwd(const float* x, float* y, int batch, int positions, int channels, void* hip_stream) {
  if (batch <= 0 || positions <= 0 || channels <= 0) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(y)) return XBAR_EALIGN;
  const size_t outputs = (size_t)batch * channels;
  void (*launch)(const float*, float*, size_t, int, int, hipStream_t) =
      positions < 4 ? launch_avgpool<1, 1> : positions < 8 || outputs >= 131072 ? launch_avgpool<1, 4> : outputs > 16384 ? launch_avgpool<4, 4> : launch_avgpool<16, 4>;
  launch(x, y, outputs, positions, channels, reinterpret_cast<hipStream_t>(hip_stream));
  return launched();
}

int xbar_avgpool_bwd(const float* dy, float* dx, int batch, int positions, int channels, void* hip_stream) {
  if (batch <= 0 || positions <= 0 || channels <= 0) return XBAR_ESHAPE;
  if (!aligned16(dy) || !aligned16(dx)) return XBAR_EALIGN;
  hipLaunchKernelGGL(avgpool_bwd_kernel, dim3(blocks_for((size_t)batch * positions * channels)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), dy, dx, batch, positions, channels);
  return launched();
}

static int pool_geom(const xbar_conv_geom* q, PoolGeom* g) {
  if (!q) return XBAR_EINVAL;
  if (q->batch <= 0 || q->in_h <= 0 || q->in_w <= 0 || q->in_c <= 0 || q->k_h <= 0 || q->k_h != q->k_w || q->stride <= 0 ||
      q->pad < 0 || 2 * q->pad > q->k_h || q->in_h + 2 * q->pad < q->k_h || q->in_w + 2 * q->pad < q->k_w)
    return XBAR_ESHAPE;
  if (q->out_h != (q->in_h + 2 * q->pad - q->k_h) / q->stride + 1 ||
      q->out_w != (q->in_w + 2 * q->pad - q->k_w) / q->stride + 1)
    return XBAR_ESHAPE;
  if ((long long)q->in_h * q->in_w >= (1ll << 31)) return XBAR_ESHAPE;
  g->B = q->batch; g->H = q->in_h; g->W = q->in_w; g->C = q->in_c; g->k = q->k_h; g->stride = q->stride; g->pad = q->pad;
  g->OH = q->out_h; g->OW = q->out_w;
  return XBAR_OK;
}

int xbar_maxpool_fwd(const float* x, float* y, int32_t* argmax, const xbar_conv_geom* geom, void* hip_stream) {
  PoolGeom g;
  const int rc = pool_geom(geom, &g);
  if (rc) return rc;
  if (!aligned16(x) || !aligned16(y) || !aligned16(argmax)) return XBAR_EALIGN;
  const int vec = (g.C & 3) == 0 ? 4 : 1;
  const size_t threads = (size_t)g.B * g.OH * g.OW * (g.C / vec);
  hipLaunchKernelGGL(vec == 4 ? maxpool_fwd_kernel<4> : maxpool_fwd_kernel<1>, dim3(blocks_for(threads)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), x, y, argmax, g, (uint32_t)threads);
  return launched();
}

int xbar_maxpool_bwd(const float* dy, const int32_t* argmax, float* dx, const xbar_conv_geom* geom, void* hip_stream) {
  PoolGeom g;
  const int rc = pool_geom(geom, &g);
  if (rc) return rc;
  if (!aligned16(dy) || !aligned16(dx) || !aligned16(argmax)) return XBAR_EALIGN;
  const int vec = (g.C & 3) == 0 ? 4 : 1;
  const size_t threads = (size_t)g.B * g.H * g.W * (g.C / vec);
  hipLaunchKernelGGL(vec == 4 ? maxpool_bwd_kernel<4> : maxpool_bwd_kernel<1>, dim3(blocks_for(threads)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), dy, argmax, dx, g, (uint32_t)threads);
  return launched();
}

static int shortcut_geom(int batch, int h, int w, int channels, int stride, int out_channels, ShortcutGeom* g) {
  if (batch <= 0 || h <= 0 || w <= 0 || channels <= 0 || stride <= 0 || out_channels < channels) return XBAR_ESHAPE;
  g->B = batch; g->H = h; g->W = w; g->C = channels; g->stride = stride;
  g->OH = (h + stride - 1) / stride; g->OW = (w + stride - 1) / stride; g->OC = out_channels;
  g->lo = (out_channels - channels) / 2;
  return XBAR_OK;
}

int xbar_shortcut_fwd(const float* x, float* y, int batch, int h, int w, int channels, int stride, int out_channels,
                      void* hip_stream) {
  ShortcutGeom g;
  const int rc = shortcut_geom(batch, h, w, channels, stride, out_channels, &g);
  if (rc) return rc;
  if (!aligned16(x) || !aligned16(y)) return XBAR_EALIGN;
  hipLaunchKernelGGL(shortcut_fwd_kernel, dim3(blocks_for((size_t)g.B * g.OH * g.OW * g.OC)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), x, y, g);
  return launched();
}

int xbar_shortcut_bwd(const float* dy, float* dx, int batch, int h, int w, int channels, int stride, int out_channels,
                      void* hip_stream) {
  ShortcutGeom g;
  const int rc = shortcut_geom(batch, h, w, channels, stride, out_channels, &g);
  if (rc) return rc;
  if (!aligned16(dy) || !aligned16(dx)) return XBAR_EALIGN;
  hipLaunchKernelGGL(shortcut_bwd_kernel, dim3(blocks_for((size_t)g.B * g.H * g.W * g.C)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), dy, dx, g);
  return launched();
}

int xbar_absmax(const float* x, size_t n, float* result, void* ws, size_t ws_bytes, void* hip_stream) {
  if (n == 0) return XBAR_ESHAPE;
  if (!aligned16(x) || !aligned16(result) || !aligned16(ws)) return XBAR_EALIGN;
  if (ws_bytes < 1024 * sizeof(uint32_t)) return XBAR_EWORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  const unsigned blocks = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
  uint32_t* part = reinterpret_cast<uint32_t*>(ws);
  hipLaunchKernelGGL(absmax_kernel, dim3(blocks), dim3(256), 0, st, x, n, part);
  if (launched()) return XBAR_EHIP;
  // the partial maxima are bit patterns of non-negative floats: the same kernel reduces them once more
  hipLaunchKernelGGL(absmax_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<const float*>(part), (size_t)blocks,
                     reinterpret_cast<uint32_t*>(result));
  return launched();
}

int xbar_softmax_xent(const float* logits, const int32_t* labels, float* loss, float* dlogits, int batch, int classes,
                      float scale, void* hip_stream) {
  if (batch <= 0 || classes <= 0) return XBAR_ESHAPE;
  if (!aligned16(logits) || !aligned16(labels) || !aligned16(loss) || !aligned16(dlogits)) return XBAR_EALIGN;
  if (!std::isfinite(scale)) return XBAR_EINVAL;
  hipLaunchKernelGGL(softmax_xent_kernel, dim3((unsigned)batch), dim3(64), 0, reinterpret_cast<hipStream_t>(hip_stream),
                     logits, labels, loss, dlogits, classes, scale);
  return launched();
}

}  // extern "C"
