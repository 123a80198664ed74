// Pulse-level weight update with stochastic pulse trains (Sec. IV-C): kernels and xbar_update_pulsed.
#include "xbar_common.h"
#include <type_traits>

using namespace xbar_detail;

namespace {

// Deterministic pulse coding: the bl slots form tx frames of td sub-slots, tx = floor(sqrt(bl)), td = floor(bl / tx).
void coded_frames(int bl, int* tx, int* td) {
  int t = 1;
  while ((t + 1) * (t + 1) <= bl) ++t;
  *tx = t;
  *td = bl / t;
}


// ---------------------------------------------------------------------------------------------
// pulse-level update (Sec. IV-C names the parallel update schemes; this is the one with stochastic
// pulse trains, whose coincidences multiply): every sample drives rows and columns with random
// trains of `bl` slots, a value fires with probability min(1, |value| / range) per slot, and a device
// is pulsed once per slot in which its row and its column both fire, against the sign of x d.
//   train: slot j of element i fires when uniform word j (Philox block 8 i + j / 4, word j % 4,
//          stream 3 for rows, 4 for columns) is below rne(p 2^32); bit 31 carries the value's sign
//   pulse: g += dir dw_min [exp(-v x) up | exp(-v (1 - x)) down, x = (g + 1) / 2]
//               + gamma sqrt(lr dw_min) normal(m 32 + j of stream 5 keyed (step << 31) | device),
//               lr = bl dw_min w_max / (x_range d_range): the aggregate model's noise for one pulse,
//          clamped to [-1, 1]; samples in order, pulses of a sample in order
// ---------------------------------------------------------------------------------------------
struct PulseArgs {
  float* W;
  const float* X;        // [M][K]
  const float* D;        // [M][N]
  uint32_t* rows;        // [mc][K] trains of the current chunk of samples
  uint32_t* cols;        // [mc][N]
  double* state;         // [K][N] g between chunks
  long long* pulses;     // optional [K][N] signed pulse counts
  int M, K, N, bl, m0, mc, first, last;
  uint32_t flags;
  double w_max, x_range, d_range, dw_min, v, sigma;
  uint64_t seed, step;
  const unsigned long long* step_add;   // optional device counter added to step
  ConvGeom conv;                        // convolution layer: X is the NHWC image and row m of the layer's
                                        //   input matrix is gathered from it (CONV variant of the train kernel)
  int coded, tx, td;                    // 1: deterministic time coding, tx frames of td sub-slots; 2: magnitude coding
  unsigned long long* marks;            // two-phase walk: one bit per sample and device, word w of device d at
  size_t mark_device, mark_word;        //   d mark_device + w mark_word: [K N][n_words] for the streamed walk, whose lanes read
                                        //   words of one device; else [n_words][K N], read by lanes of neighbouring devices
  unsigned long long* summary;          //   [ceil(n_words / 64)][K N] one bit per word that is not empty
  int n_words;                          //   64-sample words of the current chunk
  int seg_words;                        //   words per block of the marking pass (a multiple of 4)
  double series[7];                     // streamed walk, v up to 1 / 32: dw_min exp(-v (g + 1) / 2) = sum of series[i] g^i
};

__device__ __forceinline__ uint32_t pulse_train(uint32_t k0, uint32_t k1, uint64_t step, uint64_t index, double p, int bl) {
  const uint64_t threshold = (uint64_t)::rint(clampd(p, 0.0, 1.0) * 4294967296.0);
  const uint32_t last = (uint32_t)(threshold - 1);   // word < threshold as word <= last; threshold 0 is dealt with at the end
  // slot 0 first, four slots at a time: it ends up in the highest of the bits made
  uint32_t bits = 0;
  const int blocks = (bl + 3) >> 2;
  for (int j = 0; j < blocks; ++j) {
    const uint64_t blk = index * 8 + (uint64_t)j;
    uint32_t w[4];
    philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), (uint32_t)step, (uint32_t)(step >> 32), k0, k1, w);
#pragma unroll
    for (int e = 0; e < 4; ++e) bits = bits + bits + (w[e] <= last ? 1u : 0u);
  }
  bits = __builtin_bitreverse32(bits) >> (32 - 4 * blocks);   // slot j at bit j
  return threshold ? bits & ((1u << bl) - 1u) : 0u;
}

// Deterministic code of a value: slot = frame * td + sub-slot; a row takes the first rne(p tx) frames
// whole, a column the first rne(p td) sub-slots of every frame.
__device__ __forceinline__ uint32_t pulse_code(double p, int tx, int td, bool is_col) {
  const int level = (int)::rint(clampd(p, 0.0, 1.0) * (double)(is_col ? td : tx));
  if (!is_col) return level * td >= 32 ? 0xFFFFFFFFu : (1u << (level * td)) - 1u;      // level * td <= 31 slots
  const uint32_t frame = (1u << level) - 1u;                                          // level <= td <= 31
  uint32_t bits = 0;
  for (int f = 0; f < tx; ++f) bits |= frame << (f * td);
  return bits;
}

// Magnitude coding: ONE pulse per sample whose height is the level rne(p bl) of bl; bit 30 marks a pulse that
// is there at all, so that "row and column share a set bit" still means "this device is written".
__device__ __forceinline__ uint32_t pulse_height(double p, int bl) {
  const uint32_t level = (uint32_t)::rint(clampd(p, 0.0, 1.0) * (double)bl);
  return level ? (level | 0x40000000u) : 0u;
}

// One thread per element of the chunk's inputs, then of its errors.
template <bool CONV>
__global__ __launch_bounds__(256) void pulse_trains_kernel(PulseArgs a) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long n_rows = (long long)a.mc * a.K, n_cols = (long long)a.mc * a.N;
  if (t < n_rows) {
    const uint64_t index = (uint64_t)a.m0 * a.K + (uint64_t)t;               // m K + k
    double x;
    if constexpr (CONV) {        // element (m, k) of the patch matrix: k = (kh KW + kw) C + c
      const int sample = n_rows < (1ll << 32) ? (int)((uint32_t)t / (uint32_t)a.K) : (int)(t / a.K);   // the short division
      const uint32_t k = (uint32_t)(t - (long long)sample * a.K), kk = k / (uint32_t)a.conv.C, kh = kk / (uint32_t)a.conv.KW;
      x = (double)conv_fetch(a.X, a.conv, conv_row(a.conv, a.m0 + sample), (int)kh, (int)(kk - kh * (uint32_t)a.conv.KW),
                             (int)(k - kk * (uint32_t)a.conv.C));
    } else {
      x = (double)a.X[index];
    }
    const uint32_t k0 = (uint32_t)a.seed ^ (0x9E3779B9u * kStreamPulseRows);
    const uint32_t k1 = (uint32_t)(a.seed >> 32) ^ (0xBB67AE85u * kStreamPulseRows);
    const uint32_t train = a.coded == 2 ? pulse_height(::fabs(x) / a.x_range, a.bl)
                           : a.coded  ? pulse_code(::fabs(x) / a.x_range, a.tx, a.td, false)
                                      : pulse_train(k0, k1, effective_step(a.step, a.step_add), index, ::fabs(x) / a.x_range, a.bl);
    a.rows[t] = train | (x < 0.0 ? 0x80000000u : 0u);
  } else if (t < n_rows + n_cols) {
    const long long u = t - n_rows;
    const uint64_t index = (uint64_t)a.m0 * a.N + (uint64_t)u;
    const double d = (double)a.D[index];
    const uint32_t k0 = (uint32_t)a.seed ^ (0x9E3779B9u * kStreamPulseCols);
    const uint32_t k1 = (uint32_t)(a.seed >> 32) ^ (0xBB67AE85u * kStreamPulseCols);
    const uint32_t train = a.coded == 2 ? pulse_height(::fabs(d) / a.d_range, a.bl)
                           : a.coded  ? pulse_code(::fabs(d) / a.d_range, a.tx, a.td, true)
                                      : pulse_train(k0, k1, effective_step(a.step, a.step_add), index, ::fabs(d) / a.d_range, a.bl);
    a.cols[u] = train | (d < 0.0 ? 0x80000000u : 0u);
  }
}

// One pulse of device `dev` (ordinal `ord` within sample m), upwards when `up`.  The device model is
// chosen at compile time, and the step of the noise stream is read before the walk: nothing that is the
// same for all lanes is tested (and no pointer that may be null is followed) inside the per-lane walk.
// `units`: quanta of dw_min that this one write carries (1 for a pulse of a train; the product of the two pulse
// heights with magnitude coding, where the non-linearity and the noise belong to the write as a whole).
template <bool NL, bool NOISE, bool MAG = false>
__device__ __forceinline__ double one_pulse(const PulseArgs& a, double g, bool up, int m, int ord, uint64_t dev,
                                            uint64_t step, int units = 1) {
#pragma clang fp contract(off)   // every product and sum rounds on its own
  double move = MAG ? a.dw_min * (double)units : a.dw_min;
  if constexpr (NL) {
    const double x = clampd(0.5 * (g + 1.0), 0.0, 1.0);
    move *= up ? ::exp(-a.v * x) : ::exp(-a.v * (1.0 - x));
  }
  double next = g + (up ? 1.0 : -1.0) * move;
  if constexpr (NOISE) {
    NormalStream rng(a.seed, kStreamPulseNoise, (step << 31) | dev);
    if constexpr (MAG) next += a.sigma * ::sqrt((double)units) * rng.get((uint64_t)m * 32 + (uint64_t)ord);
    else next += a.sigma * rng.get((uint64_t)m * 32 + (uint64_t)ord);
  }
  return clampd(next, -1.0, 1.0);
}

// Block = (16 P) x (16 P) devices, thread = P x P of them with their states in registers; the trains
// of a stage of samples go through LDS, transposed ([row or column][sample]) so that a lane reads
// the trains of consecutive samples of its row and of its column with 16-byte loads.
// A device's pulses are sequential, but devices do not wait for each other sample by sample: all
// lanes first mark, in step, the samples of the stage in which their row and column share a slot (one
// bit per sample and device), then every lane works through its own marked samples one pulse per turn,
// so a wave runs for as long as its busiest device has pulses in the stage, not for the sum over the
// samples of the busiest device of each.
// MARKED: the marks come from pulse_mark_kernel (layers with few devices: that pass fills the chip, this
// one cannot) instead of being worked out here, stage by stage.
template <int P, bool NL, bool NOISE, bool MARKED = false, bool MAG = false>
__global__ __launch_bounds__(256) void pulse_apply_kernel(PulseArgs a) {
  constexpr int TE = 16 * P;              // tile edge
  constexpr int ST = 4096 / TE;           // samples per stage (a multiple of 16)
  constexpr int LD = ST + 4;              // words per row or column: 16-byte aligned, spread over the banks
  __shared__ __align__(16) uint32_t rt[TE * LD];
  __shared__ __align__(16) uint32_t ct[TE * LD];
  const int nb = (a.N + TE - 1) / TE;
  const int kt = (blockIdx.x / nb) * TE, nt = (blockIdx.x % nb) * TE;
  const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
  const int k0 = kt + P * ty, n0 = nt + P * tx;
  const uint64_t step = effective_step(a.step, a.step_add);
  double g[P][P];
  int cnt[P][P];
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int k = k0 + i, n = n0 + j;
      cnt[i][j] = 0;
      g[i][j] = 0.0;
      if (k < a.K && n < a.N)
        g[i][j] = a.first ? (double)a.W[(size_t)k * a.N + n] / a.w_max : a.state[(size_t)k * a.N + n];
    }
  for (int s0 = 0; s0 < a.mc; s0 += ST) {
    const int ns = min(ST, a.mc - s0);
    const int ns16 = (ns + 15) & ~15;      // whole groups of 16 (ST is a multiple): samples past the end hold no train
    // the stage's trains: all loads of a thread are issued before the first one is needed
    constexpr int PER = ST * TE / 256;     // 16 elements of either matrix per thread
    uint32_t rv[PER], cv[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = threadIdx.x + 256 * u, sm = e / TE, c = e % TE;
      const bool live = sm < ns;
      rv[u] = (live && kt + c < a.K) ? a.rows[(size_t)(s0 + sm) * a.K + kt + c] : 0u;
      cv[u] = (live && nt + c < a.N) ? a.cols[(size_t)(s0 + sm) * a.N + nt + c] : 0u;
    }
    __syncthreads();                       // everyone is done with the previous stage
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = threadIdx.x + 256 * u, sm = e / TE, c = e % TE;
      rt[c * LD + sm] = rv[u];
      ct[c * LD + sm] = cv[u];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const uint64_t dev = (uint64_t)(k0 + i) * a.N + (uint64_t)(n0 + j);
        const uint32_t* rp = &rt[(P * ty + i) * LD];
        const uint32_t* cp = &ct[(P * tx + j) * LD];
        double gs = g[i][j];
        int moved = 0;
        // all lanes together: which samples of the stage have a slot in which row and column both fire
        constexpr int NW = ST / 64;
        uint64_t live[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          live[w] = 0;
          if constexpr (MARKED) {
            const int word = s0 / 64 + w;
            if (word < a.n_words && k0 + i < a.K && n0 + j < a.N) live[w] = a.marks[(size_t)dev * a.mark_device + (size_t)word * a.mark_word];
            continue;
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int at = 64 * w + 4 * v;
            if (at < ns16) {
              const u32x4 r = *reinterpret_cast<const u32x4*>(rp + at);
              const u32x4 c = *reinterpret_cast<const u32x4*>(cp + at);
              const uint32_t four = (min(r.x & c.x & 0x7FFFFFFFu, 1u)) | (min(r.y & c.y & 0x7FFFFFFFu, 1u) << 1) |
                                    (min(r.z & c.z & 0x7FFFFFFFu, 1u) << 2) | (min(r.w & c.w & 0x7FFFFFFFu, 1u) << 3);
              live[w] |= (uint64_t)four << (4 * v);
            }
          }
        }
        // every lane for itself, one pulse per turn: its marked samples in order, the pulses of a
        // sample in order
        uint32_t q = 0;
        bool up = false;
        int m = 0, ord = 0, units = 1;
        for (;;) {
          if (q == 0) {
            int w = -1;
            uint64_t word = 0;
#pragma unroll
            for (int t = NW - 1; t >= 0; --t)
              if (live[t]) {
                w = t;
                word = live[t];
              }
            if (w < 0) break;                          // the stage is done for this device
            const int e = __builtin_ctzll(word);
#pragma unroll
            for (int t = 0; t < NW; ++t)
              if (t == w) live[t] = word & (word - 1);
            const int at = 64 * w + e;
            const uint32_t rw = rp[at], cw = cp[at];
            q = rw & cw & 0x7FFFFFFFu;
            if constexpr (MAG) {                        // one write of (row height) x (column height) quanta
              units = (int)(rw & 31u) * (int)(cw & 31u);
              q = 1u;
            }
            up = ((rw ^ cw) >> 31) != 0;               // against the sign of x d
            m = a.m0 + s0 + at;
            ord = 0;
          }
          q &= q - 1;
          gs = one_pulse<NL, NOISE, MAG>(a, gs, up, m, ord, dev, step, units);
          ++ord;
          moved += up ? units : -units;
        }
        g[i][j] = gs;
        cnt[i][j] += moved;
      }
  }
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int k = k0 + i, n = n0 + j;
      if (k < a.K && n < a.N) {
        const size_t at = (size_t)k * a.N + n;
        if (a.last) a.W[at] = (float)(a.w_max * g[i][j]);
        else a.state[at] = g[i][j];
        if (a.pulses) a.pulses[at] = (a.first ? 0 : a.pulses[at]) + cnt[i][j];
      }
    }
}

// Two-phase walk for layers with few devices and many samples (convolution layers: a 144 x 16 layer has
// 9 blocks of devices and 131072 samples).  Phase 1, one block per 16 x 16 devices and segment of samples
// (256 at a time), fills the chip: it marks the samples in which a device's row and column share a slot,
// one bit per sample and device, plus, for the plain walk, one summary bit per 64-sample word that is not
// empty.  Phase 2 walks only the marked samples, in order: pulse_stream_kernel where the layer has few
// devices, else one thread per device (summary -> word -> sample), fetching their two trains from memory:
// the sequential part shrinks to the pulses.
__global__ __launch_bounds__(256) void pulse_mark_kernel(PulseArgs a) {
  constexpr int TE = 16, ST = 256, LD = ST + 4, PER = ST * TE / 256, NW = ST / 64;
  __shared__ __align__(16) uint32_t rt[TE * LD];
  __shared__ __align__(16) uint32_t ct[TE * LD];
  const int nb = (a.N + TE - 1) / TE, tiles = ((a.K + TE - 1) / TE) * nb;
  const int tile = blockIdx.x % tiles, seg = blockIdx.x / tiles, seg_samples = 64 * a.seg_words;
  const int kt = (tile / nb) * TE, nt = (tile % nb) * TE;
  const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
  const int k = kt + ty, n = nt + tx;
  const bool valid = k < a.K && n < a.N;
  const uint32_t* rp = &rt[ty * LD];
  const uint32_t* cp = &ct[tx * LD];
  const size_t kn = (size_t)a.K * a.N, dev = (size_t)k * a.N + n;
  unsigned long long summary = 0;                  // bit = word of the segment that has a marked sample
  for (int s0 = seg * seg_samples; s0 < min(a.mc, (seg + 1) * seg_samples); s0 += ST) {
    const int ns = min(ST, a.mc - s0);
    __syncthreads();                               // everyone is done with the previous stage
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = threadIdx.x + 256 * u, sm = e / TE, c = e % TE;
      const bool live = sm < ns;
      rt[c * LD + sm] = (live && kt + c < a.K) ? a.rows[(size_t)(s0 + sm) * a.K + kt + c] : 0u;
      ct[c * LD + sm] = (live && nt + c < a.N) ? a.cols[(size_t)(s0 + sm) * a.N + nt + c] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int word = s0 / 64 + w;
      unsigned long long bits = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int at = 64 * w + 4 * v;
        const u32x4 r = *reinterpret_cast<const u32x4*>(rp + at);
        const u32x4 c = *reinterpret_cast<const u32x4*>(cp + at);
        const uint32_t four = (min(r.x & c.x & 0x7FFFFFFFu, 1u)) | (min(r.y & c.y & 0x7FFFFFFFu, 1u) << 1) |
                              (min(r.z & c.z & 0x7FFFFFFFu, 1u) << 2) | (min(r.w & c.w & 0x7FFFFFFFu, 1u) << 3);
        bits |= (unsigned long long)four << (4 * v);
      }
      if (valid && word < a.n_words) {
        a.marks[dev * a.mark_device + (size_t)word * a.mark_word] = bits;
        if (bits) summary |= 1ull << ((word - a.seg_words * seg) & 63);
      }
    }
  }
  if (valid && a.seg_words == 64) a.summary[(size_t)seg * kn + dev] = summary;   // one word of it per segment (the plain walk's)
}

template <bool NL, bool NOISE>
__global__ __launch_bounds__(256) void pulse_walk_kernel(PulseArgs a) {
  const size_t kn = (size_t)a.K * a.N;
  const size_t dev = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (dev >= kn) return;
  const int k = (int)(dev / a.N), n = (int)(dev % a.N);
  const uint64_t step = effective_step(a.step, a.step_add);
  const int n_seg = (a.n_words + 63) / 64;
  double gs = a.first ? (double)a.W[dev] / a.w_max : a.state[dev];
  int moved = 0, next_seg = 0, word_base = 0, seg_base = 0, m = 0, ord = 0;
  unsigned long long word = 0, summary = 0;
  uint32_t q = 0;
  bool up = false;
  // every lane for itself, one pulse per turn (as in pulse_apply_kernel)
  for (;;) {
    if (q == 0) {
      if (word == 0) {                               // next word with a marked sample, by way of the summaries
        while (summary == 0 && next_seg < n_seg) {
          summary = a.summary[(size_t)next_seg * kn + dev];
          seg_base = 64 * next_seg;
          ++next_seg;
        }
        if (summary == 0) break;                     // no marked sample left
        const int wi = seg_base + __builtin_ctzll(summary);
        summary &= summary - 1;
        word = a.marks[dev * a.mark_device + (size_t)wi * a.mark_word];        // not empty: its summary bit is set
        word_base = 64 * wi;
      }
      const int at = word_base + __builtin_ctzll(word);
      word &= word - 1;
      const uint32_t rw = a.rows[(size_t)at * a.K + k], cw = a.cols[(size_t)at * a.N + n];
      q = rw & cw & 0x7FFFFFFFu;                     // not empty: the sample is marked
      up = ((rw ^ cw) >> 31) != 0;
      m = a.m0 + at;
      ord = 0;
    }
    q &= q - 1;
    gs = one_pulse<NL, NOISE>(a, gs, up, m, ord, (uint64_t)dev, step);
    ++ord;
    moved += up ? 1 : -1;
  }
  if (a.last) a.W[dev] = (float)(a.w_max * gs);
  else a.state[dev] = gs;
  if (a.pulses) a.pulses[dev] = (a.first ? 0 : a.pulses[dev]) + moved;
}

// The streamed walk: a block has one wave that walks and, for each of its devices, one that feeds it.  Only the moves of a
// device are sequential; which samples it is pulsed in, the trains and the normal numbers of its pulses are not.  A feeding
// wave lists its device's marked samples (ring in LDS), fetches the trains of 64 of them side by side, lists their pulses (a
// second ring) and makes a batch of moves of them; the walking wave, a lane per device, takes the batch before while the next
// is made.  One barrier per batch of every device hands them over.  Without marks (MARKED false: too few samples for a marking pass
// to pay) a feeding wave takes the trains of 256 samples at a time, marked or not.
// What bounds it: few devices, the instructions of the walking wave, each of which takes it 8 to 10 cycles (so its moves are
// read two groups at a time, without copies, in a scalar loop where all devices are full); many, with noise the normal numbers (some
// 300 instructions per 64 pulses), without it the lists.  64 registers, for two blocks to a compute unit.
// ms of a whole update, series, trains of 12 pulses a sample / of one in 30 samples, against one to four devices per wave that all its
// lanes walk (or above 20480 devices, 40960 with noise, a lane per device that does everything by itself): 144 x 16 devices, 32768
// samples 51.0 -> 20.4 / 2.97 -> 1.43, with noise 60.6 -> 30.8 / 3.46 -> 2.10; 27 x 16 x 32768 22.9 -> 18.0 / 1.49 -> 0.98; 128 x 128 x 4096 14.1 ->
// 10.2 / 1.06 -> 0.88; 576 x 64 x 4096 24.3 -> 14.8 / 1.76 -> 1.37, with noise 45.7 -> 41.2 / 3.04 -> 2.65.  A pulse handed over as a double
// and a noise also without noise, out of rings of 256: 576 x 64, linear 22.6 / 1.17, now 7.1 / 0.95.
// NL: 0 linear device; 1 write non-linearity by its power series about mid-range (v <= 1/32: six powers leave less than 1e-18
// of exp(-v y) on 0 <= y <= 1); 2 by exp().
// With the series an upward pulse moves the state g by dw_min exp(-v (1 + g) / 2), a downward one back by dw_min exp(-v (1 - g) / 2),
// that is by direction times the even powers of g plus the odd ones as they are.  A move is complete, noise included, before it
// joins the state, which is rounded once per pulse: 2.4e-16 rms after 200 pulses against 113-bit arithmetic (noise joining the state
// by itself: 3.5e-16; a state held on 0 .. 1, which the last operation could clamp by itself: 1.2e-15).
constexpr int kStreamMaxDevices = 15;                // per block: 16 waves
constexpr int kSampleRing = 256;                     // marked samples of a device: up to 127 wait, and a word of 64 fits beside them
                                                     //   (what does not fit is fetched again)
// What a feeding wave hands over.  With noise 64 moves, each a noise and a direction, out of a ring of pulses: up to 127 wait, and those
// of 64 samples with 14 each fit beside them, so that the 31 turns of the list that makes them are shared by as many (the rest
// is fetched again).  Without noise a pulse is its direction: 128 of them out of a ring of bits (1 downwards), which always has room
// for 64 samples beside the 255 pulses that wait; a sample sets all of its bits at once, and its device's wave spreads them, so
// that the walking wave has a load for two moves and nothing else but the moves.
template <bool NOISE>
struct Stream {
  using Move = std::conditional_t<NOISE, double2, double>;       // noise and direction, or the direction
  static constexpr int kBatch = NOISE ? 64 : 128;
  static constexpr int kGroup = NOISE ? 4 : 8;                   // moves that the walking wave reads together
  static constexpr int kStride = kBatch + (NOISE ? 1 : 2);       // spreads the devices over the banks
  static constexpr int kRoom = NOISE ? 1024 : 4096;              // pulses that the ring holds
  static constexpr int kRingWords = NOISE ? kRoom : kRoom / 32;
  static constexpr size_t lds_bytes(int devices) {
    return (size_t)devices * (2 * kStride * sizeof(Move) + (kSampleRing + kRingWords) * sizeof(uint32_t)) + 2 * 16 * sizeof(int) + 2 * sizeof(int);
  }
};

// Inclusive sum over the lanes of a wave: DPP row shifts by 1, 2, 4 and 8, then the last lane of a row or half to the rows behind.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

template <int NL, bool NOISE, bool MARKED>
__global__ __launch_bounds__(1024, 8) void pulse_stream_kernel(PulseArgs a, int devices) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) char stream_lds[];
  using S = Stream<NOISE>;
  // a direction: dw_min of a linear device, 1 with the series, a half with exp(), or less than 0 by as much
  using Move = typename S::Move;
  Move* moves = reinterpret_cast<Move*>(stream_lds);            // [2][devices][kStride]
  uint32_t* rings = reinterpret_cast<uint32_t*>(moves + 2 * devices * S::kStride);     // [devices][samples, then pulses]
  int* runs = reinterpret_cast<int*>(rings + devices * (kSampleRing + S::kRingWords)); // [2][16] moves of a device in a batch
  int* alive = runs + 2 * 16;                                   // [2] batch number + 1 where a device had moves in it
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const size_t kn = (size_t)a.K * a.N, dev0 = (size_t)blockIdx.x * devices;
  if (threadIdx.x < 2) alive[threadIdx.x] = 0;
  __syncthreads();

  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);                   // the chain: what feeds it has time
    const bool valid = lane < devices && dev0 + lane < kn;
    const size_t dev = valid ? dev0 + lane : kn - 1;
    auto begin = [&]() __attribute__((always_inline)) { return a.first ? (double)a.W[dev] / a.w_max : a.state[dev]; };
    double g = begin();
    double gx = clampd(g, -1.0, 1.0);                // where the non-linearity finds the state
    bool pulsed = false;
    const double up_down = 2.0 * a.dw_min;
    auto move = [&](const Move b) __attribute__((always_inline)) {      // the state after it
      double next, direction, noise = 0.0;
      if constexpr (NOISE) direction = b.y, noise = b.x;
      else direction = b;
      if constexpr (NL == 1) {
        const double z = gx * gx, zz = z * z;
        const double odd = __builtin_fma(zz, a.series[5], __builtin_fma(z, a.series[3], a.series[1]));
        const double even = __builtin_fma(zz, __builtin_fma(z, a.series[6], a.series[4]), __builtin_fma(z, a.series[2], a.series[0]));
        const double directed = NOISE ? __builtin_fma(direction, even, noise) : direction * even;
        next = g + __builtin_fma(gx, odd, directed);
      } else {
        if constexpr (NL == 0) next = g + direction;
        else next = g + direction * up_down * ::exp(-a.v * __builtin_fma(direction, gx, 0.5));   // x upwards, 1 - x downwards
        if constexpr (NOISE) next += noise;
      }
      return ::fmin(::fmax(next, -1.0), 1.0);
    };
    for (int batch = 0;; ++batch) {
      if (batch > 0) {                               // the moves before, while the next ones are made
        const int run = valid ? runs[((batch - 1) & 1) * 16 + lane] : 0;
        pulsed = pulsed || run > 0;
        const Move* mv = moves + (((batch - 1) & 1) * devices + min(lane, devices - 1)) * S::kStride;
        // Two groups of moves in registers, one read under the moves of the other
        constexpr int G = S::kGroup;
        Move one[G], other[G];
        auto load = [&](Move (&group)[G], int t) __attribute__((always_inline)) {
          const int from = min(t, S::kBatch - G);
#pragma unroll
          for (int i = 0; i < G; ++i) group[i] = mv[from + i];
          __builtin_amdgcn_sched_barrier(0);         // here, not where the first of them is needed
        };
        load(one, 0);
        auto two_groups = [&](int t0) __attribute__((always_inline)) {
          load(other, t0 + G);
#pragma unroll
          for (int t = 0; t < G; ++t) g = gx = move(one[t]);
          load(one, t0 + 2 * G);
#pragma unroll
          for (int t = 0; t < G; ++t) g = gx = move(other[t]);
        };
        int t0 = 0;
        if (__all(!valid || run == S::kBatch)) {     // a scalar loop: a move of 50 cycles is 5 shorter
#pragma unroll 1
          for (int t = 0; t < S::kBatch; t += 2 * G) two_groups(t);
          t0 = S::kBatch;
        } else {
#pragma unroll 1
          for (; t0 + 2 * G <= run; t0 += 2 * G) two_groups(t0);         // lanes that have run out wait
        }
        if (__any(t0 < run)) {                       // a device without a pulse keeps its state, also beyond the range
          load(other, t0 + G);
#pragma unroll
          for (int t = 0; t < 2 * G - 1; ++t) {
            const double next = move(t < G ? one[t] : other[t - G]);
            if (t0 + t < run) g = gx = next;
          }
        }
      }
      __syncthreads();
      if (alive[batch & 1] != batch + 1) break;      // no device had moves in this batch: none has any left
    }
    // The moves' minimum and maximum drop a NaN, which a clamp by comparison keeps; a step is finite, so the state is NaN
    // at the end only if it began as one.  A device without a pulse keeps what it held to the bit (a moved -0 is +0).
    // Read again rather than held in registers through the walk.
    const double g_begin = begin();
    if (!pulsed || g_begin != g_begin) g = g_begin;
    if (valid) {
      if (a.last) a.W[dev] = (float)(a.w_max * g);
      else a.state[dev] = g;
    }
    return;
  }

  const int slot = wave - 1;
  const bool valid = dev0 + slot < kn;
  const size_t dev = valid ? dev0 + slot : kn - 1;
  const int k = (int)(dev / a.N), n = (int)(dev % a.N);
  NormalStream rng(a.seed, kStreamPulseNoise, (effective_step(a.step, a.step_add) << 31) | dev);
  uint32_t* sq = rings + slot * (kSampleRing + S::kRingWords);   // marked samples
  uint32_t* pq = sq + kSampleRing;                   // pulses: sample << 6 | ordinal << 1 | upwards; without noise a bit each
  if constexpr (!NOISE) {
    for (int i = lane; i < S::kRingWords; i += 64) pq[i] = 0;
    wave_exchange();
  }
  const double unit = NL == 0 ? a.dw_min : NL == 1 ? 1.0 : 0.5;
  int n_s = 0, s_head = 0, n_p = 0, p_head = 0, moved = 0;   // entries waiting, and where they begin
  // Marked: the next word of marks, this lane's word and its sample; else the next sample and four of this lane
  constexpr int U = MARKED ? 1 : 4;
  const unsigned long long* marks = MARKED ? a.marks + dev * a.n_words : nullptr;
  const int n_next = !valid ? 0 : MARKED ? a.n_words : a.mc;
  int next = 0;
  uint32_t at[U], q[U], up[U];                       // number, shared slots, direction
  unsigned long long word = 0;

  auto trains = [&](int u) __attribute__((always_inline)) {
    const uint32_t rw = a.rows[(size_t)at[u] * a.K + k], cw = a.cols[(size_t)at[u] * a.N + n];
    q[u] = rw & cw & 0x7FFFFFFFu;
    up[u] = (rw ^ cw) >> 31;                         // against the sign of x d
  };
  auto left = [&]() __attribute__((always_inline)) { return n_s > 0 || next < n_next; };
  // Trains of up to 64 marked samples, and the next 64 words where they may be needed; or of the next 256 samples.
  auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      q[u] = 0;
      if constexpr (MARKED) {
        if (lane < n_s) {
          at[u] = sq[(s_head + lane) & (kSampleRing - 1)];
          trains(u);
        }
      } else {
        at[u] = (uint32_t)(next + 64 * u + lane);
        if ((int)at[u] < n_next) trains(u);
      }
    }
    if constexpr (MARKED) word = (n_s < 128 && next + lane < n_next) ? marks[next + lane] : 0ull;
  };
  // The pulses of 64 samples into their ring, as many samples as there is room for; returns how many.
  auto append_pulses = [&](int u, bool there) __attribute__((always_inline)) {
    const int c = __popc(q[u]), inc = wave_scan(c);
    const bool fits = there && n_p + inc <= S::kRoom;
    const int taken = __popcll(__ballot(fits));      // the first lanes: inc does not fall with the lane
    uint32_t pos = (uint32_t)(p_head + n_p + inc - c);
    if constexpr (NOISE) {
      uint32_t bits = fits ? q[u] : 0u;
      for (uint32_t ord = 0; __any(bits != 0); ++ord)
        if (bits) {
          pq[pos++ & (S::kRoom - 1)] = (at[u] << 6) | (ord << 1) | up[u];
          bits &= bits - 1;
        }
    } else if (fits) {
      moved += up[u] ? c : -c;
      if (c > 0 && !up[u]) {
        const uint64_t ones = ((1ull << c) - 1) << (pos & 31);
        atomicOr(&pq[(pos >> 5) & (S::kRingWords - 1)], (uint32_t)ones);
        if (ones >> 32) atomicOr(&pq[((pos >> 5) + 1) & (S::kRingWords - 1)], (uint32_t)(ones >> 32));
      }
    }
    if (taken > 0) n_p += __builtin_amdgcn_readlane(inc, taken - 1);
    return taken;
  };
  auto append = [&]() __attribute__((always_inline)) {
    if constexpr (MARKED) {
      const bool more_words = n_s < 128 && next < n_next;
      if (n_s > 0) {
        const int taken = append_pulses(0, lane < n_s);
        n_s -= taken;
        s_head += taken;
      }
      if (more_words) {
        const int c = __popcll(word), inc = wave_scan(c);
        const bool fits = n_s + inc <= kSampleRing;
        const int taken = __popcll(__ballot(fits));
        unsigned long long bits = fits ? word : 0ull;
        uint32_t pos = (uint32_t)(s_head + n_s + inc - c);
        const uint32_t base = (uint32_t)(next + lane) * 64u;
        while (__any(bits != 0))
          if (bits) {
            sq[pos++ & (kSampleRing - 1)] = base + (uint32_t)__builtin_ctzll(bits);
            bits &= bits - 1;
          }
        if (taken > 0) n_s += __builtin_amdgcn_readlane(inc, taken - 1);
        next += taken;
      }
    } else {
      int taken = 64;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (taken == 64) {                           // else the rest is fetched again
          taken = append_pulses(u, true);
          next += taken;
        }
    }
    wave_exchange();
  };
  // With fewer pulses waiting than a batch has there is room for a sample's (at most 31); where no marked sample waits, for a
  // word's: every turn of this loop takes one of them.
  auto fill = [&]() __attribute__((always_inline)) {
    while (n_p < S::kBatch && left()) {
      fetch();
      append();
    }
  };
  bool ahead = false;
  for (int batch = 0;; ++batch) {
    if (ahead) append();
    fill();
    // the loads of the batch after this one are on their way under the normal numbers
    ahead = n_p < 2 * S::kBatch && left();
    if (ahead) fetch();
    const int run = min(n_p, S::kBatch);
    Move* mine = moves + ((batch & 1) * devices + slot) * S::kStride;
    if constexpr (NOISE) {
      double2 e = {0.0, 0.0};
      if (lane < run) {
        const uint32_t p = pq[(p_head + lane) & (S::kRoom - 1)];
        const bool upwards = (p & 1u) != 0;
        e.y = upwards ? unit : -unit;
        moved += upwards ? 1 : -1;
        e.x = a.sigma * rng.get((uint64_t)(a.m0 + (int)(p >> 6)) * 32 + ((p >> 1) & 31u));
      }
      mine[lane] = e;
    } else {                                         // whole words of bits: only a device's last batch is not full
      const uint32_t down = pq[((p_head >> 5) + (lane >> 4)) & (S::kRingWords - 1)] >> (2 * (lane & 15));
      reinterpret_cast<double2*>(mine)[lane] = double2{down & 1u ? -unit : unit, down & 2u ? -unit : unit};
      wave_exchange();
      if (lane < S::kBatch / 32) pq[((p_head >> 5) + lane) & (S::kRingWords - 1)] = 0;
    }
    if (lane == 0) {
      runs[(batch & 1) * 16 + slot] = run;
      if (run > 0) alive[batch & 1] = batch + 1;
    }
    n_p -= run;
    p_head += run;
    __syncthreads();
    if (alive[batch & 1] != batch + 1) break;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) moved += __shfl_xor(moved, d, 64);
  if (a.pulses && valid && lane == 0) a.pulses[dev] = (a.first ? 0 : a.pulses[dev]) + moved;
}

int move_mode(const PulseArgs& a, bool nl) { return !nl ? 0 : a.v <= 1.0 / 32.0 ? 1 : 2; }   // NL of pulse_stream_kernel

template <bool MARKED>
hipError_t launch_pulse_stream(const PulseArgs& a, bool nl, bool noise, hipStream_t st) {
  const int mode = move_mode(a, nl);
  void (*k)(PulseArgs, int);
  if (noise) k = mode == 0 ? pulse_stream_kernel<0, true, MARKED> : mode == 1 ? pulse_stream_kernel<1, true, MARKED> : pulse_stream_kernel<2, true, MARKED>;
  else k = mode == 0 ? pulse_stream_kernel<0, false, MARKED> : mode == 1 ? pulse_stream_kernel<1, false, MARKED> : pulse_stream_kernel<2, false, MARKED>;
  // a block per compute unit at a time, the devices spread evenly over the rounds that takes
  const long long kn = (long long)a.K * a.N, per_round = 256 * kStreamMaxDevices, rounds = (kn + per_round - 1) / per_round;
  const int devices = (int)((kn + 256 * rounds - 1) / (256 * rounds));
  const size_t lds = noise ? Stream<true>::lds_bytes(devices) : Stream<false>::lds_bytes(devices);
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)((kn + devices - 1) / devices)), dim3(64 * (devices + 1)), lds, st, a, devices);
  return hipGetLastError();
}

constexpr int kTwoPhaseBlocks = 4096;

struct PulsePlan {
  int mc;                       // samples per chunk (the trains of one chunk are resident at a time)
  size_t rows_bytes, cols_bytes, ws_bytes;
  int two_phase;                // mark, then walk the marked samples (few devices, many samples)
  size_t marks_bytes;
};

PulsePlan plan_pulsed(int M, int K, int N) {
  PulsePlan p;
  const long long per_sample = 4ll * ((long long)K + N);
  long long mc = std::max(64ll, ((64ll << 20) / per_sample) / 64 * 64);
  // mark-then-walk where one device per thread does not already come in thousands of blocks and there are
  // enough samples for the marking pass to pay; its marks (one bit per sample and device) stay within 256 MiB
  const long long kn = (long long)K * N;
  const long long mark_samples = ((8ll << 28) / kn) / 4096 * 4096;
  p.two_phase = (long long)cdiv(K, 16) * cdiv(N, 16) < kTwoPhaseBlocks && M >= 2048 && mark_samples >= 4096;
  if (p.two_phase) mc = std::min(mc, mark_samples);
  p.mc = (int)std::min<long long>(mc, M);
  p.rows_bytes = align256((size_t)4 * p.mc * K);
  p.cols_bytes = align256((size_t)4 * p.mc * N);
  p.ws_bytes = p.rows_bytes + p.cols_bytes + align256((size_t)8 * K * N);
  p.marks_bytes = 0;
  if (p.two_phase) {
    p.marks_bytes = align256((size_t)cdiv(p.mc, 64) * 8 * (size_t)K * N) + align256((size_t)cdiv(p.mc, 4096) * 8 * (size_t)K * N);
    p.ws_bytes += p.marks_bytes;
  }
  return p;
}

}  // namespace

namespace xbar_detail {
size_t pulsed_workspace_bytes(int M, int K, int N) { return plan_pulsed(M, K, N).ws_bytes; }
}  // namespace xbar_detail

namespace {
int run_update_pulsed(const xbar_config* cfg, float* W, const float* X, const float* dY, int M, int K, int N, float w_max,
                      float x_range, float d_range, int bl, float dw_min, uint64_t step, long long* pulses, void* ws,
                      size_t ws_bytes, void* hip_stream, const ConvGeom* conv) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(M, K, N))) return rc;
  if (!aligned16(W) || !aligned16(X) || !aligned16(dY) || !aligned16(ws)) return XBAR_EALIGN;
  if (pulses && (reinterpret_cast<uintptr_t>(pulses) & 7u)) return XBAR_EALIGN;
  if (!finite_pos(w_max) || !finite_pos(x_range) || !finite_pos(d_range) || !finite_pos(dw_min)) return XBAR_EINVAL;
  if (bl < 1 || bl > 31 || step >= (1ull << 33)) return XBAR_EINVAL;
  const PulsePlan p = plan_pulsed(M, K, N);
  if (ws_bytes < p.ws_bytes) return XBAR_EWORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  PulseArgs a;
  a.W = W; a.X = X; a.D = dY;
  a.rows = reinterpret_cast<uint32_t*>(ws);
  a.cols = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(ws) + p.rows_bytes);
  a.state = reinterpret_cast<double*>(reinterpret_cast<char*>(ws) + p.rows_bytes + p.cols_bytes);
  a.pulses = pulses;
  a.marks = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(ws) + p.rows_bytes + p.cols_bytes +
                                                  align256((size_t)8 * K * N));
  a.summary = reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(a.marks) +
                                                    align256((size_t)cdiv(p.mc, 64) * 8 * (size_t)K * N));
  a.M = M; a.K = K; a.N = N; a.bl = bl;
  a.flags = cfg->flags;
  a.w_max = (double)w_max; a.x_range = (double)x_range; a.d_range = (double)d_range; a.dw_min = (double)dw_min;
  a.v = (double)cfg->upd_nl_v;
  // the aggregate model's noise for one pulse: its standard deviation gamma sqrt(dG) belongs to the ideal change
  // before the learning rate, and this scheme's mean equals the aggregate update at lr = bl dw_min w_max / (x_range d_range)
  a.coded = (cfg->flags & XBAR_PULSE_CODED) ? 1 : (cfg->flags & XBAR_PULSE_MAGNITUDE) ? 2 : 0;
  coded_frames(bl, &a.tx, &a.td);
  const int slots = a.coded == 1 ? a.tx * a.td : a.coded == 2 ? bl * bl : bl;
  const double lr_eq = (double)slots * (double)dw_min * (double)w_max / ((double)x_range * (double)d_range);
  a.sigma = (double)cfg->upd_noise_gamma * std::sqrt(lr_eq * (double)dw_min);
  a.seed = cfg->seed; a.step = step; a.step_add = current_step_source();
  a.conv = conv ? *conv : ConvGeom{};
  a.series[0] = a.dw_min * std::exp(-0.5 * a.v);
  for (int i = 1; i < 7; ++i) a.series[i] = a.series[i - 1] * (-0.5 * a.v) / (double)i;
  // the seventh power, spread over the lower odd ones: on -1 .. 1 it is (112 g^5 - 56 g^3 + 7 g) / 64 but for a 64th
  const double seventh = a.series[6] * (-0.5 * a.v) / 7.0;
  a.series[5] += seventh * (112.0 / 64.0);
  a.series[3] -= seventh * (56.0 / 64.0);
  a.series[1] += seventh * (7.0 / 64.0);
  // 4 x 4 devices per thread when that still fills the chip, else one device per thread
  const bool patch4 = (long long)cdiv(K, 64) * cdiv(N, 64) >= 512;
  const int edge = patch4 ? 64 : 16;
  const unsigned tiles = (unsigned)(cdiv(K, edge) * cdiv(N, edge));
  for (int m0 = 0; m0 < M; m0 += p.mc) {
    a.m0 = m0;
    a.mc = std::min(p.mc, M - m0);
    a.first = m0 == 0;
    a.last = m0 + a.mc >= M;
    const long long elems = (long long)a.mc * ((long long)K + N);
    if (conv) hipLaunchKernelGGL(pulse_trains_kernel<true>, dim3((unsigned)((elems + 255) / 256)), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(pulse_trains_kernel<false>, dim3((unsigned)((elems + 255) / 256)), dim3(256), 0, st, a);
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
    const bool nl = (cfg->flags & XBAR_NI_UPD_NL) != 0, noise = (cfg->flags & XBAR_NI_UPD_NOISE) != 0;
    if (a.coded == 2) {
      // magnitude coding: a device is written in every sample in which both of its lines carry a pulse, so
      // there is little for a marking pass to skip; always the staged kernel
      void (*k)(PulseArgs);
      if (patch4)
        k = nl ? (noise ? pulse_apply_kernel<4, true, true, false, true> : pulse_apply_kernel<4, true, false, false, true>)
               : (noise ? pulse_apply_kernel<4, false, true, false, true> : pulse_apply_kernel<4, false, false, false, true>);
      else
        k = nl ? (noise ? pulse_apply_kernel<1, true, true, false, true> : pulse_apply_kernel<1, true, false, false, true>)
               : (noise ? pulse_apply_kernel<1, false, true, false, true> : pulse_apply_kernel<1, false, false, false, true>);
      hipLaunchKernelGGL(k, dim3(tiles), dim3(256), 0, st, a);
      if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
      continue;
    }
    if (p.two_phase) {
      a.n_words = cdiv(a.mc, 64);
      const long long devices = (long long)K * N;
      // Up to where the streamed walk beats a lane per device that does everything by itself: the walk that others feed does
      // not take longer for more devices until the feeding waves fill the chip, from then on it does, and an exp() per move
      // fills it sooner.  Streamed / not, around each line, trains of 12 pulses a sample | one per sample | one in 30 samples, whichever
      // lets it lose first, 128 rows and 4096 samples:
      //   linear  400 columns 0.55 | 0.72 | 0.94, 448 0.60 | 0.79 | 1.03; series 352 0.72 | 0.83 | 0.93, 384 0.81 | 0.90 | 1.01; exp() 192 0.94 |
      //   0.98 | 1.00, 208 0.94 | 0.93 | 0.89; with noise: linear 576 0.93 | 0.91 | 1.00; series 544 0.96 | 0.93 | 0.97, 576 1.00 | 0.97 |
      //   1.01; exp() 240 0.99 | 0.95 | 0.91, 256 1.12 | 1.09 | 1.03
      const int line[2][3] = {{55296, 47104, 26624}, {73728, 69632, 30720}};
      const bool stream = devices < line[noise ? 1 : 0][move_mode(a, nl)];
      const unsigned tiles16 = (unsigned)(cdiv(K, 16) * cdiv(N, 16));
      // measured, ms per update, [n_words][K N] / [K N][n_words], walks of one lane per device: noise, 65536 devices x 12544
      // samples 2.23 / 2.27, x 50176 8.53 / 8.93, 524288 x 4096 4.12 / 4.23; without, 65536 x 50176 4.19 / 4.60, 44100 x 100352
      // 7.06 / 7.60, 524288 x 4096 1.75 / 1.89
      a.mark_device = stream ? (size_t)a.n_words : 1;
      a.mark_word = stream ? 1 : (size_t)devices;
      // the plain walk needs whole summary words (64-word segments); else short ones, for some thousand blocks
      a.seg_words = !stream || tiles16 >= 256 ? 64 : tiles16 >= 64 ? 16 : 4;
      hipLaunchKernelGGL(pulse_mark_kernel, dim3(tiles16 * (unsigned)cdiv(a.n_words, a.seg_words)), dim3(256), 0, st, a);
      if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
      if (stream) {
        if (launch_pulse_stream<true>(a, nl, noise, st) != hipSuccess) return XBAR_EHIP;
      } else if (noise) {
        // lanes decoupled over the whole chunk: with a normal number per pulse every turn counts
        void (*walk)(PulseArgs) = nl ? pulse_walk_kernel<true, true> : pulse_walk_kernel<false, true>;
        hipLaunchKernelGGL(walk, dim3((unsigned)cdiv(K * N, 64)), dim3(64), 0, st, a);     // one wave per block: spread over the chip
      } else {
        // cheap pulses: the trains of a stage in LDS beat the walk's loads from memory (measured 6.7 against
        // 9.6 ms on a 144 x 16 layer with 131072 samples; with noise 21 against 15 ms)
        void (*staged)(PulseArgs) = nl ? pulse_apply_kernel<1, true, false, true> : pulse_apply_kernel<1, false, false, true>;
        hipLaunchKernelGGL(staged, dim3(tiles16), dim3(256), 0, st, a);
      }
      if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
      continue;
    }
    // Few devices and samples: streamed without marks.  Streamed / staged, us per update with noise | without: 64 x 10 devices, 64
    // samples 15 / 21 | 14 / 14, 2000 samples 40 / 232 | 37 / 138; 784 x 10, 32 samples 28 / 21 | 20 / 15, 64 29 / 32 | 21 / 21, 1024
    // 91 / 236 | 72 / 135; 400 x 40, 256 samples 61 / 60 | 47 / 35, 2000 253 / 328 | 248 / 192
    if ((long long)K * N <= 8192 && M >= 64) {
      if (launch_pulse_stream<false>(a, nl, noise, st) != hipSuccess) return XBAR_EHIP;
      continue;
    }
    void (*k)(PulseArgs);
    if (patch4)
      k = nl ? (noise ? pulse_apply_kernel<4, true, true> : pulse_apply_kernel<4, true, false>)
             : (noise ? pulse_apply_kernel<4, false, true> : pulse_apply_kernel<4, false, false>);
    else
      k = nl ? (noise ? pulse_apply_kernel<1, true, true> : pulse_apply_kernel<1, true, false>)
             : (noise ? pulse_apply_kernel<1, false, true> : pulse_apply_kernel<1, false, false>);
    hipLaunchKernelGGL(k, dim3(tiles), dim3(256), 0, st, a);
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  }
  return XBAR_OK;
}
}  // namespace

extern "C" {

int xbar_update_pulsed(const xbar_config* cfg, float* W, const float* X, const float* dY, int M, int K, int N, float w_max,
                       float x_range, float d_range, int bl, float dw_min, uint64_t step, long long* pulses, void* ws,
                       size_t ws_bytes, void* hip_stream) {
  return run_update_pulsed(cfg, W, X, dY, M, K, N, w_max, x_range, d_range, bl, dw_min, step, pulses, ws, ws_bytes,
                           hip_stream, nullptr);
}

int xbar_conv_update_pulsed(const xbar_config* cfg, float* W, const float* X, const float* dY, const xbar_conv_geom* geom,
                            int N, float w_max, float x_range, float d_range, int bl, float dw_min, uint64_t step,
                            long long* pulses, void* ws, size_t ws_bytes, void* hip_stream) {
  ConvGeom g;
  int M, K;
  const int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  return run_update_pulsed(cfg, W, X, dY, M, K, N, w_max, x_range, d_range, bl, dw_min, step, pulses, ws, ws_bytes,
                           hip_stream, conv_is_dense(geom) ? nullptr : &g);
}

int xbar_pulse_slots(const xbar_config* cfg, int bl) {
  const int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if (bl < 1 || bl > 31) return XBAR_EINVAL;
  if (cfg->flags & XBAR_PULSE_MAGNITUDE) return bl * bl;
  if (!(cfg->flags & XBAR_PULSE_CODED)) return bl;
  int tx, td;
  coded_frames(bl, &tx, &td);
  return tx * td;
}

}  // extern "C"
