// Forward and backward passes of small layers: input stage, contraction, ADC, shift-and-add over tiles, slices, cycles and
// phases and scaling in one kernel (Sec. IV, IV-B).  Same arithmetic, code for code, as the input quantiser, the contraction
// kernels and the adding-up pass that larger layers run one after the other.
#include "vmm_device.h"

#include <atomic>
#include <chrono>

namespace xbar_detail {

namespace {

// A wave owns one item: an output patch of 32 batch rows x 32 outputs, one virtual tile (phase, array, tile) and one slice.
// A block is NW slices (four or eight) of one patch and virtual tile: its waves quantise the tile's inputs into LDS together while the
// items' plane fragments are on their way (to registers or to the wave's own LDS: no other wave reads them), contract
// them with the digits of every cycle, convert, and add their codes up through LDS.  A patch that takes one block is
// scaled and written by it; else the blocks add to the patch's sums in the workspace (integers: the order does not matter),
// which the first block to come has cleared, and the last one to arrive scales and writes them.
// Bound by latency, from memory and, since every line of code runs a handful of times, from the instruction cache: loads
// are issued as early as they can be, loops stay rolled, nothing is divided.  One wave per item spreads a layer
// of a few patches over the chip, in one launch instead of three.
// Waves of a block.  Weights of more than four slices take eight where their fragments have room in LDS: twice the items share
// the staged inputs, and half as many blocks meet in the patch's sums (or one is left, and none meet).  Where the blocks are few
// and meet all the same, four on more compute units are faster: up to one block of four per compute unit.  us, four / eight waves:
// one block a patch, 73 x 14, 31 rows 12.8 / 10.8, 42 x 32, 1280 rows 9.5 / 8.0; several, 131 x 111, 20 rows backward 11.1 / 12.3,
// 188 x 225, 49 rows 14.1 / 14.9; beyond the line 144 x 82, 646 rows 13.7 / 12.6, 113 x 1396, 736 rows 50.4 / 30.3, 212 x 1116, 200
// rows 50.0 / 37.5; but with few rows of inputs to share, up to four terms and a little more than one block of eight per compute
// unit: signed inputs, 4 terms, 25 x 416, 363 rows, 312 blocks 12.9 / 14.0, 16 x 1056, 150 rows, 330 blocks 12.4 / 13.8, 64 x 192, 900 rows, 348 blocks
// 13.4 / 14.2, 1 term 11.0 / 11.7, 10.8 / 11.6, 11.9 / 12.0, fp16 planes of 2 terms 13.5 / 14.1, 13.1 / 13.3, 15.0 / 15.3 (with 5 terms 19.1 / 15.5,
// 18.5 / 14.6, 18.9 / 15.1).  (Same results.)
int waves_of(const VmmPlan& p, const Derived& d) {
  if (d.S_w <= 4 || (d.fmt == kFmtF16 && d.terms * p.g.ks > 16)) return 4;
  const long long tiles = (long long)p.MP * p.g.OP * p.VT, eights = tiles * cdiv(d.S_w, 8);
  if (p.VT * cdiv(d.S_w, 8) == 1) return 8;
  if (d.terms < 5 && std::min(p.Lin, p.g.tile) <= 64 && eights > 256 && eights <= 384) return 4;
  return tiles * cdiv(d.S_w, 4) > 256 ? 8 : 4;
}

// The sums of a patch that several blocks share, in a workspace whose content is unknown when the launch begins: one
// 64-byte head per patch, then 1024 sums per patch, [4][256 threads], 32-bit where they fit.  Every block begins with an
// exchange of the head's `claim` for the launch's tag, an odd 64-bit number that no other launch of the process carries and
// that no data hold but by a chance of 2^-64: the one block that finds another number there clears the sums and then sets
// `ready`; the others look for it before they add, a few microseconds later, and wait if need be -- for a block that is
// running and waits for nobody.  The last to arrive takes the tag back out: a launch that is replayed from a graph
// carries the same tag again.  Two launches that overlap on one workspace, which callers must not let happen, take
// `claim` and `ready` from each other: the wait therefore has an end, after which a block takes the tag out, writes
// NaN (unscaled sums: the lowest integer) to its patch and is done.  Everything here is a relaxed device-scope operation on memory that all XCDs share, ordered
// by waiting until it has been acknowledged: a device-scope fence would write back a whole L2 per block (it took ten times the
// kernel's time).  A kernel of its own to clear cost each pass 1.9 us and a second launch.
struct PatchHead {
  unsigned long long claim, ready;
  uint32_t tickets, pad[11];
};
__device__ __forceinline__ PatchHead* patch_head(const SmallArgs& s, int patch) { return reinterpret_cast<PatchHead*>(s.ws) + patch; }
__device__ __forceinline__ char* patch_sums(const SmallArgs& s, int patch) {
  return reinterpret_cast<char*>(s.ws) + (size_t)s.v.MP * s.v.OP * sizeof(PatchHead) + (size_t)patch * (s.narrow ? 4096 : 8192);
}
template <class T>
__device__ __forceinline__ void put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class T>
__device__ __forceinline__ T look(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// First wave of every block, before its loads: what `claim` held (lane 0).
__device__ __forceinline__ unsigned long long claim_patch(const SmallArgs& s, int patch, int wave, int lane) {
  unsigned long long before = s.tag;
  if (s.blocks_per_patch > 1 && wave == 0 && lane == 0)
    before = __hip_atomic_exchange(&patch_head(s, patch)->claim, s.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return before;
}
// The same wave, before its block's work begins in earnest: clears the sums if it came first.
__device__ __forceinline__ bool clear_patch(const SmallArgs& s, int patch, unsigned long long before, int lane) {
  if (__ballot(before != s.tag) == 0) return false;
  unsigned long long* sums = reinterpret_cast<unsigned long long*>(patch_sums(s, patch)) + lane;
#pragma unroll 1
  for (int i = 0; i < (s.narrow ? 8 : 16); ++i) put(sums + 64 * i, 0ull);
  if (lane == 0) put(&patch_head(s, patch)->tickets, 0u);
  return true;
}
// ... and a little later, when that has been acknowledged.
__device__ __forceinline__ void open_patch(const SmallArgs& s, int patch, int lane) {
  acknowledged();
  if (lane == 0) put(&patch_head(s, patch)->ready, s.ready_tag);
}

// The inputs of this wave's 16-input steps of the tile: steps wave, wave + NW, .. (up to NSTEP of them).
template <int NW, int NSTEP>
struct Inputs {
  float x[NSTEP][8];
  __device__ __forceinline__ void load(const SmallArgs& s, int mp, int t, int wave, int lane) {
    const int m = mp * 32 + (lane & 31), lend = min(s.v.Lin, (t + 1) * s.v.tile);
#pragma unroll
    for (int i = 0; i < NSTEP; ++i) {
      const int l0 = t * s.v.tile + 16 * (wave + NW * i) + 8 * (lane >> 5);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[i][e] = 0.0f;
      if (l0 < lend && m < s.v.M) {
        if (s.is_conv) load_inputs8<true>(s.q, m, l0, lend, x[i]);
        else load_inputs8<false>(s.q, m, l0, lend, x[i]);
      }
    }
  }
  // their magnitudes into `raw`: [16-input step][64 lanes]
  __device__ __forceinline__ void stage(const SmallArgs& s, u32x2* raw, int mp, int t, int p, int steps, int wave, int lane) const {
    const int m = mp * 32 + (lane & 31), lend = min(s.v.Lin, (t + 1) * s.v.tile);
#pragma unroll
    for (int i = 0; i < NSTEP; ++i) {
      const int j = wave + NW * i;
      if (j >= steps) break;
      u32x2 pos, neg;
      input_codes8(s.q, m, t * s.v.tile + 16 * j + 8 * (lane >> 5), lend, x[i], pos, neg);
      raw[j * 64 + lane] = p ? neg : pos;
    }
  }
};

// Thread (q, lane)'s four outputs when the patch's sums cannot be had.
__device__ __forceinline__ void write_poison(const SmallArgs& s, int m, int o) {
  const VmmArgs& a = s.v;
  if (m >= a.M) return;
#pragma unroll 1
  for (int e = 0; e < 4; ++e) {
    if (o + e >= a.Lout) return;
    const size_t at = (size_t)m * a.Lout + o + e;
    if (a.part && s.narrow) reinterpret_cast<uint32_t*>(a.part)[at] = 0x80000000u;
    else if (a.part) reinterpret_cast<unsigned long long*>(a.part)[at] = 0x8000000000000000ull;
    else a.out[at] = __builtin_nanf("");
  }
}

// The items' codes, summed over their cycles, to the patch's sums, or scaled and written.  Thread (q, lane) of the first four
// waves ends up with the four consecutive outputs 8 q + 4 (lane / 32) .. of batch row lane % 32.
template <int NW>
__device__ __forceinline__ void add_and_write(const SmallArgs& s, u32x4* xch, const uint32_t (&y)[16], int wave, int slice0,
                                              int patch, int mp, int op, int lane) {
#pragma clang fp contract(off)   // product, product, difference: each rounded on its own
  const VmmArgs& a = s.v;
  __syncthreads();                                     // everyone has read what the exchange area held before
#pragma unroll
  for (int q = 0; q < 4; ++q) xch[(wave * 4 + q) * 64 + lane] = u32x4{y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]};
  PatchHead* head = patch_head(s, patch);
  const int m = mp * 32 + (lane & 31), o = op * 32 + 8 * wave + 4 * (lane >> 5);
  __shared__ uint32_t opened, arrived;
  if (s.blocks_per_patch > 1 && threadIdx.x == 0) {
    bool ready = look(&head->ready) == s.tag;
#pragma unroll 1
    for (int turn = 0; !ready && turn < s.wait_turns; ++turn) {
      __builtin_amdgcn_s_sleep(1);
      ready = look(&head->ready) == s.tag;
    }
    if (!ready) {                                      // the tag must not meet the next replay
      put(&head->claim, 0ull);
      put(&head->ready, 0ull);
    }
    opened = ready;
  }
  __syncthreads();
  const bool sums = NW == 4 || wave < 4;
  if (s.blocks_per_patch > 1 && !opened) {
    if (sums) write_poison(s, m, o);
    return;
  }
  if (!sums && s.blocks_per_patch == 1) return;
  long long sum[4] = {0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (slice0 + w >= a.S_w) break;
    const u32x4 v = xch[w * 256 + (threadIdx.x & 255)];
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += (long long)(int32_t)(v[e] - s.bias_item) << (a.slice_bits * (slice0 + w));
  }
  if (s.blocks_per_patch > 1) {
    unsigned long long* wide = reinterpret_cast<unsigned long long*>(patch_sums(s, patch)) + (threadIdx.x & 255);
    uint32_t* narrow = reinterpret_cast<uint32_t*>(patch_sums(s, patch)) + (threadIdx.x & 255);
    if (sums) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (s.narrow) atomicAdd(&narrow[256 * e], (uint32_t)sum[e]);
        else atomicAdd(&wide[256 * e], (unsigned long long)sum[e]);
      }
    }
    acknowledged();                                    // the sums before the ticket
    __syncthreads();
    if (threadIdx.x == 0) arrived = atomicAdd(&head->tickets, 1u);
    __syncthreads();
    if (!sums || arrived != (uint32_t)s.blocks_per_patch - 1) return;
    if (threadIdx.x == 0) {
      put(&head->claim, 0ull);
      put(&head->ready, 0ull);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      sum[e] = s.narrow ? (long long)(int32_t)look(&narrow[256 * e]) : (long long)look(&wide[256 * e]);
  }
  if (m >= a.M) return;
  const size_t at = (size_t)m * a.Lout + o;
  float r[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    double v = (double)sum[e] * a.scale;
    if (s.wsum && o + e < a.Lout) v = v - (double)s.wsum[o + e] * s.half_range;
    r[e] = (float)v;
  }
  if (!a.part && (a.Lout & 3) == 0) {
    if (o < a.Lout) *reinterpret_cast<float4*>(a.out + at) = make_float4(r[0], r[1], r[2], r[3]);
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (o + e < a.Lout) {
      if (a.part && s.narrow) reinterpret_cast<int32_t*>(a.part)[at + e] = (int32_t)sum[e];
      else if (a.part) reinterpret_cast<long long*>(a.part)[at + e] = sum[e];
      else a.out[at + e] = r[e];
    }
}

// What a wave of the launch works on: grid = (virtual tile x group of slices, output patch, row patch).
template <int NW, bool PER_ARRAY>
struct Item {
  int patch, mp, op, p, pol, t, slice0, slice;
  __device__ __forceinline__ Item(const SmallArgs& s, int wave) {
    const VmmArgs& a = s.v;
    op = (int)blockIdx.y;
    mp = (int)blockIdx.z;
    patch = mp * a.OP + op;
    const int vt = (int)((blockIdx.x * s.groups_inv) >> 16);      // blockIdx.x / slice groups
    slice0 = ((int)blockIdx.x - vt * s.slice_groups) * NW;
    slice = min(slice0 + wave, a.S_w - 1);             // a wave without a slice works along, its codes are not added
    const int pa = (vt >= a.T ? 1 : 0) + (vt >= 2 * a.T ? 1 : 0) + (vt >= 3 * a.T ? 1 : 0);   // (phase, array)
    t = vt - pa * a.T;
    p = PER_ARRAY ? pa >> 1 : pa;
    pol = PER_ARRAY ? pa & 1 : 0;
  }
};

// fp16 planes: the wave's fragments go from memory into its share of LDS (no registers in between, all in flight at
// once), and a short loop takes them in order (leading term first; one array alone: the residual first), every fragment
// with the digits of all cycles at once, reading one pair of fragments ahead.
template <int NW, int TERMS, int S_IN, bool PER_ARRAY, int NSTEP>
__global__ __launch_bounds__(64 * NW) void vmm_small_f16_kernel(SmallArgs s) {
  extern __shared__ u32x4 small_lds[];
  const VmmArgs& a = s.v;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Item<NW, PER_ARRAY> it(s, wave);
  u32x2* raw = reinterpret_cast<u32x2*>(small_lds);    // [16-input step][64 lanes]
  u32x4* frags = small_lds + a.ks16 * 32 + (size_t)wave * TERMS * a.ks * 64;
  const int nk = (min(a.tile, a.Lin - it.t * a.tile) + 15) >> 4, nf = TERMS * nk;
  const unsigned long long before = claim_patch(s, it.patch, wave, lane);
  Inputs<NW, NSTEP> inputs;
  inputs.load(s, it.mp, it.t, wave, lane);
  const u32x4* src = a.B + (((size_t)it.t * a.OP + it.op) * a.S_w + it.slice) * TERMS * a.ks * 64 + lane;
  if constexpr (PER_ARRAY) src += (size_t)it.pol * a.pol_stride;
#pragma unroll
  for (int i = 0; i < TERMS; ++i) {
    const int term = PER_ARRAY ? TERMS - 1 - i : i;
#pragma unroll 1
    for (int j = 0; j < nk; ++j) copy16_global_to_lds(src + (term * a.ks + j) * 64, frags + (i * nk + j) * 64);
  }
  inputs.stage(s, raw, it.mp, it.t, it.p, nk, wave, lane);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const bool first = clear_patch(s, it.patch, before, lane);
  __syncthreads();
  const uint32_t digit_mask8 = ((1u << a.stream_bits) - 1u) * 0x01010101u;
  float16v acc[S_IN];
#pragma unroll
  for (int b = 0; b < S_IN; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;
  const u32x2* in = raw + lane;
  auto read = [&](int f, u32x2& x, u32x4& w) __attribute__((always_inline)) {   // behind the end: the last one again
    const int i = min(f, nf - 1);
    x = in[(i >= nk ? i - nk : i) * 64];
    w = frags[i * 64 + lane];
  };
  u32x2 x0, x1;
  u32x4 w0, w1;
  read(0, x0, w0);
  read(1, x1, w1);
#pragma unroll 1
  for (int f = 0; f < nf; f += 2) {
    u32x2 nx0, nx1;
    u32x4 nw0, nw1;
    read(f + 2, nx0, nw0);
    read(f + 3, nx1, nw1);
#pragma unroll
    for (int b = 0; b < S_IN; ++b)
      acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, w0),
                                                      digit_fragment(x0, digit_mask8 << (a.stream_bits * b)), acc[b], 0, 0, 0);
    if (f + 1 < nf) {
#pragma unroll
      for (int b = 0; b < S_IN; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, w1),
                                                        digit_fragment(x1, digit_mask8 << (a.stream_bits * b)), acc[b], 0, 0, 0);
    }
    x0 = nx0; x1 = nx1; w0 = nw0; w1 = nw1;
  }
  if (first) open_patch(s, it.patch, lane);
  float gain, lo, hi;
  adc_sign_and_range<PER_ARRAY>(a, it.p, it.pol, gain, lo, hi);
  uint32_t y[1][16];
#pragma unroll
  for (int r = 0; r < 16; ++r) y[0][r] = 0;
#pragma unroll
  for (int b = 0; b < S_IN; ++b) {
    const float16v one[1] = {acc[b]};
    // operand lanes hold digit * 2^(shift - 24); undo that power of two in the ADC gain
    vmm_adc_narrow<1>(one, ldexpf(gain, 24 - a.stream_bits * b), lo, hi, a.stream_bits * b, y);
  }
  add_and_write<NW>(s, small_lds + a.ks16 * 32, y[0], wave, it.slice0, it.patch, it.mp, it.op, lane);
}

// 6-bit planes: the item's fragments stay in registers while its cycles pass, two at a time (two chains of sums); with eight waves and
// two k-steps one at a time, which leaves room for a second block on the compute unit (113 x 1396, 736 rows, 5 terms: 38.7 -> 30.3 us).
template <int NW, int NT, int NK, bool PER_ARRAY>
__global__ __launch_bounds__(64 * NW, NW == 8 && NK <= 2 ? 4 : 1) void vmm_small_f6_kernel(SmallArgs s) {
  constexpr int CH = NW == 8 && NK == 2 ? 1 : 2;
  extern __shared__ u32x4 small_lds[];
  const VmmArgs& a = s.v;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Item<NW, PER_ARRAY> it(s, wave);
  u32x2* raw = reinterpret_cast<u32x2*>(small_lds);
  const int nk = (min(a.tile, a.Lin - it.t * a.tile) + 63) >> 6;
  const unsigned long long before = claim_patch(s, it.patch, wave, lane);
  Inputs<NW, (4 * NK + NW - 1) / NW> inputs;
  inputs.load(s, it.mp, it.t, wave, lane);
  const char* src = reinterpret_cast<const char*>(a.B + (PER_ARRAY ? (size_t)it.pol * a.pol_stride : 0)) +
                    (((size_t)it.t * a.OP + it.op) * a.S_w + it.slice) * NT * a.ks * 1536;
  u32x4 fx[NT][NK];
  u32x2 fy[NT][NK];
#pragma unroll
  for (int term = 0; term < NT; ++term)
#pragma unroll
    for (int J = 0; J < NK; ++J) {
      const char* f = src + (size_t)(term * a.ks + min(J, nk - 1)) * 1536;   // a step the tile does not reach is not used
      fx[term][J] = *reinterpret_cast<const u32x4*>(f + lane * 16);
      fy[term][J] = *reinterpret_cast<const u32x2*>(f + 1024 + lane * 8);
    }
  inputs.stage(s, raw, it.mp, it.t, it.p, 4 * NK, wave, lane);   // zero beyond the tile
  if (clear_patch(s, it.patch, before, lane)) open_patch(s, it.patch, lane);
  __syncthreads();
  const uint32_t nibble_mask = ((1u << a.stream_bits) - 1u) * 0x11111111u;
  float gain, lo, hi;
  adc_sign_and_range<PER_ARRAY>(a, it.p, it.pol, gain, lo, hi);
  gain *= 2.0f;                                        // a digit enters as d / 2
  uint32_t y[1][16];
#pragma unroll
  for (int r = 0; r < 16; ++r) y[0][r] = 0;
#pragma unroll 1
  for (int b = 0; b < ((a.S_in + 1) & ~1); b += CH) {
    float16v acc[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[c][r] = 0.0f;
    int4v dg[CH][NK];
#pragma unroll
    for (int J = 0; J < NK; ++J)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const u32x2 x = raw[(4 * J + w) * 64 + lane];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int at = a.stream_bits * (b + c);      // the digit's place: low or high nibbles (none behind the last cycle)
          dg[c][J][w] = (int)(((at & 4 ? x.y : x.x) >> (at & 3)) & (b + c < a.S_in ? nibble_mask : 0u));
        }
      }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int J = 0; J < NK; ++J)
        if (J < nk) {                                  // the same for the whole block
          const int term = PER_ARRAY ? NT - 1 - i : i;
          const u32x4 x = fx[term][J];
          const u32x2 w = fy[term][J];
          const int8v pa = {(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)w.x, (int)w.y, 0, 0};
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            const int8v pb = {dg[c][J][0], dg[c][J][1], dg[c][J][2], dg[c][J][3], 0, 0, 0, 0};
            acc[c] = mfma_f6_term(term, pa, pb, acc[c], a.scale_lo, a.scale_hi);
          }
        }
    // a cycle that is not there leaves zero codes: their constant alone goes into the sums, and out again with the bias
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const float16v one[1] = {acc[c]};
      vmm_adc_narrow<1>(one, gain, lo, hi, a.stream_bits * (b + c), y);
    }
  }
  add_and_write<NW>(s, small_lds + NK * 128, y[0], wave, it.slice0, it.patch, it.mp, it.op, lane);
}

// Another odd 64-bit number at every call: even steps, the golden ratio's, from an odd start that differs from process to process.
unsigned long long launch_tag() {
  static std::atomic<unsigned long long> next{(unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0xD6E8FEB86659FD93ull | 1};
  return next.fetch_add(0x9E3779B97F4A7C16ull, std::memory_order_relaxed);
}

// Turns of the wait, 0.13 us each on an idle chip: what it waits for takes microseconds, so 0.14 s is out of reach of a
// launch that has its workspace to itself, also on a chip that others use.
constexpr int kWaitTurns = 1 << 20;
thread_local int g_withheld_turns = -1;

int blocks_per_patch(const VmmPlan& p, const Derived& d) { return p.VT * cdiv(d.S_w, waves_of(p, d)); }
// the staged inputs and the area of the final exchange (4 KiB a wave), which the fragments of fp16 planes occupy before
size_t small_lds_bytes(const VmmPlan& p, const Derived& d) {
  const int steps = d.fmt == kFmtF6 ? 4 * (p.g.ks == 3 ? 4 : p.g.ks) : p.ks16, waves = waves_of(p, d);
  const size_t frags = d.fmt == kFmtF16 ? (size_t)waves * d.terms * p.g.ks * 1024 : 0;
  return (size_t)steps * 512 + std::max((size_t)4096 * waves, frags);
}

template <int NW, int NSTEP>
void (*pick_f16(int terms, int s_in, bool per_array))(SmallArgs) {
  if (per_array) return s_in == 1 ? vmm_small_f16_kernel<NW, 2, 1, true, NSTEP> : vmm_small_f16_kernel<NW, 2, 2, true, NSTEP>;
  if (terms == 2) return s_in == 1 ? vmm_small_f16_kernel<NW, 2, 1, false, NSTEP> : vmm_small_f16_kernel<NW, 2, 2, false, NSTEP>;
  return s_in == 1 ? vmm_small_f16_kernel<NW, 1, 1, false, NSTEP> : vmm_small_f16_kernel<NW, 1, 2, false, NSTEP>;
}

template <int NW, int NK>
void (*pick_f6(int terms, bool per_array))(SmallArgs) {
  if (per_array) return vmm_small_f6_kernel<NW, 5, NK, true>;
  if (terms == 1) return vmm_small_f6_kernel<NW, 1, NK, false>;
  return terms == 4 ? vmm_small_f6_kernel<NW, 4, NK, false> : vmm_small_f6_kernel<NW, 5, NK, false>;
}

template <int NW>
void (*pick_small(const VmmPlan& p, const Derived& d))(SmallArgs) {
  const bool per_array = d.npol == 2;
  if (d.fmt == kFmtF6) return p.g.ks == 1 ? pick_f6<NW, 1>(d.terms, per_array) : p.g.ks == 2 ? pick_f6<NW, 2>(d.terms, per_array) : pick_f6<NW, 4>(d.terms, per_array);
  const int steps = cdiv(p.ks16, NW);                  // 16-input steps that a wave stages
  if (steps <= 1) return pick_f16<NW, 1>(d.terms, d.S_in, per_array);
  if (steps <= 2 || NW == 8) return pick_f16<NW, 2>(d.terms, d.S_in, per_array);
  return pick_f16<NW, NW == 8 ? 2 : 4>(d.terms, d.S_in, per_array);
}

}  // namespace

size_t vmm_small_ws_bytes(const VmmPlan& p, const Derived& d) {
  if (blocks_per_patch(p, d) == 1) return 0;
  const size_t patches = (size_t)p.MP * p.g.OP;
  return align256(patches * (sizeof(PatchHead) + (p.narrow ? 4096 : 8192)));
}

// When the one launch beats the three it replaces: where 95 % of its estimate in us is below theirs, up to 16384 items of one
// patch, tile and slice, with 6-bit planes and eight waves 65536, beyond which neither was measured closely.  It costs whole
// blocks, whether or not they hold as many slices as waves; a block's time grows with the fragments it reads (terms x k-steps, of
// a tile with fp16 planes those that the layer reaches), and with fp16 planes a round of as many blocks as the LDS of the compute
// units holds takes 5 us at least.  The three take what the plan expects of the chunked kernel, what each of its waves stages,
// and two launches.  Fitted in graphs of 10 calls to random layers, matrices and convolutions, 75000 with blocks of four waves and
// 800 with eight (us, three / one: 2000 x 300, 64 rows, 64-row arrays, fp16: 32 / 22; four waves, 256 rows, 1 tile, 4 terms, 8192
// items: 42 / 50; eight, 113 x 1396, 736 rows, 5 terms, 8096 items: 47 / 30, 1396 x 113 backward, 16192 items: 85 / 58).  From the
// better side the layers are 0.3 % away on average with 6-bit planes, 0.1 % with fp16 planes.
// fp16 planes of tiles beyond 128 rows leave one to three blocks the LDS of a compute unit: 4096 items and one round
// (us, three / one: 192 rows, 1122 blocks, one resident: 20 / 51; 256 rows, 2448 blocks: 31 / 119).
bool vmm_small_pays(const VmmPlan& p, const Derived& d) {
  const int waves = waves_of(p, d);
  const long long patches = (long long)p.MP * p.g.OP, items = patches * p.VT * d.S_w;
  const long long blocks = patches * blocks_per_patch(p, d);
  if (p.g.OP >= 65536 || p.MP >= 65536 || (long long)blocks_per_patch(p, d) * cdiv(d.S_w, waves) >= 65536) return false;
  if (items > (d.fmt == kFmtF6 && waves == 8 ? 65536 : 16384)) return false;
  const int rows = std::min(p.Lin, p.g.tile);
  if (d.fmt == kFmtF16) {
    // in groups of four waves
    const double groups = (double)(patches * p.VT * cdiv(d.S_w, 4));
    const double resident = 256.0 * (double)std::min<size_t>(32 / waves, 160 * 1024 / small_lds_bytes(p, d)) * (waves / 4);
    if (p.ks16 > 8) return items <= 4096 && groups <= resident;
    const double group_us = (waves == 8 ? 0.85e-3 : 1e-3) * (1.1 + 0.93 * d.terms * cdiv(rows, 16));
    const double one = 6.5 + std::max(groups * group_us + (blocks > patches ? 1.2 : 0.0), 5.0 * groups / resident);
    return one <= 0.95 * (10.3 + 1.27 * p.chunked_us - 1.03 * p.vt_planned + 0.35 * p.nchunk);
  }
  const int read_steps = p.g.ks == 3 ? 4 : p.g.ks;                  // k-steps of a block, and those that a tile reaches
  const int frags = d.S_w * d.terms * cdiv(rows, 64);
  const double one = waves == 8 ? 8.5 + 1e-3 * (double)blocks * (5.5 + 2.15 * d.terms * read_steps) + (blocks > patches ? 0.7 : 0.0)
                                : 8.4 + 1e-3 * (double)blocks * (6.7 + d.terms * read_steps + 0.94 * (d.npol - 1)) + (p.VT > 1 ? 0.5 : 0.0);
  return one <= 0.95 * (9.1 + 0.98 * p.chunked_us + p.vt_planned * (0.32 * frags / p.nw - 1.4) + 0.33 * p.nchunk);
}

hipError_t launch_vmm_small(SmallArgs a, const VmmPlan& p, const Derived& d, hipStream_t st) {
  a.blocks_per_patch = blocks_per_patch(p, d);
  a.slice_groups = cdiv(d.S_w, waves_of(p, d));
  a.groups_inv = (65536 + a.slice_groups - 1) / a.slice_groups;   // exact for quotients of numbers below 65536 / groups
  a.tag = a.ready_tag = launch_tag();
  a.wait_turns = kWaitTurns;
  if (g_withheld_turns >= 0) {
    a.ready_tag = 0;
    a.wait_turns = g_withheld_turns;
    g_withheld_turns = -1;
  }
  const int waves = waves_of(p, d);
  void (*k)(SmallArgs) = waves == 8 ? pick_small<8>(p, d) : pick_small<4>(p, d);
  const size_t lds = small_lds_bytes(p, d);
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)a.blocks_per_patch, (unsigned)p.g.OP, (unsigned)p.MP), dim3(64 * waves), lds, st, a);
  return hipGetLastError();
}

}  // namespace xbar_detail

extern "C" void xbar_withhold_next_small_vmm(int turns) { xbar_detail::g_withheld_turns = turns; }
