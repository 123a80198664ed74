// xbar: emulation of non-ideal resistive-crossbar training operations on MI355X (gfx950).
// HIP kernels and the C-ABI entry points declared in include/xbar.h.
//
// Method: TxSim (arXiv 2002.11151) Sec. IV (DAC -> array -> ADC per layer, forward and backward),
// Sec. IV-A (non-ideal conductance matrix generator), Sec. IV-C (update model), Sec. IV-D
// (approximate analytical wire model / stored distortion profile).
//
// Kernel plan
//   tile_planes     weights -> quantise -> bit slices -> device conductances -> variation -> wire model
//                   -> stitched signed planes U, written as fp16 MFMA B-operand fragments
//                   (one term when U is an exact digit, hi + lo terms when U is a real number)
//   quantize_input  activations / errors -> integer magnitudes, written as MFMA A-operand fragments
//                   that keep the raw 8-bit magnitude in each 16-bit lane
//   vmm             per (tile, slice, cycle, phase): MFMA contraction (fp16 operands, fp32
//                   accumulate) + ADC + shift-and-add fused in registers
//   vmm_finish      sum of the integer partial results over tile chunks -> scaled fp32 output
//   grad_gemm       X^T dY with fp32 MFMA, split over the batch
//   update_write    batch-partial sum -> non-linear, noisy conductance write, in place
//
// Operand trick of vmm: a 16-bit lane that holds the integer field `digit << shift` (shift < 10) is,
// read as fp16, the subnormal number digit * 2^(shift-24).  The matrix cores of gfx950 take fp16
// subnormals exactly, so one AND with a digit mask turns the raw magnitudes into the A operand of
// any streaming cycle; the power of two is folded into the ADC gain.
//
// Cycles of 1 or 2 bits (the paper's streaming scheme) run on the block-scaled 6-bit / 4-bit matrix
// instruction instead (v_mfma_scale_f32_32x32x64_f8f6f4: 64 rows per instruction in the time fp16 takes
// for 16): a digit d is the E2M1 code d (value d / 2), a plane value is a sum of E2M3 numbers times
// powers of two that the instruction applies as block scales (xbar_common.h), accumulated in fp32 with
// the leading term first.
#include "vmm_device.h"

using namespace xbar_detail;

namespace {

// ---------------------------------------------------------------------------------------------
// generator: weights -> operand planes (Sec. IV-A, IV-D)
// ---------------------------------------------------------------------------------------------
struct TileArgs {
  const float* W;
  const float* profile;
  const uint32_t* codes; // term codes of every plane value (single-path wire model alone), this copy's orientation
  const double* wire_u;  // all-paths wire model: plane values [S_w][2][K][N], array index 0 (else unused)
  uint16_t* planes;  // start of this copy
  int K, N, R, C, S_w, slice_bits, terms;
  int tile, ks, T, OP;
  int spt;           // table-driven generator: slices per thread
  uint32_t flags;
  double g_min, dg, inv_dg, var_sigma, r_row, r_col, r_source, r_sense, hi_scale, hi_inv_scale;
  double qw, q_per_w;    // 2^weight_bits - 1, and that over w_max
  float w_max;
  uint64_t seed, step;
  const unsigned long long* step_add;   // optional device counter added to step
  long long n_threads;
  int term_exp[kMaxTermsF6];            // kFmtF6: power of two of every term
};

// Plane value of slice s of weight (k, n), which sits at place (i, j) of its array, in units of one device level: the
// signed difference of the device pair, or the conductance of one of the two devices.
//   NPOL 1: u[0] = array 0 minus array 1;  2: u[0], u[1] = the arrays alone.
template <int NPOL>
__device__ __forceinline__ void plane_values(const TileArgs& a, NormalStream& rng, int sign, int digit, int s, int k, int n, int i,
                                             int j, double (&u)[NPOL]) {
  if (a.flags & XBAR_NI_WIRE_AAM2) {
#pragma unroll
    for (int pol = 0; pol < NPOL; ++pol) u[pol] = a.wire_u[((size_t)(2 * s + pol) * a.K + k) * a.N + n];
    return;
  }
  if (NPOL == 1 && !(a.flags & (XBAR_NI_VARIATION | XBAR_NI_WIRE_AAM | XBAR_NI_WIRE_PROFILE))) {
    u[0] = (double)(sign * digit);
    return;
  }
  double g[2];
  g[0] = a.g_min + (sign > 0 ? digit * a.dg : 0.0);
  g[1] = a.g_min + (sign < 0 ? digit * a.dg : 0.0);
  if (a.flags & XBAR_NI_VARIATION) {
    double z[2];                                     // the two devices of a pair: consecutive numbers, one draw
    rng.pair((((uint64_t)k * (uint64_t)a.N + (uint64_t)n) * (uint64_t)a.S_w + (uint64_t)s) * 2, z[0], z[1]);
    g[0] *= 1.0 + a.var_sigma * z[0];
    g[1] *= 1.0 + a.var_sigma * z[1];
  }
  if (a.flags & XBAR_NI_WIRE_AAM) {
    const double rho = a.r_source + (double)(j + 1) * a.r_row + (double)(a.R - i) * a.r_col + a.r_sense;
    if constexpr (NPOL == 1) {   // g0 / (1 + rho g0) - g1 / (1 + rho g1), with one division
      u[0] = (g[0] - g[1]) * a.inv_dg / ((1.0 + rho * g[0]) * (1.0 + rho * g[1]));
      return;
    }
    g[0] = g[0] / (1.0 + rho * g[0]);
    g[1] = g[1] / (1.0 + rho * g[1]);
  } else if (a.flags & XBAR_NI_WIRE_PROFILE) {
#pragma unroll
    for (int pol = 0; pol < 2; ++pol)
      g[pol] = g[pol] * (1.0 - (double)a.profile[(((size_t)s * 2 + pol) * a.K + k) * a.N + n]);
  }
  if (NPOL == 1) {
    u[0] = (g[0] - g[1]) * a.inv_dg;
  } else {
#pragma unroll
    for (int pol = 0; pol < NPOL; ++pol) u[pol] = g[pol] * a.inv_dg;
  }
}

// Both copies of one layer's planes.
struct BothCopies {
  TileArgs a;                // K, N, physics; the per-copy members are unused
  uint8_t* base[2];          // forward copy, backward copy
  int OP[2], ks[2], tile[2]; // output patches, k-steps per tile, tile length of either copy
  size_t pol_bytes[2];
  int nb;                    // blocks along n
};

// Nearest half of a double: rounded to odd in single precision on the way, so that the second rounding decides as one
// would (the compiler's own sequence takes some forty integer instructions, and it was most of a plane value's cost).
__device__ __forceinline__ _Float16 half_of(double x) {
  const float f = (float)x;
  const double back = (double)f;
  uint32_t b = __builtin_bit_cast(uint32_t, f);
  if (back != x && !(b & 1)) b += ::fabs(back) < ::fabs(x) ? 1u : ~0u;
  return (_Float16)__builtin_bit_cast(float, b);
}

// fp16 planes, both copies at once: a block owns 32 x 32 weights and two slices (blockIdx.y counts slice pairs), computes
// every device of them once -- in double precision -- turns the values through LDS as (leading term, residual) pairs
// of halves and writes the operand chunks of both directions, 16 bytes each.  A layer of few blocks is bound by latency and
// by the instruction cache (a line of code that runs once costs some 115 cycles to fetch), so it takes 1024 threads
// with one weight and one chunk each; one with many blocks takes 256.  256 x 256 weights, 4 slices: one kernel per copy
// with 8 devices of a column per thread took 14 + 11 us, this with 4 weights per thread unrolled 9.4 - 10, this 6.2;
// 784 x 500: 12.3 instead of 19, 2048 x 1024, 8 slices: 64 instead of 114.
template <int NPOL, int NTH>
__global__ __launch_bounds__(NTH) void tile_f16_kernel(BothCopies b) {
  __shared__ uint32_t uv[NPOL][2][32][33];           // [array][slice of the pair][k][n]: leading half | residual << 16
  const TileArgs& a = b.a;
  const int kb = (int)(blockIdx.x / b.nb), k0 = kb * 32, n0 = ((int)blockIdx.x - kb * b.nb) * 32;
  const int s0 = 2 * (int)blockIdx.y, ns = min(2, a.S_w - s0);
  const int nl = threadIdx.x & 31;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
  const uint32_t dmask = (1u << a.slice_bits) - 1;
  const int n = n0 + nl;
  // place in the array: a patch of 32 reaches into the next array or two where arrays are no whole patches
  int j = n0 % a.C + nl;
  if (j >= a.C) j -= a.C;
  if (j >= a.C) j -= a.C;
  const int kl0 = threadIdx.x >> 5;
  const float* wn = a.W + min(n, a.N - 1);             // one weight ahead
  float w = wn[(size_t)min(k0 + kl0, a.K - 1) * a.N];
#pragma unroll 1
  for (int kl = kl0; kl < 32; kl += NTH / 32) {
    const int k = k0 + kl;
    const float w_now = w;
    if (NTH < 1024) w = wn[(size_t)min(k + NTH / 32, a.K - 1) * a.N];
    int i = k0 % a.R + kl;
    if (i >= a.R) i -= a.R;
    if (i >= a.R) i -= a.R;
    const bool real = k < a.K && n < a.N;
    const int q = real ? quantized_weight(w_now, (double)a.w_max, a.qw, a.q_per_w) : 0;
    const int sign = (q > 0) - (q < 0);
    const uint32_t mag = (uint32_t)::abs(q);
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
      double u[NPOL];
#pragma unroll
      for (int pol = 0; pol < NPOL; ++pol) u[pol] = 0.0;
      if (real && sl < ns)
        plane_values<NPOL>(a, rng, sign, (int)((mag >> (a.slice_bits * (s0 + sl))) & dmask), s0 + sl, k, n, i, j, u);
#pragma unroll
      for (int pol = 0; pol < NPOL; ++pol) {
        // leading term on the grid 2^-hi_frac (coarser where fp16 cannot hold it), residual in fp16
        // (on the grid: exact in single precision)
        const _Float16 h = a.terms == 2 ? (_Float16)(float)(::rint(u[pol] * a.hi_scale) * a.hi_inv_scale) : half_of(u[pol]);
        const _Float16 l = half_of(u[pol] - (double)(float)h);
        uv[pol][sl][kl][nl] = (uint32_t)__builtin_bit_cast(uint16_t, h) | ((uint32_t)__builtin_bit_cast(uint16_t, l) << 16);
      }
    }
  }
  __syncthreads();
  const int t_k = k0 / b.tile[0], r_k = k0 - t_k * b.tile[0], t_n = n0 / b.tile[1], r_n = n0 - t_n * b.tile[1];
  // chunk = (slice, direction, term, 16-row step, lane): entries c0 .. c0 + 7 of one output
#pragma unroll 1
  for (int chunk = threadIdx.x; chunk < 1024 * NPOL; chunk += NTH) {
    const int lane = chunk & 63, js = (chunk >> 6) & 1, term = (chunk >> 7) & 1, dir = (chunk >> 8) & 1, sl = (chunk >> 9) & 1;
    const int pol = NPOL == 2 ? chunk >> 10 : 0;
    const int ol = lane & 31, c0 = 16 * js + 8 * (lane >> 5);
    const int c = (dir == 0 ? k0 : n0) + 16 * js, op = (dir == 0 ? n0 : k0) >> 5;
    if (term >= a.terms || sl >= ns || c >= (dir == 0 ? a.K : a.N)) continue;   // the contraction never reads that k-step
    const bool next = (dir == 0 ? r_k : r_n) + 16 * js >= b.tile[dir];         // a step of 16 lies in one tile
    const int t = (dir == 0 ? t_k : t_n) + (next ? 1 : 0), step = ((dir == 0 ? r_k : r_n) + 16 * js - (next ? b.tile[dir] : 0)) >> 4;
    const uint32_t* from = &uv[pol][sl][0][0] + (dir == 0 ? c0 * 33 + ol : ol * 33 + c0);
    const int stride = dir == 0 ? 33 : 1;
    const uint32_t pick = term == 0 ? 0x05040100u : 0x07060302u;                // the low or the high halves of two words
    u32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_perm(from[(2 * e + 1) * stride], from[2 * e * stride], pick);
    const size_t at = (((((size_t)t * b.OP[dir] + op) * a.S_w + s0 + sl) * a.terms + term) * b.ks[dir] + step) * 64 + lane;
    reinterpret_cast<u32x4*>(b.base[dir] + (size_t)pol * b.pol_bytes[dir])[at] = v;
  }
}

// Codes of a plane value in the 6-bit format: E2M3 numbers (1 sign, 2 exponent, 3 mantissa bits, bias 1: multiples of
// 1/8 up to 2, of 1/4 up to 4, of 1/2 up to 7.5) times 2^term_exp[j], each the nearest to what the terms before it
// left; term j's code at bit 6 j.  Adding 1.5 x 2^52 steps rounds to a multiple of the step (half to even) and leaves
// the multiple in the low bits, so a term costs two additions and integer work (rndne and ldexp are quarter-rate).
__device__ __forceinline__ uint32_t term_codes(double left, int terms, const int (&term_exp)[kMaxTermsF6]) {
  uint32_t word = 0;
#pragma unroll
  for (int j = 0; j < kMaxTermsF6; ++j) {
    if (j >= terms) break;
    const uint32_t bias = (uint32_t)(1023 + term_exp[j]) << 20;
    const uint32_t sign = (uint32_t)__double2hiint(left) & 0x80000000u;
    const double a = ::fmin(::fabs(left), __hiloint2double((int)(bias + (2u << 20) + 0xE0000u), 0));   // 7.5 units at most
    const uint32_t high = (uint32_t)__double2hiint(a);
    const uint32_t binade = (high >= bias + (1u << 20) ? 1u : 0u) + (high >= bias + (2u << 20) ? 1u : 0u);
    const double magic = __hiloint2double((int)(bias + ((49u + binade) << 20) + 0x80000u), 0);
    const double sum = a + magic;
    const uint32_t code = (uint32_t)__double2loint(sum) + 8u * binade;
    const double v = sum - magic;
    left -= __hiloint2double((int)((uint32_t)__double2hiint(v) | sign), __double2loint(v));
    word |= (code | (code ? sign >> 26 : 0u)) << (6 * j);
  }
  return word;
}

// Planes in the 6-bit format: one thread produces the 8 contraction entries (48 bits per term) that one
// byte pair group of the input stage covers, for one output column and one slice (blockIdx.y).
// Thread -> (output index fastest, then the 8-entry slot of the tile, then the tile); slots of k-steps
// that the tile does not reach are skipped, slots beyond its rows inside a k-step are written as zeros.
template <bool TRANSPOSED>
__global__ __launch_bounds__(256) void tile_planes_f6_kernel(TileArgs a) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= a.n_threads) return;
  const int out_len_pad = a.OP * 32;
  const int o = (int)(tid % out_len_pad);
  const int cg = (int)(tid / out_len_pad);
  const int slots = a.ks * 8;                       // 8-entry slots per tile (whole k-steps of 64)
  const int t = cg / slots, slot = cg - t * slots;
  const int within = slot * 8;
  const int Lc = TRANSPOSED ? a.N : a.K;
  const int Lo = TRANSPOSED ? a.K : a.N;
  const int rows = min(a.tile, Lc - t * a.tile);
  const int J = within >> 6;
  if (J * 64 >= rows) return;                       // the contraction never reads this k-step
  const int w = (within & 63) >> 4, half = (within & 15) >> 3;
  const int lane = (o & 31) + 32 * half;
  const int op = o >> 5;
  const int c0 = t * a.tile + within;
  const int s = blockIdx.y;

  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
  const uint32_t dmask = (1u << a.slice_bits) - 1;
  unsigned long long bits[kMaxTermsF6];
#pragma unroll
  for (int j = 0; j < kMaxTermsF6; ++j) bits[j] = 0ull;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int c = c0 + e;
    if (within + e >= rows || o >= Lo) continue;
    const int k = TRANSPOSED ? o : c, n = TRANSPOSED ? c : o;
    const int q = quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w);
    const int sign = (q > 0) - (q < 0);
    const uint32_t mag = (uint32_t)::abs(q);
    double u[1];
    plane_values<1>(a, rng, sign, (int)((mag >> (a.slice_bits * s)) & dmask), s, k, n, k % a.R, n % a.C, u);
    const uint32_t word = term_codes(u[0], a.terms, a.term_exp);
    const int nibble = 2 * (e & 3) + (e >> 2);       // where the input stage's byte e lands in the digit word
#pragma unroll
    for (int j = 0; j < kMaxTermsF6; ++j) {
      if (j >= a.terms) break;
      bits[j] |= (unsigned long long)((word >> (6 * j)) & 63u) << (6 * nibble);
    }
  }
  // 24-byte record of the lane: bytes 0..15 in the fragment's first KiB, 16..23 in its last half KiB
  const size_t frag0 = (((size_t)t * a.OP + op) * a.S_w + s) * a.terms * a.ks + J;
  uint8_t* base = reinterpret_cast<uint8_t*>(a.planes);
#pragma unroll
  for (int j = 0; j < kMaxTermsF6; ++j) {
    if (j >= a.terms) break;
    uint8_t* frag = base + (frag0 + (size_t)j * a.ks) * 1536;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      const int off = 6 * w + 2 * h;
      uint8_t* dst = off < 16 ? frag + lane * 16 + off : frag + 1024 + lane * 8 + (off - 16);
      *reinterpret_cast<uint16_t*>(dst) = (uint16_t)(bits[j] >> (16 * h));
    }
  }
}


// General 6-bit generator, first pass: one thread per device pair (k, n) and slice (blockIdx.y) computes the plane
// value -- quantisation, variation draw, wire model: the arithmetic of tile_planes_f6_kernel -- once, splits it
// into the terms of the schedule and stores the codes as one word per array: words[array][slice][k][n].
template <int NPOL>
__global__ __launch_bounds__(256) void device_words_kernel(TileArgs a, uint32_t* words) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= (long long)a.K * a.N) return;
  const int n = (int)(tid % a.N), k = (int)(tid / a.N);
  const int s = blockIdx.y;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
  const uint32_t dmask = (1u << a.slice_bits) - 1;
  const int q = quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w);
  const int sign = (q > 0) - (q < 0);
  const uint32_t mag = (uint32_t)::abs(q);
  double u[NPOL];
  plane_values<NPOL>(a, rng, sign, (int)((mag >> (a.slice_bits * s)) & dmask), s, k, n, k % a.R, n % a.C, u);
#pragma unroll
  for (int pol = 0; pol < NPOL; ++pol)
    words[(((size_t)pol * a.S_w + s) * a.K + k) * a.N + n] = term_codes(u[pol], a.terms, a.term_exp);
}

// Second pass: one plane copy from the words of its array (a.codes: [slice][k][n]), integer work only.  One wave
// per fragment group (tile, output patch of 32, k-step of 64, slice): it reads the 64 x 32 words of its patch with
// whole-line loads (along n, the fastest index of the words, whichever index this copy contracts over), turns them
// through LDS, and every lane packs the 32 codes of its record for each term and writes it with one 16-byte and one
// 8-byte store.  a.n_threads: 64 x the number of fragment groups.
template <bool TRANSPOSED>
__global__ __launch_bounds__(256) void tile_planes_f6_words_kernel(TileArgs a) {
  __shared__ uint32_t turn[4][64][33];              // [wave][contraction entry][output], one word of padding per row
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long grp = (long long)blockIdx.x * 4 + wave;
  if (grp * 64 >= a.n_threads) return;              // whole waves leave: no block-wide barrier below
  const int J = (int)(grp % a.ks);
  const int op = (int)((grp / a.ks) % a.OP);
  const int t = (int)(grp / ((long long)a.ks * a.OP));
  const int s = blockIdx.y;
  const int Lc = TRANSPOSED ? a.N : a.K;
  const int Lo = TRANSPOSED ? a.K : a.N;
  const int rows = min(a.tile, Lc - t * a.tile);
  if (J * 64 >= rows) return;                       // the contraction never reads this k-step
  const int c_first = t * a.tile + J * 64;          // first contraction index of the group
  const int c_count = min(64, rows - J * 64);       // entries beyond it are padding (zero codes)
  const int o_first = op * 32;
  const uint32_t* words = a.codes + (size_t)s * a.K * a.N;
  uint32_t (&mine)[64][33] = turn[wave];
  if (TRANSPOSED) {                                 // words[k = output][n = contraction]: a row of 64 entries per output
    for (int ol = 0; ol < 32; ++ol) {
      const int o = o_first + ol;
      mine[lane][ol] = (o < Lo && lane < c_count) ? words[(size_t)o * a.N + c_first + lane] : 0u;
    }
  } else {                                          // words[k = contraction][n = output]: two rows of 32 outputs at a time
    for (int cl = lane >> 5; cl < 64; cl += 2) {
      const int o = o_first + (lane & 31);
      mine[cl][lane & 31] = (o < Lo && cl < c_count) ? words[(size_t)(c_first + cl) * a.N + o] : 0u;
    }
  }
  wave_exchange();
  const int ol = lane & 31, half = lane >> 5;
  uint32_t rec[kMaxTermsF6][6];
#pragma unroll
  for (int j = 0; j < kMaxTermsF6; ++j)
#pragma unroll
    for (int x = 0; x < 6; ++x) rec[j][x] = 0u;
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t word = mine[w * 16 + half * 8 + e][ol];
      const int code_at = 8 * w + 2 * (e & 3) + (e >> 2);   // place of this entry among the lane's 32 codes
      const int bit = 6 * code_at, x = bit >> 5, sh = bit & 31;
#pragma unroll
      for (int j = 0; j < kMaxTermsF6; ++j) {
        if (j >= a.terms) break;
        const uint32_t code = (word >> (6 * j)) & 63u;
        rec[j][x] |= code << sh;
        if (sh > 26) rec[j][x + 1] |= code >> (32 - sh);
      }
    }
  const size_t frag0 = (((size_t)t * a.OP + op) * a.S_w + s) * a.terms * a.ks + J;
  uint8_t* base = reinterpret_cast<uint8_t*>(a.planes);
#pragma unroll
  for (int j = 0; j < kMaxTermsF6; ++j) {
    if (j >= a.terms) break;
    uint8_t* frag = base + (frag0 + (size_t)j * a.ks) * 1536;
    *reinterpret_cast<u32x4*>(frag + lane * 16) = u32x4{rec[j][0], rec[j][1], rec[j][2], rec[j][3]};
    *reinterpret_cast<u32x2*>(frag + 1024 + lane * 8) = u32x2{rec[j][4], rec[j][5]};
  }
}

// 32 values as E2M3 numbers of unit `scale` (a power of two; nearest, ties to even, saturating), one 6-bit code after the other,
// and back: value i < 16 is code 2 i, value 16 + i code 2 i + 1.  Inline because the instructions write their result while
// they still read, and the builtins of this compiler let it share registers with the sources; the wait states cover what the
// compiler would know of a builtin.
typedef float float32v __attribute__((ext_vector_type(32)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));

__device__ __forceinline__ u32x6 e2m3_codes(const float16v& even, const float16v& odd, float scale) {
  u32x6 r;
  asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3\n\ts_nop 1" : "=&v"(r) : "v"(even), "v"(odd), "s"(scale));
  return r;
}

__device__ __forceinline__ float32v e2m3_values(const u32x6& codes, float scale) {
  float32v r;
  asm("v_cvt_scalef32_pk32_f32_fp6 %0, %1, %2\n\ts_nop 1" : "=&v"(r) : "v"(codes), "s"(scale));
  return r;
}

// Plane value as a whole number of 2^(x0 - kTermGrid), x0 the exponent of the first term: towards zero, and odd unless exact.
// The midpoints between the numbers that a term can take are even on this grid (those of the last of five terms, two apart at
// least), so the terms of the result are the terms of the value itself.  Beyond 15 units of the first term all of them saturate:
// what is larger, infinite or no number becomes that.
constexpr int kTermGrid = 24;

__device__ __forceinline__ int on_term_grid(double u, int x0) {
  const double most = 15.0 * (1 << kTermGrid), y = ::fmin(::fabs(u) * __hiloint2double((1023 + kTermGrid - x0) << 20, 0), most);
  uint32_t whole = (uint32_t)y;
  whole |= (double)whole != y ? 1u : 0u;
  return __double2hiint(u) < 0 ? -(int)whole : (int)whole;
}

// Where tile_f6_kernel gets its term codes from.
constexpr int kFromDigits = 0;    // ideal arrays: the plane value is the digit
constexpr int kFromTable = 1;     // single-path wire model alone: looked up by (sign, digit, place in the array)
constexpr int kFromDevices = 2;   // anything else: every device of the patch computed

// Planes in the 6-bit format, both copies at once, for arrays of whole 64-row and 64-column steps: a block owns 64 x 64
// weights and two slices at a time, gets the plane values (devices: two single-precision words) or term codes (table,
// digits: one word) of every one of them once, into LDS, and its waves pack the records of the 2 x 2 fragments per slice that
// either direction reads, each lane one 24-byte record per term.  Devices: bound by the double-precision arithmetic of the normal
// numbers and the wire model (one Philox block for the four devices of a slice pair); each weight is quantised once per slice
// pair.  The terms of 32 values come out of the conversion instructions a record at a time, twice (either direction), which is
// a tenth of the integer work of finding every value's term codes and picking the records' bits from them: 4096 x 4096 weights
// with variation, 8 slices, 5 terms, 1485 -> 1197 us, and 1658 -> 1485 with the shorter normal numbers; 1133 -> 1000 with the
// constants of the normal numbers and the Philox keys in scalar registers.
template <int SRC, int NPOL, int NTH>
__global__ __launch_bounds__(NTH, 4) void tile_f6_kernel(BothCopies b, int turns) {
  constexpr int SL = NPOL == 2 ? 1 : 2;              // slices per turn: as many words in LDS either way
  constexpr int WORDS = SRC == kFromDevices ? 2 : 1; // plane values in two single-precision words, or term codes
  __shared__ uint32_t words[WORDS][NPOL][SL][64][65];   // [word][array][slice of the turn][k][n]
  const TileArgs& a = b.a;
  constexpr int NW = NTH / 64, PER = 64 / NW;        // waves; weights per thread
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k0 = (int)(blockIdx.x / b.nb) * 64, n0 = (int)(blockIdx.x % b.nb) * 64;
  const int n = n0 + lane;
  const uint32_t dmask = (1u << a.slice_bits) - 1;
  const int i0 = k0 % a.R, j = n0 % a.C + lane;      // place in the array: whole steps of 64 do not straddle arrays
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
  const uint32_t key0 = rng.k0, key1 = rng.k1;
  int q[PER];
  if constexpr (SRC != kFromDevices) {
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int k = k0 + wave + NW * r;
      q[r] = k < a.K && n < a.N ? quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w) : 0;
    }
  }
  for (int turn = (int)blockIdx.y * turns; turn < ((int)blockIdx.y + 1) * turns; ++turn) {
    const int s0 = SL * turn, ns = min(SL, a.S_w - s0);
    if (ns <= 0) return;
    if (turn != (int)blockIdx.y * turns) __syncthreads();   // everyone has packed the previous turn
    if constexpr (SRC == kFromDevices) {
#pragma unroll 1
      for (int r = 0; r < PER; ++r) {
        const int kl = wave + NW * r, k = k0 + kl;
        const bool real = k < a.K && n < a.N;
        const int w = real ? quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w) : 0;
        const int sign = (w > 0) - (w < 0);
        const uint32_t mag = (uint32_t)::abs(w);
        // the keys of the ten Philox rounds are made anew by scalar additions: kept across the loop they outgrow the scalar
        // registers and come back from vector registers one by one
        uint32_t first = __builtin_amdgcn_readfirstlane(key0), second = __builtin_amdgcn_readfirstlane(key1);
        asm volatile("" : "+s"(first), "+s"(second));
        rng.k0 = first;
        rng.k1 = second;
#pragma unroll
        for (int sl = 0; sl < SL; ++sl) {
          double u[NPOL];
#pragma unroll
          for (int pol = 0; pol < NPOL; ++pol) u[pol] = 0.0;
          if (real && sl < ns)
            plane_values<NPOL>(a, rng, sign, (int)((mag >> (a.slice_bits * (s0 + sl))) & dmask), s0 + sl, k, n, i0 + kl, j, u);
#pragma unroll
          for (int pol = 0; pol < NPOL; ++pol) {
            const int whole = on_term_grid(u[pol], a.term_exp[0]), low = whole & 31, high = (whole & ~31) | (low ? 16 : 0);
            words[0][pol][sl][kl][lane] = __builtin_bit_cast(uint32_t, (float)high);
            words[WORDS - 1][pol][sl][kl][lane] = __builtin_bit_cast(uint32_t, (float)(whole - high));
          }
        }
      }
    } else {
#pragma unroll
      for (int sl = 0; sl < SL; ++sl)
#pragma unroll
        for (int r = 0; r < PER; ++r) {
          const int kl = wave + NW * r;
          const uint32_t digit = ((uint32_t)::abs(q[r]) >> (a.slice_bits * (s0 + sl))) & dmask;   // zero beyond K, N and S_w
          uint32_t word = 0;                         // both devices of the pair in the same state: exactly zero
          if constexpr (SRC == kFromTable) {
            if (digit) word = a.codes[((size_t)((q[r] < 0 ? dmask : 0u) + digit - 1) * a.R + i0 + kl) * a.C + j];
          } else {
            word = term_codes(q[r] < 0 ? -(double)digit : (double)digit, 1, a.term_exp);
          }
          words[0][0][sl][kl][lane] = word;
        }
    }
    __syncthreads();
    const int ol = lane & 31, half = lane >> 5;
    if constexpr (SRC == kFromDevices) {
      // one wave per fragment group = (array, slice, direction, half of 32 outputs): a lane reads the 32 plane values of its
      // record and takes the terms off them one after the other, all exact in single precision: the first words are whole
      // multiples of 16 on the terms' grid below 2^28 (odd multiples where the second word is not zero, so that they lie on no
      // midpoint of the first two terms), and the second words join when at most 2^18 is left of a value in range.
#pragma unroll 1
      for (int grp = wave; grp < 8; grp += NW) {
        const int hh = grp & 1, dir = (grp >> 1) & 1, sl = NPOL == 2 ? 0 : grp >> 2, pol = NPOL == 2 ? grp >> 2 : 0;
        const int op = ((dir ? k0 : n0) >> 5) + hh, c = dir ? n0 : k0;
        if (sl >= ns || op >= b.OP[dir]) continue;
        const int t = c / b.tile[dir], J = (c - t * b.tile[dir]) >> 6;
        const uint32_t* from = &words[0][pol][sl][0][0] + (dir ? (32 * hh + ol) * 65 + half * 8 : 32 * hh + ol + half * 8 * 65);
        const uint32_t* second = from + (&words[WORDS - 1][0][0][0][0] - &words[0][0][0][0][0]);
        const int stride = dir ? 1 : 65;
        float16v left[2];                            // rows 16 w + e of the half's eights at 4 w + e, rows 16 w + 4 + e in the other
#pragma unroll
        for (int x = 0; x < 32; ++x) left[(x >> 2) & 1][4 * (x >> 3) + (x & 3)] = __builtin_bit_cast(float, from[(16 * (x >> 3) + (x & 7)) * stride]);
        uint8_t* at = b.base[dir] + (size_t)pol * b.pol_bytes[dir] +
                      ((((size_t)t * b.OP[dir] + op) * a.S_w + s0 + sl) * a.terms * b.ks[dir] + J) * 1536;
#pragma unroll 1
        for (int term = 0; term < a.terms; ++term, at += (size_t)b.ks[dir] * 1536) {
          const float scale = __builtin_bit_cast(float, (uint32_t)(127 + kTermGrid + a.term_exp[term] - a.term_exp[0]) << 23);
          if (term == 2) {
#pragma unroll
            for (int x = 0; x < 32; ++x) left[(x >> 2) & 1][4 * (x >> 3) + (x & 3)] += __builtin_bit_cast(float, second[(16 * (x >> 3) + (x & 7)) * stride]);
          }
          const u32x6 rec = e2m3_codes(left[0], left[1], scale);
          *reinterpret_cast<u32x4*>(at + lane * 16) = u32x4{rec[0], rec[1], rec[2], rec[3]};
          *reinterpret_cast<u32x2*>(at + 1024 + lane * 8) = u32x2{rec[4], rec[5]};
          const float32v v = e2m3_values(rec, scale);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            left[0][i] -= v[2 * i];
            left[1][i] -= v[2 * i + 1];
          }
        }
      }
    } else {
      // one wave per (fragment group, term): a short loop over the lane's 32 codes of one term
#pragma unroll 1
      for (int item = wave; item < 8 * a.terms; item += NW) {
        const int term = item >> 3, grp = item & 7;
        const int hh = grp & 1, dir = (grp >> 1) & 1, sl = grp >> 2;
        const int op = ((dir ? k0 : n0) >> 5) + hh, c = dir ? n0 : k0;
        if (sl >= ns || op >= b.OP[dir]) continue;
        const int t = c / b.tile[dir], J = (c - t * b.tile[dir]) >> 6;
        const uint32_t* from = &words[0][0][sl][0][0] + (dir ? (32 * hh + ol) * 65 + half * 8 : 32 * hh + ol + half * 8 * 65);
        const int stride = dir ? 1 : 65, from_bit = 6 * term;
        uint32_t rec[6];
#pragma unroll
        for (int x = 0; x < 6; ++x) rec[x] = 0u;
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t code = (from[(w * 16 + e) * stride] >> from_bit) & 63u;
            const int bit = 6 * (8 * w + 2 * (e & 3) + (e >> 2)), x = bit >> 5, sh = bit & 31;   // place among the lane's 32 codes
            rec[x] |= code << sh;
            if (sh > 26) rec[x + 1] |= code >> (32 - sh);
          }
        uint8_t* at = b.base[dir] + (((((size_t)t * b.OP[dir] + op) * a.S_w + s0 + sl) * a.terms + term) * b.ks[dir] + J) * 1536;
        *reinterpret_cast<u32x4*>(at + lane * 16) = u32x4{rec[0], rec[1], rec[2], rec[3]};
        *reinterpret_cast<u32x2*>(at + 1024 + lane * 8) = u32x2{rec[4], rec[5]};
      }
    }
  }
}

// Term codes of the plane value of every (sign, digit, row, column): one thread per (digit, row, column)
// computes the value with the arithmetic of plane_values, splits it into the terms of the schedule and
// writes both signs, and with `both` the second orientation.
__global__ __launch_bounds__(256) void code_table_kernel(TileArgs a, uint32_t* table, int both) {
  const int nd = (1 << a.slice_bits) - 1;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= nd * a.R * a.C) return;
  const int j = idx % a.C, i = (idx / a.C) % a.R, digit = idx / (a.C * a.R) + 1;
  NormalStream rng(a.seed, kStreamVariation, 0);    // not drawn from: the table exists without variation only
  const size_t words = (size_t)2 * nd * a.R * a.C;
#pragma unroll
  for (int neg = 0; neg < 2; ++neg) {
    double u[1];
    plane_values<1>(a, rng, neg ? -1 : 1, digit, 0, i, j, i, j, u);
    const uint32_t word = term_codes(u[0], a.terms, a.term_exp);
    const size_t plane = (size_t)(neg * nd + digit - 1) * a.R * a.C;
    table[plane + (size_t)i * a.C + j] = word;
    if (both) table[words + plane + (size_t)j * a.R + i] = word;
  }
}

// Planes in the 6-bit format from the table of term codes: the thread mapping and the records of
// tile_planes_f6_kernel; a plane value is one table word, looked up by (sign, digit, place in the array).
template <bool TRANSPOSED>
__global__ __launch_bounds__(256) void tile_planes_f6_table_kernel(TileArgs a) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= a.n_threads) return;
  const int out_len_pad = a.OP * 32;
  const int o = (int)(tid % out_len_pad);
  const int cg = (int)(tid / out_len_pad);
  const int slots = a.ks * 8;
  const int t = cg / slots, slot = cg - t * slots;
  const int within = slot * 8;
  const int Lc = TRANSPOSED ? a.N : a.K;
  const int Lo = TRANSPOSED ? a.K : a.N;
  const int rows = min(a.tile, Lc - t * a.tile);
  const int J = within >> 6;
  if (J * 64 >= rows) return;
  const int w = (within & 63) >> 4, half = (within & 15) >> 3;
  const int lane = (o & 31) + 32 * half;
  const int op = o >> 5;
  const int c0 = t * a.tile + within;
  const uint32_t dmask = (1u << a.slice_bits) - 1;
  const int nd = (int)dmask;
  // table of this orientation: [sign][digit - 1][contraction place][output place]
  const int out_len = TRANSPOSED ? a.R : a.C;       // places along the output index
  const uint32_t* codes = a.codes + (size_t)within * out_len + o % out_len;
  const size_t plane_words = (size_t)a.R * a.C;
  uint32_t mag[8];                                  // 0 for padding
  int first[8];                                     // table plane of digit 1 with the sign of the weight
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    mag[e] = 0;
    first[e] = 0;
    if (within + e >= rows || o >= Lo) continue;
    const int c = c0 + e;
    const int k = TRANSPOSED ? o : c, n = TRANSPOSED ? c : o;
    const int q = quantized_weight(a.W[(size_t)k * a.N + n], (double)a.w_max, a.qw, a.q_per_w);
    mag[e] = (uint32_t)::abs(q);
    first[e] = q < 0 ? nd : 0;
  }
  uint8_t* base = reinterpret_cast<uint8_t*>(a.planes);
  const int s_end = min(a.S_w, ((int)blockIdx.y + 1) * a.spt);
  for (int s = (int)blockIdx.y * a.spt; s < s_end; ++s) {
    unsigned long long bits[kMaxTermsF6];
#pragma unroll
    for (int j = 0; j < kMaxTermsF6; ++j) bits[j] = 0ull;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int digit = (int)((mag[e] >> (a.slice_bits * s)) & dmask);
      if (!digit) continue;                          // both devices of the pair in the same state: exactly zero
      const uint32_t word = codes[(size_t)(first[e] + digit - 1) * plane_words + (size_t)e * out_len];
      const int nibble = 2 * (e & 3) + (e >> 2);     // where the input stage's byte e lands in the digit word
#pragma unroll
      for (int j = 0; j < kMaxTermsF6; ++j) {
        if (j >= a.terms) break;
        bits[j] |= (unsigned long long)((word >> (6 * j)) & 63u) << (6 * nibble);
      }
    }
    const size_t frag0 = (((size_t)t * a.OP + op) * a.S_w + s) * a.terms * a.ks + J;
#pragma unroll
    for (int j = 0; j < kMaxTermsF6; ++j) {
      if (j >= a.terms) break;
      uint8_t* frag = base + (frag0 + (size_t)j * a.ks) * 1536;
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const int off = 6 * w + 2 * h;
        uint8_t* dst = off < 16 ? frag + lane * 16 + off : frag + 1024 + lane * 8 + (off - 16);
        *reinterpret_cast<uint16_t*>(dst) = (uint16_t)(bits[j] >> (16 * h));
      }
    }
  }
}


// ---------------------------------------------------------------------------------------------
// sums of the quantised weights over rows and columns: what the digital correction of offset-binary
// inputs multiplies the half-range with (the digital side knows the programmed weights)
// ---------------------------------------------------------------------------------------------
struct SumArgs {
  const float* W;
  long long* colsum;   // [N] sum over k
  long long* rowsum;   // [K] sum over n
  int K, N, weight_bits;
  float w_max;
};

__global__ __launch_bounds__(256) void clear_sums_kernel(SumArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < a.N) a.colsum[i] = 0;
  if (i < a.K) a.rowsum[i] = 0;
}

// Block = 64 rows x 64 columns; wave w takes rows w, w + 4, ..: lane = column.  Integer atomics: the
// result does not depend on the order.
__global__ __launch_bounds__(256) void weight_sums_kernel(SumArgs a) {
  const int nb = (a.N + 63) / 64;
  const int k0 = (blockIdx.x / nb) * 64, n = (blockIdx.x % nb) * 64 + (threadIdx.x & 63);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double qw = (double)((1u << a.weight_bits) - 1);
  long long col = 0;
  for (int k = k0 + wave; k < min(k0 + 64, a.K); k += 4) {
    long long q = 0;
    if (n < a.N) q = (long long)::rint(clampd((double)a.W[(size_t)k * a.N + n] / (double)a.w_max, -1.0, 1.0) * qw);
    col += q;
    long long r = q;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) r += __shfl_xor(r, d, 64);
    if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long*>(&a.rowsum[k]), (unsigned long long)r);
  }
  if (n < a.N) atomicAdd(reinterpret_cast<unsigned long long*>(&a.colsum[n]), (unsigned long long)col);
}

// ---------------------------------------------------------------------------------------------
// input quantiser (Sec. IV: inputs are scaled and sent to the DAC)
// ---------------------------------------------------------------------------------------------
template <bool CONV>
__global__ __launch_bounds__(256) void quantize_input_kernel(QuantArgs a) {
  // one wave = 32 rows x one pair of k-steps (32 consecutive inputs of a row = one 128-byte line); a launch has
  // fewer than 2^32 threads, so 32 bits hold a wave's index, and its parts are scalar arithmetic (64-bit divisions per lane before:
  // layers of a ResNet-20 at batch 128 from images 21.8 us on average, now 18.9).  Steps that the last tile does not reach are not
  // written: the contraction reads those of the layer alone
  const int lane = threadIdx.x & 63;
  const uint32_t wv = blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (mp, t, jp)
  if ((long long)wv * 64 >= a.n_threads) return;
  const uint32_t npair = (uint32_t)(a.ks + 1) >> 1, mpu = wv / (uint32_t)a.pairs, rest = wv - mpu * (uint32_t)a.pairs, tu = rest / npair;
  const int jp = (int)(rest - tu * npair), t = (int)tu, mp = (int)mpu;
  const int m = mp * 32 + (lane & 31);
  u32x2* out = reinterpret_cast<u32x2*>(a.A);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = 2 * jp + h, lend = min(a.L, (t + 1) * a.tile);
    if (j >= a.ks || t * a.tile + j * 16 >= lend) break;
    const int l0 = t * a.tile + j * 16 + (lane >> 5) * 8;
    float x[8];
    u32x2 pos, neg;
    load_inputs8<CONV>(a, m, l0, lend, x);
    input_codes8(a, m, l0, lend, x, pos, neg);
    const size_t blk = ((size_t)mp * a.T + t) * a.ks + j;
    out[blk * 64 + lane] = pos;
    if (a.P == 2) out[((size_t)a.MP * a.T * a.ks + blk) * 64 + lane] = neg;
  }
}

struct FinishArgs {
  const void* part;
  float* out;
  long long n;   // M * Lout
  int nchunk, wide, Lout;
  double scale;
  const long long* wsum;   // offset-binary inputs: weight sum per output, else null
  double half_range;       //   and the half-range it is multiplied with
};

// V consecutive outputs per thread (V = 4 where the row length allows it: 16-byte loads).
template <int V>
__global__ __launch_bounds__(256) void vmm_finish_kernel(FinishArgs a) {
#pragma clang fp contract(off)   // product, product, difference: each rounded on its own
  const long long i = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * V;
  if (i >= a.n) return;
  long long sum[V];
#pragma unroll
  for (int v = 0; v < V; ++v) sum[v] = 0;
  for (int c = 0; c < a.nchunk; ++c) {
    if (a.wide) {
      const long long* src = reinterpret_cast<const long long*>(a.part) + (size_t)c * a.n + i;
      if constexpr (V == 4) {
        const longlong2 w0 = *reinterpret_cast<const longlong2*>(src), w1 = *reinterpret_cast<const longlong2*>(src + 2);
        sum[0] += w0.x; sum[1] += w0.y; sum[2] += w1.x; sum[3] += w1.y;
      } else {
        sum[0] += src[0];
      }
    } else {
      const int32_t* src = reinterpret_cast<const int32_t*>(a.part) + (size_t)c * a.n + i;
      if constexpr (V == 4) {
        const int4 w = *reinterpret_cast<const int4*>(src);
        sum[0] += w.x; sum[1] += w.y; sum[2] += w.z; sum[3] += w.w;
      } else {
        sum[0] += src[0];
      }
    }
  }
  float y[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    double r = (double)sum[v] * a.scale;
    if (a.wsum) r = r - (double)a.wsum[(i + v) % a.Lout] * a.half_range;
    y[v] = (float)r;
  }
  if constexpr (V == 4) *reinterpret_cast<float4*>(a.out + i) = make_float4(y[0], y[1], y[2], y[3]);
  else a.out[i] = y[0];
}

// ---------------------------------------------------------------------------------------------
// update model (Sec. IV-C)
// ---------------------------------------------------------------------------------------------
struct GradArgs {
  const float* X;   // [M][K], or the NHWC image with CONV
  const float* D;   // [M][N]
  float* part;      // [mchunks][K][N]
  int M, K, N, KB, NB, m_per_chunk;
  int total_wg, per_xcd;   // blocks of the launch; logical blocks per XCD (the grid is 8 x per_xcd)
  int tile_rows;           // grad_quads_kernel: rows of W per block
  int shares, partials;    // update_small_kernel: partial sums of a batch chunk (its k-steps in turn) and of the batch
  ConvGeom conv;
};

constexpr int kGradMS = 32;   // batch rows per LDS stage = two k-steps of the bf16 matrix instruction
constexpr int kGradKS = kGradMS / 16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// fp32 value as a leading bf16 and a bf16 residual (together 16 significant bits).
__device__ __forceinline__ void split_bf16(float x, __bf16& hi, __bf16& lo) {
  hi = (__bf16)x;
  lo = (__bf16)(x - (float)hi);
}

// 128 x 128 tile of X^T dY per block, 4 waves as 2 x 2, each wave 64 x 64 = 2 x 2 MFMA tiles of
// v_mfma_f32_32x32x16_bf16.  Both operands are split into two bf16 terms while they are staged into
// LDS and hi.hi + hi.lo + lo.hi is accumulated in fp32: three bf16 matrix instructions of 16 rows do
// the work of eight fp32 ones of 2 rows at a relative error near 2^-16 per product, far inside the
// tolerance of the update.  When the layer has at most 64 rows (SPLIT_K) or columns (SPLIT_N) the
// waves that would work on padding take a share of the batch rows instead and write a partial sum of
// their own.  CONV: X is an NHWC image and the patch rows are gathered on the fly.  (Layers whose rows are no whole quads.)
template <bool SPLIT_K, bool SPLIT_N, bool CONV>
__global__ __launch_bounds__(256, 2) void grad_gemm_kernel(GradArgs a) {
  // [term][group of 8 batch rows][column] -> 8 bf16 along the batch
  __shared__ bf16x8 xs[2][kGradMS / 8][128];
  __shared__ bf16x8 ds[2][kGradMS / 8][128];
  __shared__ ConvRow crow[2][kGradMS];               // patches of the rows of the stage being fetched
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave >> 1, wn = wave & 1;
  // consecutive block ids go to different XCDs; give each XCD a contiguous range of logical blocks, tiles
  // fastest, so that the tiles of one batch chunk (which read the same rows of X and dY) share one L2
  const int logical = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (logical >= a.total_wg) return;
  const int tile_id = logical % (a.KB * a.NB), chunk_id = logical / (a.KB * a.NB);
  const int kb = tile_id % a.KB, nb = tile_id / a.KB;
  const int k0 = kb * 128, n0 = nb * 128;
  const int m_begin = chunk_id * a.m_per_chunk;
  const int m_end = min(a.M, m_begin + a.m_per_chunk);
  constexpr int PARTS = (SPLIT_K ? 2 : 1) * (SPLIT_N ? 2 : 1);     // batch shares
  const int share = (SPLIT_K ? wk : 0) * (SPLIT_N ? 2 : 1) + (SPLIT_N ? wn : 0);
  const int koff = SPLIT_K ? 0 : wk * 64, noff = SPLIT_N ? 0 : wn * 64;
  float16v acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // staging: this thread fetches column (tid & 127) of half the rows of a stage: the groups of 8 rows
  // (tid >> 7), (tid >> 7) + 2, ...
  const int col = tid & 127, g_first = __builtin_amdgcn_readfirstlane(tid >> 7);   // the same for a whole wave
  float px[8 * kGradKS], pd[8 * kGradKS];
  int ckh = 0, ckw = 0, cc = 0;
  if (CONV) {                                        // the kernel position of this thread's column is fixed
    const int k = min(k0 + col, a.K - 1);
    cc = k % a.conv.C;
    ckw = (k / a.conv.C) % a.conv.KW;
    ckh = (k / a.conv.C) / a.conv.KW;
  }
  auto stage_rows = [&](int m0, int buf) {            // CONV: the first threads decompose the stage's rows
    if (CONV && tid < kGradMS) crow[buf][tid] = conv_row(a.conv, min(m0 + tid, a.M - 1));
  };
  // Loads without branches (a load behind a per-element bounds test costs two jumps and an execution-mask
  // round trip each): indices are clamped into the tensors here, and what lies outside is replaced by zero
  // where the values are used, one stage later, so that no load is waited for before the matrix instructions.
  const bool k_ok = k0 + col < a.K, n_ok = n0 + col < a.N;
  const int kc = min(k0 + col, a.K - 1), nc = min(n0 + col, a.N - 1);
  const long long conv_col = CONV ? ((long long)ckh * a.conv.W + ckw) * a.conv.C + cc : 0;
  uint32_t inside = 0;       // CONV: bit (q * 8 + e) set when that element of the fetched stage lies inside the image
  auto prefetch = [&](int m0, int buf) {
    // one 64-bit product per stage and operand; the row offsets are the same for every lane (scalar arithmetic)
    const float* xrow = a.X + (size_t)m0 * a.K + kc;
    const float* drow = a.D + (size_t)m0 * a.N + nc;
    const int last = a.M - 1 - m0;
    uint32_t in = 0;
#pragma unroll
    for (int q = 0; q < kGradKS; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int row = (g_first + 2 * q) * 8 + e;
        const int rc = min(row, last);
        if (CONV) {
          const ConvRow r = crow[buf][row];
          const int ih = r.ih0 + ckh, iw = r.iw0 + ckw;
          const bool ok = (ih >= 0) & (ih < a.conv.H) & (iw >= 0) & (iw < a.conv.W);
          px[q * 8 + e] = a.X[ok ? r.off + conv_col : 0];
          in |= (ok ? 1u : 0u) << (q * 8 + e);
        } else {
          px[q * 8 + e] = xrow[(size_t)rc * a.K];
        }
        pd[q * 8 + e] = drow[(size_t)rc * a.N];
      }
    inside = in;
  };
  int stage = 0;
  stage_rows(m_begin, 0);
  if (CONV) __syncthreads();
  prefetch(m_begin, 0);
  for (int m0 = m_begin; m0 < m_end; m0 += kGradMS, stage ^= 1) {
    if (m0 + kGradMS < m_end) stage_rows(m0 + kGradMS, stage ^ 1);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kGradKS; ++q) {
      bf16x8 xh, xl, dh, dl;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int row = (g_first + 2 * q) * 8 + e;
        const bool row_ok = m0 + row < m_end;
        const bool x_ok = row_ok & k_ok & (!CONV || ((inside >> (q * 8 + e)) & 1u) != 0);
        __bf16 h, l;
        split_bf16(x_ok ? px[q * 8 + e] : 0.0f, h, l);
        xh[e] = h; xl[e] = l;
        split_bf16((row_ok & n_ok) ? pd[q * 8 + e] : 0.0f, h, l);
        dh[e] = h; dl[e] = l;
      }
      xs[0][g_first + 2 * q][col] = xh;
      xs[1][g_first + 2 * q][col] = xl;
      ds[0][g_first + 2 * q][col] = dh;
      ds[1][g_first + 2 * q][col] = dl;
    }
    __syncthreads();
    if (m0 + kGradMS < m_end) prefetch(m0 + kGradMS, stage ^ 1);
#pragma unroll
    for (int ks = 0; ks < kGradKS; ++ks) {
      // batch shares: two shares alternate over the k-steps of a stage, four take one k-step in four
      if (PARTS == 2 && (ks & 1) != share) continue;
      if (PARTS == 4 && (ks & 3) != share) continue;
      const int g8 = 2 * ks + (lane >> 5);
      bf16x8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ah[i] = xs[0][g8][koff + 32 * i + (lane & 31)];
        al[i] = xs[1][g8][koff + 32 * i + (lane & 31)];
        bh[i] = ds[0][g8][noff + 32 * i + (lane & 31)];
        bl[i] = ds[1][g8][noff + 32 * i + (lane & 31)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
        }
    }
  }
  float* out = a.part + ((size_t)chunk_id * PARTS + share) * a.K * a.N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int k = k0 + koff + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int n = n0 + noff + j * 32 + (lane & 31);
        if (k < a.K && n < a.N) out[(size_t)k * a.N + n] = acc[i][j][r];
      }
}

// The same product for layers whose rows are whole quads (of inputs, or of channels of a pixel, and of columns).  A thread
// stages four columns of eight batch rows of either matrix, by eight 16-byte loads; what lies outside is read from zeros, which
// takes no selects behind the loads.  A block's tile has all columns of a layer of up to 64 (NJ x 32) and up to 192 rows of W
// (KW = 2: wave w contracts rows 32 w .. and 32 (w + 4) ..), so that little is staged for padding, else 128 x 128 (KW = 1, NJ = 4).
// G: groups of eight batch rows per stage, eight where the tile has at most 32 quads.  The partial sums are grad_gemm_kernel's, of
// the same batch rows in the same order: the same weights, bit for bit.  Bound by the latency of a stage: two or three blocks share
// a compute unit.  (256 registers at most, by the launch bounds: with more to have, the compiler keeps the sums in accumulation
// registers and copies them every stage.)
// us of a whole update against grad_gemm_kernel above: 144 x 16 weights from 128 images of 32 x 32 77.1 -> 30.8, 576 x 64 from 64 of
// 56 x 56 292 -> 120, 1152 x 128 from 28 x 28 141 -> 98, 2304 x 256 from 14 x 14 160 -> 114, 64 x 256, 200704 rows 81 -> 71, 4096 x 4096,
// 128 rows 127 -> 121.
constexpr int kQuadRows = 192;
typedef float float4v __attribute__((ext_vector_type(4)));
typedef const float4v __attribute__((address_space(1))) global_quad;
__device__ float4v g_zeros;
template <int KW, int NJ, int G, bool CONV>
__global__ __launch_bounds__(256, KW == 1 ? 2 : 3) void grad_quads_kernel(GradArgs a) {
  constexpr int kRows = G == 8 || KW == 1 ? 128 : kQuadRows;   // eight groups: at most 32 quads
  __shared__ bf16x8 xs[2][G][kRows];
  __shared__ bf16x8 ds[2][G][32 * NJ];
  __shared__ ConvRow crow[2][8 * G];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int logical = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);   // tiles of a batch chunk on one XCD, as above
  if (logical >= a.total_wg) return;
  const int tiles = a.KB * a.NB, part_id = logical / tiles, tile = logical - part_id * tiles, nb = tile / a.KB;
  const int k0 = (tile - nb * a.KB) * a.tile_rows, kt = min(a.tile_rows, a.K - k0), n0 = nb * 32 * NJ, nt = min(32 * NJ, a.N - n0);
  // A block's rows of the batch chunk: all of them, or of every 32 the first or the last 16 (grad_gemm_kernel's shares)
  const int chunk_id = a.shares == 2 ? part_id >> 1 : part_id, share = a.shares == 2 ? part_id & 1 : 0;
  const int m_begin = chunk_id * a.m_per_chunk, m_end = min(a.M, m_begin + a.m_per_chunk);
  const int rows = a.shares == 2 ? ((m_end - m_begin + 31) >> 5) << 4 : m_end - m_begin;
  auto row_of = [&](int r) __attribute__((always_inline)) { return m_begin + (a.shares == 2 ? ((r >> 4) << 5) + 16 * share + (r & 15) : r); };
  // this thread's quad of columns and group of rows
  const int xq = kt >> 2, quads = xq + (nt >> 2), g = tid / quads, q = tid - g * quads;
  const bool is_x = q < xq, works = g < G;
  const int col = 4 * (is_x ? q : q - xq);
  const float* from;
  int row_stride = 0, ckh = 0, ckw = 0;
  if (!is_x) {
    from = a.D + n0 + col;
    row_stride = a.N;
  } else if (CONV) {
    const int k = k0 + col, kk = k / a.conv.C;
    ckh = kk / a.conv.KW;
    ckw = kk - ckh * a.conv.KW;
    from = a.X + (((long long)ckh * a.conv.W + ckw) * a.conv.C + (k - kk * a.conv.C));
  } else {
    from = a.X + k0 + col;
    row_stride = a.K;
  }
  bf16x8* to = is_x ? &xs[0][works ? g : 0][col] : &ds[0][works ? g : 0][col];
  const int to_term = is_x ? G * kRows : G * 32 * NJ;
  float4v v[8];
  global_quad* zeros = (global_quad*)&g_zeros;
  auto patches_of = [&](int r0, int buf) __attribute__((always_inline)) {
    if (CONV && tid < 8 * G) crow[buf][tid] = conv_row(a.conv, min(row_of(r0 + tid), a.M - 1));
  };
  auto load = [&](int r0, int buf) __attribute__((always_inline)) {
    const int r8 = 8 * min(g, G - 1), m = row_of(r0 + r8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      long long off = (long long)(m + e) * row_stride;
      bool there = m + e < m_end;
      if (CONV) {
        const ConvRow r = crow[buf][r8 + e];
        const int ih = r.ih0 + ckh, iw = r.iw0 + ckw;
        const bool inside = (ih >= 0) & (ih < a.conv.H) & (iw >= 0) & (iw < a.conv.W);
        off = is_x ? r.off : off;
        there = there & (inside | !is_x);
      }
      v[e] = *(there ? (global_quad*)(from + off) : zeros);
    }
  };
  float16v acc[KW][NJ];
#pragma unroll
  for (int i = 0; i < KW; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  const int blocks = (kt + 31) >> 5;                 // of 32 rows of W
  patches_of(0, 0);
  if (CONV) __syncthreads();
  load(0, 0);
  int buf = 0;
  for (int r0 = 0; r0 < rows; r0 += 8 * G, buf ^= 1) {
    if (r0 + 8 * G < rows) patches_of(r0 + 8 * G, buf ^ 1);
    __syncthreads();                                 // everyone is done with the stage before
    if (works) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          __bf16 h, l;
          split_bf16(v[e][c], h, l);
          hi[e] = h;
          lo[e] = l;
        }
        to[c] = hi;
        to[to_term + c] = lo;
      }
    }
    __syncthreads();
    if (r0 + 8 * G < rows) load(r0 + 8 * G, buf ^ 1);
    if (wave < blocks) {
#pragma unroll
      for (int ks = 0; ks < G / 2; ++ks) {
        const int g8 = 2 * ks + (lane >> 5);
        bf16x8 bh[NJ], bl[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          bh[j] = ds[0][g8][32 * j + (lane & 31)];
          bl[j] = ds[1][g8][32 * j + (lane & 31)];
        }
#pragma unroll
        for (int i = 0; i < KW; ++i)
          if (wave + 4 * i < blocks) {
            const bf16x8 ah = xs[0][g8][32 * (wave + 4 * i) + (lane & 31)], al = xs[1][g8][32 * (wave + 4 * i) + (lane & 31)];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[j], acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[j], acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[j], acc[i][j], 0, 0, 0);
            }
          }
      }
    }
  }
  float* out = a.part + (size_t)part_id * a.K * a.N;
#pragma unroll
  for (int i = 0; i < KW; ++i)
    if (wave + 4 * i < blocks) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int k = k0 + 32 * (wave + 4 * i) + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n = n0 + 32 * j + (lane & 31);
          if (k < a.K && n < a.N) out[(size_t)k * a.N + n] = acc[i][j][r];
        }
    }
}

// Backward pass of a convolution layer: the crossbars give the error of every patch element
// (dXcol[M][K]); an input pixel collects, digitally, the errors of every patch it belongs to.
// The adding-up pass of a backward convolution: every input pixel gathers the patch errors that its
// places in the patches received, straight from the partial sums: the value of a patch entry is the one
// vmm_finish_kernel would store, and the entries of a pixel are added in single precision in the order
// (kernel row, kernel column).  The [M][K] matrix of patch errors is never written.
struct FinishCol2imArgs {
  FinishArgs f;      // f.out unused; f.n = M * K
  float* dX;         // NHWC
  ConvGeom conv;
  int K;
  long long n_img;
};

// V consecutive channels of a pixel per thread (V = 4 where the channel count allows it: 16-byte loads).  Bound by the
// loads in flight and by index arithmetic: only the kernel positions that a pixel has are visited (one division per axis, not
// two per position), the loads of three of them are issued before the first is used, and indices are 32-bit (a launch has
// fewer than 2^32 threads).  The layers of a ResNet-20 at batch 128: 21.0 us on average before, 17.1 now.
template <int V>
__global__ __launch_bounds__(256) void vmm_finish_col2im_kernel(FinishCol2imArgs a) {
#pragma clang fp contract(off)   // product, product, difference: each rounded on its own
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if ((long long)t * V >= a.n_img) return;
  const ConvGeom& g = a.conv;
  const uint32_t groups = (uint32_t)g.C / V, pixel = t / groups, row = pixel / (uint32_t)g.W, bu = row / (uint32_t)g.H;
  const int c = (int)(t - pixel * groups) * V, iw = (int)(pixel - row * (uint32_t)g.W), ih = (int)(row - bu * (uint32_t)g.H);
  const int oh0 = (int)((uint32_t)(ih + g.pad) / (uint32_t)g.stride), ow0 = (int)((uint32_t)(iw + g.pad) / (uint32_t)g.stride);
  const int kw0 = iw + g.pad - ow0 * g.stride;         // position kw0 + j stride is that of output column ow0 - j
  const int nkw = (g.KW + g.stride - 1) / g.stride;
  float sum[V];
#pragma unroll
  for (int v = 0; v < V; ++v) sum[v] = 0.0f;
  for (int kh = ih + g.pad - oh0 * g.stride, oh = oh0; kh < g.KH && oh >= 0; kh += g.stride, --oh) {
    if (oh >= g.OH) continue;
    const long long base = ((long long)bu * g.OH + oh) * g.OW * a.K + (long long)kh * g.KW * g.C + c;
    for (int j0 = 0; j0 < nkw; j0 += 3) {
      long long at[3], acc[3][V];
      bool has[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int kw = kw0 + (j0 + j) * g.stride, ow = ow0 - (j0 + j);
        has[j] = kw < g.KW && ow >= 0 && ow < g.OW;
        at[j] = has[j] ? base + (long long)ow * a.K + kw * g.C : 0;   // a position that is not there: any address
#pragma unroll
        for (int v = 0; v < V; ++v) acc[j][v] = 0;
      }
      for (int ch = 0; ch < a.f.nchunk; ++ch) {
        if (a.f.wide) {
          const long long* src = reinterpret_cast<const long long*>(a.f.part) + (size_t)ch * a.f.n;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int v = 0; v < V; v += 2) {
              if constexpr (V >= 2) {
                const longlong2 w = *reinterpret_cast<const longlong2*>(src + at[j] + v);
                acc[j][v] += w.x;
                acc[j][v + 1] += w.y;
              } else {
                acc[j][v] += src[at[j]];
              }
            }
          }
        } else {
          const int32_t* src = reinterpret_cast<const int32_t*>(a.f.part) + (size_t)ch * a.f.n;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            if constexpr (V == 4) {
              const int4 w = *reinterpret_cast<const int4*>(src + at[j]);
              acc[j][0] += w.x; acc[j][1] += w.y; acc[j][2] += w.z; acc[j][3] += w.w;
            } else {
              acc[j][0] += src[at[j]];
            }
          }
        }
      }
#pragma unroll
      for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          double y = (double)acc[j][v] * a.f.scale;
          if (a.f.wsum && has[j]) y = y - (double)a.f.wsum[(kh * g.KW + kw0 + (j0 + j) * g.stride) * g.C + c + v] * a.f.half_range;
          sum[v] += has[j] ? (float)y : 0.0f;          // adding +0 changes nothing: no sum here is ever -0
        }
    }
  }
  if constexpr (V == 4) {
    *reinterpret_cast<float4*>(a.dX + (size_t)t * 4) = make_float4(sum[0], sum[1], sum[2], sum[3]);
  } else {
    a.dX[t] = sum[0];
  }
}

struct WriteArgs {
  float* W;
  float* Gp;        // per-polarity device state (PAIR): positive device, in [0, 1]
  float* Gn;        //   negative device
  const float* part;
  long long n;      // K * N
  int mchunks;
  uint32_t flags;
  double w_max, grad_scale, lr, v, gamma;
  uint64_t seed, step;
  const unsigned long long* step_add;   // optional device counter added to step
};

// New state of one weight from its gradient: ideal change, non-linearity, noise (normal number z), clamp.
__device__ __forceinline__ float written_weight(const WriteArgs& a, float w, double grad, double z) {
  const double g = (double)w / a.w_max;
  const double delta = a.grad_scale * grad;
  double written = delta;
  if (a.flags & XBAR_NI_UPD_NL) {
    const double x = clampd(0.5 * (g + 1.0), 0.0, 1.0);
    const double change = -a.lr * delta;
    // one exponential for both directions: the lanes of a wave go either way, and with one in each branch it runs both
    const double factor = ::exp(-a.v * (change > 0.0 ? x : 1.0 - x));
    if (change > 0.0 || change < 0.0) written = delta * factor;
  }
  if (a.flags & XBAR_NI_UPD_NOISE) written += a.gamma * ::sqrt(::fabs(delta)) * z;
  return (float)(a.w_max * clampd(g - a.lr * written, -1.0, 1.0));
}

// The same write with the two devices of a weight as states of their own (a variant of Sec. IV-C's one
// conductance per weight; Sec. IV-A keeps positive and negative conductances in two arrays): half the ideal
// change to each, in opposite directions, each with the non-linearity at its own state and direction, a noise
// draw of its own (sigma = gamma sqrt(|delta| / 2), numbers 2 i and 2 i + 1 of the pair stream) and its own
// clamp to [0, 1]; W = w_max (gp - gn).
__device__ __forceinline__ float written_pair(const WriteArgs& a, float& gp, float& gn, double grad, const double (&z)[2]) {
  const double half = 0.5 * (a.grad_scale * grad);
  double state[2] = {(double)gp, (double)gn};
#pragma unroll
  for (int pol = 0; pol < 2; ++pol) {
    const double dir = pol == 0 ? -1.0 : 1.0;        // the positive device falls when the weight falls
    const double change = dir * a.lr * half;
    double written = half;
    if (a.flags & XBAR_NI_UPD_NL) {
      const double x = clampd(state[pol], 0.0, 1.0), factor = ::exp(-a.v * (change > 0.0 ? x : 1.0 - x));
      if (change > 0.0 || change < 0.0) written = half * factor;
    }
    if (a.flags & XBAR_NI_UPD_NOISE) written += a.gamma * ::sqrt(::fabs(half)) * z[pol];
    state[pol] = clampd(state[pol] + dir * a.lr * written, 0.0, 1.0);
  }
  gp = (float)state[0];
  gn = (float)state[1];
  return (float)(a.w_max * ((double)gp - (double)gn));
}

// Four consecutive weights per thread: 16-byte loads and stores where the layer's size allows them (VEC), and the
// four normal numbers of one Philox block, which is half the logarithms, roots and angles of drawing them one by
// one.  G thread groups of a block share its 1024 / G weights: group g adds up the batch partials g, g + G, ... and
// the first group adds the groups' sums and writes (fixed order: the result does not depend on scheduling).  Few
// partials or many weights: G = 1, every thread busy to the end -- the write is then bound by its double-precision
// arithmetic.  Many partials of few weights: G = 8 or 32 keeps enough loads in flight.
template <int G, bool VEC, bool PAIR>
__global__ __launch_bounds__(256) void update_write_kernel(WriteArgs a) {
  constexpr int Q = 256 / G;                         // quads of weights per block
  __shared__ double red[G > 1 ? G : 1][G > 1 ? 4 * Q : 1];
  const int quad = threadIdx.x % Q, grp = threadIdx.x / Q;
  const long long i = ((long long)blockIdx.x * Q + quad) * 4;
  const int live = (int)min(4ll, a.n - i);           // weights of this thread (may be negative)
  double grad[4] = {0.0, 0.0, 0.0, 0.0};
  if (live > 0) {
#pragma unroll 4
    for (int c = grp; c < a.mchunks; c += G) {
      const float* src = a.part + (size_t)c * a.n + i;
      float4 v;
      if (VEC) {
        v = *reinterpret_cast<const float4*>(src);
      } else {                                       // clamped, not skipped: no branch between the loads
        v.x = src[0];
        v.y = src[min(1, live - 1)];
        v.z = src[min(2, live - 1)];
        v.w = src[min(3, live - 1)];
      }
      grad[0] += (double)v.x;
      grad[1] += (double)v.y;
      grad[2] += (double)v.z;
      grad[3] += (double)v.w;
    }
  }
  if constexpr (G > 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) red[grp][4 * quad + e] = grad[e];
    __syncthreads();
    constexpr int W = 4 * Q;                         // weights of the block; 256 / W shares of the groups each
    if constexpr (G > 8) {
      const int w = threadIdx.x % W, share = threadIdx.x / W;
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < G * W / 256; ++g) s += red[share * (G * W / 256) + g][w];
      __syncthreads();
      red[share][w] = s;
      __syncthreads();
    }
    if (grp != 0) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < (G > 8 ? 256 / W : G); ++g) s += red[g][4 * quad + e];
      grad[e] = s;
    }
  }
  if (live <= 0) return;
  const bool noisy = (a.flags & XBAR_NI_UPD_NOISE) != 0;
  NormalStream rng(a.seed, PAIR ? kStreamWritePair : kStreamWrite, effective_step(a.step, a.step_add));
  if constexpr (!PAIR) {
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    if (noisy) rng.get4((uint64_t)i >> 2, z);
    float w[4];
    if (VEC) {
      const float4 v = *reinterpret_cast<const float4*>(a.W + i);
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = a.W[i + min(e, live - 1)];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = written_weight(a, w[e], grad[e], z[e]);
    if (VEC) {
      *reinterpret_cast<float4*>(a.W + i) = make_float4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < live) a.W[i + e] = w[e];
    }
  } else {
    double z[2][4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};   // numbers 2 i .. 2 i + 7
    if (noisy) {
      rng.get4((uint64_t)i >> 1, z[0]);
      rng.get4(((uint64_t)i >> 1) + 1, z[1]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e >= live) break;
      const double zz[2] = {z[e >> 1][2 * (e & 1)], z[e >> 1][2 * (e & 1) + 1]};
      float gp = a.Gp[i + e], gn = a.Gn[i + e];
      a.W[i + e] = written_pair(a, gp, gn, grad[e], zz);
      a.Gp[i + e] = gp;
      a.Gn[i + e] = gn;
    }
  }
}

// The whole update of a layer with few batch rows: a block owns 32 x 32 weights.  Its waves take one batch partial each, the
// same rows in the same order as grad_gemm_kernel's waves (split operands, v_mfma_f32_32x32x16_bf16), but straight from memory
// to the matrix instruction; the partials meet in LDS and are added up in double precision one after the other.  From five
// partials on update_write_kernel adds interleaved groups of them, so the weights are those of the two kernels bit for bit
// wherever sums of single-precision partials in double precision are exact (a weight's partials within about 2^28 of each other),
// and within the final rounding elsewhere.  One launch and short code instead of two kernels that are both latency: 256 x 256
// weights at batch 64 6.1 us instead of 10.5, 784 x 500 at batch 128 9.2 instead of 14.7.  E weights per thread: one where few
// blocks are to use the chip's lanes, four that share a Philox block where there are many.
template <int E, bool PAIR>
__global__ __launch_bounds__(1024 / E) void update_small_kernel(GradArgs a, WriteArgs w) {
  constexpr int WAVES = 16 / E;
  __shared__ float sums[WAVES][1024];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* xk = a.X + min((int)blockIdx.y * 32 + (lane & 31), a.K - 1);
  const float* dn = a.D + min((int)blockIdx.x * 32 + (lane & 31), a.N - 1);
  const int k = (int)blockIdx.y * 32 + (int)threadIdx.x * E / 32, n = (int)blockIdx.x * 32 + (int)threadIdx.x * E % 32;
  double grad[E];
#pragma unroll
  for (int e = 0; e < E; ++e) grad[e] = 0.0;
  float x[8], d[8];
  auto fetch = [&](int m0) __attribute__((always_inline)) {        // rows beyond the batch: its last one, not used
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const size_t m = (size_t)min(m0 + 8 * (lane >> 5) + e, a.M - 1);
      x[e] = xk[m * a.K];
      d[e] = dn[m * a.N];
    }
  };
  auto start = [&](int p) __attribute__((always_inline)) { return p / a.shares * a.m_per_chunk + p % a.shares * 16; };
  fetch(start(wave));
#pragma unroll 1
  for (int first = 0; first < a.partials; first += WAVES) {
    const int p = first + wave;
    if (p < a.partials) {
      const int end = min(a.M, (p / a.shares + 1) * a.m_per_chunk);
      float16v acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int m0 = start(p), next; m0 < end; m0 = next) {
        bf16x8 xh, xl, dh, dl;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool row_ok = m0 + 8 * (lane >> 5) + e < end;
          __bf16 h, l;
          split_bf16(row_ok ? x[e] : 0.0f, h, l);
          xh[e] = h; xl[e] = l;
          split_bf16(row_ok ? d[e] : 0.0f, h, l);
          dh[e] = h; dl[e] = l;
        }
        next = m0 + 16 * a.shares;
        fetch(next < end ? next : start(p + WAVES));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl, dh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh, dl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh, dh, acc, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) sums[wave][(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[r];
    }
    __syncthreads();
    for (int v = 0; v < min(WAVES, a.partials - first); ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) grad[e] += (double)sums[v][threadIdx.x * E + e];
    __syncthreads();
  }
  if (k >= a.K || n >= a.N) return;
  const bool noisy = (w.flags & XBAR_NI_UPD_NOISE) != 0;
  const uint64_t i = (uint64_t)k * a.N + n;
  NormalStream rng(w.seed, PAIR ? kStreamWritePair : kStreamWrite, effective_step(w.step, w.step_add));
  if constexpr (E == 4 && !PAIR) {                   // N a multiple of four
    double z[4] = {0.0, 0.0, 0.0, 0.0};
    if (noisy) rng.get4(i >> 2, z);
    float4 v = *reinterpret_cast<const float4*>(w.W + i);
    v.x = written_weight(w, v.x, grad[0], z[0]);
    v.y = written_weight(w, v.y, grad[1], z[1]);
    v.z = written_weight(w, v.z, grad[2], z[2]);
    v.w = written_weight(w, v.w, grad[3], z[3]);
    *reinterpret_cast<float4*>(w.W + i) = v;
  } else if constexpr (!PAIR) {
    const float before = w.W[i];
    double z = 0.0;
    if (noisy) z = rng.get(i);
    w.W[i] = written_weight(w, before, grad[0], z);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      float gp = w.Gp[i + e], gn = w.Gn[i + e];
      double z[2] = {0.0, 0.0};
      if (noisy) rng.pair(2 * (i + e), z[0], z[1]);
      w.W[i + e] = written_pair(w, gp, gn, grad[e], z);
      w.Gp[i + e] = gp;
      w.Gn[i + e] = gn;
    }
  }
}

// Weights whose batch partials one block's groups share: enough loads in flight for a layer with few weights
// and many partials (an early convolution: 2304 weights, 512 partials), every lane busy for one with many weights.
template <bool PAIR>
hipError_t launch_update_write(const WriteArgs& a, hipStream_t st) {
  const bool vec = a.n % 4 == 0;
  const long long quads = (a.n + 3) / 4;
  const int G = (a.mchunks <= 4 || quads >= 131072) ? 1 : (a.mchunks >= 64 && quads <= 8192) ? 32 : 8;
  const int Q = 256 / G;
  const dim3 grid((unsigned)((quads + Q - 1) / Q));
  void (*k)(WriteArgs);
  if (vec) k = G == 1 ? update_write_kernel<1, true, PAIR> : G == 8 ? update_write_kernel<8, true, PAIR> : update_write_kernel<32, true, PAIR>;
  else k = G == 1 ? update_write_kernel<1, false, PAIR> : G == 8 ? update_write_kernel<8, false, PAIR> : update_write_kernel<32, false, PAIR>;
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

struct PairInitArgs {
  const float* W;
  float* Gp;
  float* Gn;
  long long n;
  double w_max;
};

// A weight placed symmetrically about mid-range: gp = (1 + g) / 2, gn = (1 - g) / 2, g = clamp(W / w_max).
__global__ __launch_bounds__(256) void pair_init_kernel(PairInitArgs a) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.n) return;
  const double g = clampd((double)a.W[i] / a.w_max, -1.0, 1.0);
  a.Gp[i] = (float)(0.5 * (1.0 + g));
  a.Gn[i] = (float)(0.5 * (1.0 - g));
}

// ---------------------------------------------------------------------------------------------
// instrumentation: sustained matrix-instruction rate
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mfma_probe_kernel(float* out, int iters, int mode) {
  uint32_t x = threadIdx.x * 2654435761u + 12345u;
  union { half8 h; uint32_t u[4]; } ua, ub;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    // two fp16 values in [-4, 4) per word; sign, exponent and mantissa bits all toggle
    ua.u[i] = mode == 1 ? (x & 0x00010001u) : ((x & 0x83ff83ffu) | 0x3c003c00u);
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    ub.u[i] = (x & 0x83ff83ffu) | 0x3c003c00u;
  }
  float16v c0, c1;
#pragma unroll
  for (int r = 0; r < 16; ++r) c0[r] = c1[r] = 0.0f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(ub.h, ua.h, c0, 0, 0, 0);   // dense on A, sparse on B
      c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(ub.h, ua.h, c1, 0, 0, 0);
    }
  }
  float s = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += c0[r] + c1[r];
  out[blockIdx.x * 256 + threadIdx.x] = s;
}

// Same loop with the 8-bit integer instruction (32 x 32 x 32 per instruction, twice the products).
__global__ __launch_bounds__(256) void mfma_probe_i8_kernel(int* out, int iters, int mode) {
  uint32_t x = threadIdx.x * 2654435761u + 12345u;
  int4v a, b;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    a[i] = (int)(mode == 3 ? (x & 0x01010101u) : x);       // single-bit digits as in the emulation, or any bytes
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    b[i] = (int)x;
  }
  int16v c0, c1;
#pragma unroll
  for (int r = 0; r < 16; ++r) c0[r] = c1[r] = 0;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      c0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, a, c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, a, c1, 0, 0, 0);
    }
  }
  int s = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += c0[r] + c1[r];
  out[blockIdx.x * 256 + threadIdx.x] = s;
}

// The block-scaled 6-bit x 4-bit instruction alone: pseudo-random E2M3 codes, single-bit E2M1 digits.
__global__ __launch_bounds__(256) void mfma_probe_f6_kernel(float* out, int iters) {
  uint32_t x = threadIdx.x * 2654435761u + 12345u;
  int8v a = {0, 0, 0, 0, 0, 0, 0, 0}, b = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    a[i] = (int)x;
    x ^= x << 13; x ^= x >> 17; x ^= x << 5;
    if (i < 4) b[i] = (int)(x & 0x11111111u);
  }
  float16v c0, c1;
#pragma unroll
  for (int r = 0; r < 16; ++r) c0[r] = c1[r] = 0.0f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      c0 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c0, 2, 4, 0, 127 - 8, 0, 127);
      c1 = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c1, 2, 4, 0, 127 - 8, 0, 127);
    }
  }
  float s = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += c0[r] + c1[r];
  out[blockIdx.x * 256 + threadIdx.x] = s;
}

// The contraction kernel's own inner loop (vmm6_contract_adc: 4 terms, 128 rows, two row patches) on
// synthetic operands: plane fragments of 4 slices in LDS, digits rebuilt every 4 passes as in the kernel.
template <bool DO_ADC>
__global__ __launch_bounds__(256, 2) void contraction_loop_probe_kernel(float* out, int iters) {
  extern __shared__ u32x4 lds[];
  constexpr int SLICE = 4 * f6_term_stride(2);       // 12 KiB
  uint32_t x = (threadIdx.x + 977u * blockIdx.x) * 2654435761u + 777u;
  for (int i = threadIdx.x; i < 4 * SLICE / 16; i += 256) {
    u32x4 v;
    x ^= x << 13; x ^= x >> 17; x ^= x << 5; v.x = x;
    x ^= x << 13; x ^= x >> 17; x ^= x << 5; v.y = x;
    x ^= x << 13; x ^= x >> 17; x ^= x << 5; v.z = x;
    x ^= x << 13; x ^= x >> 17; x ^= x << 5; v.w = x;
    lds[i] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  u32x2 raw[2][8];
#pragma unroll
  for (int pm = 0; pm < 2; ++pm)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      x ^= x << 13; x ^= x >> 17; x ^= x << 5; raw[pm][j].x = x;
      x ^= x << 13; x ^= x >> 17; x ^= x << 5; raw[pm][j].y = x;
    }
  const char* xb = reinterpret_cast<const char*>(lds) + lane * 16;
  const char* yb = reinterpret_cast<const char*>(lds) + 1024 + lane * 8;
  // terms 2^0, 2^-6, 2^-11, 2^-16 as for the single-path wire model at the paper's parameters
  const int scale_lo = 127 | (121 << 8) | (116 << 16) | (111 << 24), scale_hi = 127;
  int4v dg[2][2];
  float16v acc0[2], acc1[2];
  uint32_t y[2][16];
#pragma unroll
  for (int pm = 0; pm < 2; ++pm)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc0[pm][r] = acc1[pm][r] = 0.0f;
      y[pm][r] = 0;
    }
  for (int it = 0; it < iters; ++it) {
    const int sl = (it & 1) * 2;
    if ((it & 1) == 0) {
#pragma unroll
      for (int pm = 0; pm < 2; ++pm) digit_codes_f4<2, false>(raw[pm], (it >> 1) & 3, 0x11111111u, dg[pm]);
    }
    vmm6_contract_adc<2, 2, 4, DO_ADC>(dg, xb + sl * SLICE, yb + sl * SLICE, acc0, acc1, 3.96875f, kMagic - 127.0f,
                                       kMagic + 127.0f, it & 15, y, scale_lo, scale_hi);
    vmm6_contract_adc<2, 2, 4, DO_ADC>(dg, xb + (sl + 1) * SLICE, yb + (sl + 1) * SLICE, acc1, acc0, 3.96875f,
                                       kMagic - 127.0f, kMagic + 127.0f, (it + 2) & 15, y, scale_lo, scale_hi);
    if (!DO_ADC)     // nothing consumes the sums in this variant: keep the compiler from dropping the instructions
      asm volatile("" ::"v"(acc0[0]), "v"(acc0[1]), "v"(acc1[0]), "v"(acc1[1]));
  }
  float s = 0.0f;
  uint32_t t = 0;
#pragma unroll
  for (int pm = 0; pm < 2; ++pm)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s += acc0[pm][r] + acc1[pm][r];
      t += y[pm][r];
    }
  out[blockIdx.x * 256 + threadIdx.x] = s + (float)t;
}

// ---------------------------------------------------------------------------------------------
// host dispatch
// ---------------------------------------------------------------------------------------------
thread_local hipEvent_t g_trace_before = nullptr, g_trace_after = nullptr;
thread_local const unsigned long long* g_step_source = nullptr;

__global__ void step_advance_kernel(unsigned long long* counter) { *counter += 1ull; }

// Scratch of xbar_fwd_static: one array per GPU that the library runs on, held until the process ends.
// The name is a host-side stand-in; host code uses the device address that hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[XBAR_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's copy of the scratch array (looked up once per device, with that device current).
int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return XBAR_EHIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return XBAR_EHIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return XBAR_OK;
}

// scattered: a convolution's backward pass, which gathers from the partial sums and never writes outputs directly.
VmmPlan plan_vmm(const xbar_config* c, const Derived& d, int M, int K, int N, bool transposed, bool scattered = false) {
  VmmPlan p;
  p.g = plane_geom(c, d, K, N, transposed);
  p.Lin = transposed ? N : K;
  p.Lout = transposed ? K : N;
  p.MP = cdiv(M, 32);
  const bool is_signed = transposed || (c->flags & XBAR_INPUT_SIGNED);
  p.offset = (is_signed && (c->flags & XBAR_INPUT_OFFSET)) ? 1 : 0;
  p.P = (is_signed && !p.offset) ? 2 : 1;
  p.VT = p.P * d.npol * p.g.T;
  // sum of the shift-and-add weights of one virtual tile
  unsigned long long wsum = 0;
  for (int s = 0; s < d.S_w; ++s)
    for (int b = 0; b < d.S_in; ++b) wsum += 1ull << (c->slice_bits * s + c->stream_bits * b);
  p.bias_per_vt = (uint32_t)((unsigned long long)kMagicBits * wsum);
  const unsigned long long per_vt = wsum * (unsigned long long)d.q_adc;
  const unsigned long long fit = per_vt ? ((1ull << 31) - 1) / per_vt : (1ull << 31);
  p.wide = fit < 1 ? 1 : 0;
  p.ks16 = p.g.tile / 16;
  // KiB of operand per slice and output patch in the LDS stage
  const int slice_kb = d.fmt == kFmtF6 ? d.terms * f6_term_stride(p.g.ks) / 1024 : d.terms * p.g.ks;
  p.sg = d.S_w;
  if (d.fmt == kFmtF6) {
    // all slices in one stage when they fit 72 KiB (two blocks of a compute unit share its 160 KiB); else as
    // many as fit 64 KiB, an even number (the pipelined path pairs them)
    const int fit_sg = d.S_w * slice_kb <= 72 ? d.S_w : std::max(1, 64 / slice_kb);
    if (fit_sg < d.S_w) p.sg = fit_sg >= 2 ? (fit_sg & ~1) : 1;
    p.lds_kb = p.sg * slice_kb;
  } else {
    p.lds_kb = std::max(slice_kb, std::min(d.S_w * slice_kb, 64));   // staged slice group, at most 64 KiB
  }
  p.lds_bytes = (size_t)p.lds_kb * 1024;
  // Sums beyond 32 bits: the software-pipelined path still serves with two 32-bit sums per output, one of the lower and one of
  // the upper slices, widened when the block is done -- if slices come in pairs and either sum holds a virtual tile at least.
  p.split_sg = 0;
  p.bias_split[0] = p.bias_split[1] = 0;
  unsigned long long fit_split = 0;
  if (p.wide && d.S_w % 2 == 0 && d.S_w > 2 && p.lds_kb / slice_kb >= 2) {
    const int low = (d.S_w / 2 + 1) & ~1;
    unsigned long long wg[2] = {0, 0};
    for (int s = 0; s < d.S_w; ++s)
      for (int b = 0; b < d.S_in; ++b) wg[s >= low] += 1ull << (c->slice_bits * (s >= low ? s - low : s) + c->stream_bits * b);
    fit_split = ((1ull << 31) - 1) / (std::max(wg[0], wg[1]) * (unsigned long long)d.q_adc);
    if (fit_split >= 1) {
      p.wide = 2;
      p.split_sg = low;
      for (int h = 0; h < 2; ++h) p.bias_split[h] = (uint32_t)((unsigned long long)kMagicBits * wg[h]);
    }
  }
  p.pm = (d.fmt == kFmtF6 || p.g.ks <= 8) ? 2 : 1;
  p.row_waves = std::min(4, std::max(1, cdiv(p.MP, p.pm)));
  p.MB = cdiv(p.MP, p.pm * p.row_waves);
  const int groups = p.g.OP * p.MB;
  // Chunks of the contraction: from as many as 4096 blocks down, the number that costs least in us.  A virtual tile takes a
  // block `tile_us` where two share a compute unit (128 rows, 64 passes of 16 6-bit instructions: 54; 64 rows, 8 passes of 16
  // fp16 ones: 8.5); blocks run in rounds of 512, `rounds_of` of them: half a round has its compute units to itself, the last one of
  // several overlaps those before it.  A chunk's partial sums take 9 ns per block of 256 x 32 words, written and read again.
  // Of 101 layers measured at every number of chunks this picks within 0.6 % of the best on average, 4096 blocks 4.9 %:
  // 784 x 500, 8-bit weights in 4-bit cycles, 20000 rows, 305 -> 222 us; 144 x 16, 131072 rows, 87 -> 70; 256 x 512, 50176
  // rows, 1-bit cycles, 721 -> 687; 3000 x 2000, 128 rows backward, 138 -> 103.
  int per = std::max(1, cdiv(p.VT, std::max(1, cdiv(4096, groups))));
  const unsigned long long held = p.wide == 2 ? fit_split : p.wide ? ~0ull : fit;   // virtual tiles in one sum
  const int shares = std::min(4 / p.row_waves, d.S_in);   // of the cycles, among waves that have no rows of their own
  p.a_bytes = align256((size_t)p.P * p.MP * p.g.T * p.ks16 * 512);
  auto part_bytes = [&](int n) {
    return align256((size_t)cdiv(p.VT, n) * M * p.Lout * (p.wide || (unsigned long long)n > held ? 8 : 4));
  };
  auto exchange_bytes = [&](int share) {   // LDS for the sums that a block's waves exchange
    return (size_t)p.row_waves * (share - 1) * (p.wide ? 2 : 1) * p.pm * 16 * 64 * sizeof(uint32_t);
  };
  {
    const int nk = d.fmt == kFmtF6 ? cdiv(std::min(p.g.tile, p.Lin), 64) : cdiv(std::min(p.g.tile, p.Lin), 16);
    const double work_us = d.S_w * d.S_in * p.pm * (0.175 + 0.0295 * d.terms * nk), tile_us = 1.5 + work_us / shares;
    const double sums_us = 0.0089 * p.pm * p.row_waves / 8.0 * (p.wide ? 2 : 1);
    auto rounds_of = [](double r) {
      if (r <= 1.0) return r <= 0.5 ? 0.62 : 1.0;
      return r >= 3.0 ? r + 0.45 : std::max(r + 0.45, std::min(std::ceil(r), r + 0.6));
    };
    // The single chunk of offset-binary inputs stores its sums too, yet is the better choice: with that charged, 47 of 70 random layers
    // whose chunks changed were slower by more than 1 % and 14 faster, all 4 % slower on average (314 x 129 weights, 256-row arrays,
    // 2-bit cycles, 62299 rows: 254 -> 317 us; 803 x 501, 4-bit cycles, 1457 rows backward: 44 -> 41).
    auto cost = [&](int n) {
      const double blocks = (double)cdiv(p.VT, n) * groups;
      return n * tile_us * rounds_of(blocks / 512.0) + (n < p.VT || scattered ? sums_us * blocks : 0.0);
    };
    // no more than the sums hold: widening them on the way costs more (256 x 2304, 12544 rows backward: 1445 -> 1493 us)
    const int most = (int)std::min<unsigned long long>((unsigned long long)p.VT, held);
    double best = cost(per);
    // of the numbers that give as many chunks the smallest costs least: some 2 sqrt(VT) numbers instead of VT
    for (int chunks = cdiv(p.VT, per); chunks > 1;) {
      const int n = cdiv(p.VT, chunks - 1);
      if (n > most) break;
      const double c_n = cost(n);
      if (c_n < best) { best = c_n; per = n; }
      chunks = cdiv(p.VT, n);
    }
    // Few rows: chunks of what the sums hold let waves without rows share the cycles, which sums that are widened on the way do not; they
    // leave more partial sums.  Either runs in rounds of the blocks that a compute unit holds, eight waves of them as far as LDS
    // goes: without sharing, the planes of a tile leave room for two or three waves unless they are small.  Us, widened / shared: signed
    // inputs, 64-row arrays, 8-bit converter, 4096 x 4096 weights, 16 rows: 807 / 365, 64: 842 / 434, 128: 1034 / 651; 4096 x 8192, 128-row
    // arrays, 64 rows: 917 / 575; ideal arrays (one term): 4096 x 4096, 64 rows: 247 / 284, 7131 x 1656, 9-bit, 9 rows: 172 / 230.
    // Of 100 random layers that have the choice none is 2.5 % slower than widened, those with wires are 1.7 times as fast.
    // No layer outgrows the static array, and partial sums stay below the planes that the pass reads.
    if ((unsigned long long)per > held && shares > 1) {
      const double rows = (double)M / (32 * p.pm * p.row_waves);     // of a block's, those that there are
      auto few_rows_us = [&](int n, int share) {
        const size_t lds = std::max(p.lds_bytes, exchange_bytes(share));
        const double blocks = (double)cdiv(p.VT, n) * groups;
        const int resident = std::min(8 / (p.row_waves * share), (int)(160 * 1024 / lds)), widened = share > 1 ? 0 : (int)((n - 1) / held);
        const double block_us = n * (1.5 + work_us / share) + (share > 1 ? 2.5 : 0.0);
        return block_us * blocks / (256.0 * resident) + (1 + widened) * (widened ? 2 : 1) * sums_us * rows * blocks;
      };
      const double widened_us = few_rows_us(per, 1), shared_us = few_rows_us((int)held, shares);
      const size_t more = part_bytes((int)held), less = part_bytes(per), fixed = XBAR_STATIC_SCRATCH_BYTES;
      best = widened_us;
      if (shared_us < widened_us &&
          (p.a_bytes + more <= fixed || ((transposed || p.a_bytes + less > fixed) && more <= std::max(less, p.g.bytes)))) {
        per = (int)held;
        best = shared_us;
      }
    }
    p.vt_planned = per;
    p.chunked_us = best;
  }
  // 32-bit sums hold `fit` virtual tiles: a chunk with more adds them to a 64-bit partial sum of its own in
  // between (no extra chunks, so no extra partial results for the adding-up pass to read, and no workspace that grows with
  // the tiles: 2907 x 1029 weights of 14 one-bit slices, 96-row arrays, 13-bit converter, 109547 rows: 1.6 GB instead of 28.6)
  p.flush_every = (unsigned long long)per > held ? (int)held : 0;
  p.nw = p.row_waves * (p.flush_every ? 1 : shares);   // sums that are widened on the way belong to one wave
  p.lds_bytes = std::max(p.lds_bytes, exchange_bytes(p.nw / p.row_waves));
  p.nchunk = cdiv(p.VT, per);
  p.vt_per_chunk = cdiv(p.VT, p.nchunk);                  // same number of chunks, evenly filled
  p.part_bytes = part_bytes(per);
  p.ws_bytes = p.a_bytes + p.part_bytes;
  p.narrow = (unsigned long long)p.VT <= fit ? 1 : 0;
  p.small = vmm_small_pays(p, d) ? 1 : 0;
  if (p.small) {
    // its sums, and those of a scattered pass behind them: the workspace may grow, but no layer that xbar_fwd_static holds
    // with several kernels outgrows the static array with one (32 rows of 140000 outputs of one 4-bit slice: 17.9 and 36.3 MB)
    const size_t need = align256(vmm_small_ws_bytes(p, d)) + align256((size_t)M * p.Lout * (p.narrow ? 4 : 8));
    if (need > std::max(p.ws_bytes, (size_t)XBAR_STATIC_SCRATCH_BYTES)) p.small = 0;
    else p.ws_bytes = std::max(p.ws_bytes, need);
  }
  return p;
}

struct UpdPlan {
  int KB, NB, mchunks, m_per_chunk, parts;   // parts: partial sums per batch chunk (padding waves reused)
  bool small;                                // one kernel for gradient and write (from matrices)
  size_t ws_bytes;
};

// One kernel for gradient and write: up to 1024 rows, 768 where a batch chunk has two partials (beyond, its waves take more
// rounds than two launches cost), up to 1024 blocks, with which all lanes are busy in either (2048 where few rows leave the
// write to dominate), and up to 2^19 rows x blocks, beyond which fetching every operand once per block costs more than the
// partial sums' way through memory.  Rows that are no whole quads take one weight per thread and draw every normal number's
// Philox block for itself: with few rows, where that is most of the work, up to 576 blocks.  Measured, us per call, two kernels
// / one: 256 x 256 weights, batch 64: 10.5 / 5.8, 1024: 14.4 / 10.9; 784 x 500, 128: 14.5 / 8.8, 1024: 29.4 / 20.2; 1024 x 1024, 64: 18.2 /
// 10.9, 512: 31.3 / 20.3; 784 x 1000, 640: 29.4 / 26.3, 896: 30.1 / 32.0; 6721 x 84, 1024: 32.4 / 39.0; 2048 x 1000, 64: 28.0 /
// 21.9, 512: 35.3 / 37.7; 916 x 919, 32: 16.1 / 17.9; 64 x 16, 768: 10.9 / 9.9, 1024: 10.3 / 11.7.  Of 7662 random layers inside the
// line without the product and the quads, 75 lost more than 3 % and up to 52 %; inside this one 17, up to 23 %.
bool update_is_small(int M, int K, int N) {
  const long long blocks = (long long)cdiv(K, 32) * cdiv(N, 32);
  if (M > (std::min(K, N) <= 64 ? 768 : 1024) || M * blocks > (1 << 19)) return false;
  return blocks <= (N % 4 == 0 ? (M <= 64 ? 2048 : 1024) : (M < 96 ? 576 : 1024));
}

UpdPlan plan_update(int M, int K, int N) {
  UpdPlan p;
  p.KB = cdiv(K, 128);
  p.NB = cdiv(N, 128);
  const int tiles = p.KB * p.NB;
  // two resident blocks per compute unit: more batch chunks only add partial sums (measured: 512 blocks beat 256, 1024, 2048)
  int want = std::max(1, cdiv(512, tiles));
  int per = std::max(kGradMS, cdiv(cdiv(M, want), kGradMS) * kGradMS);
  p.m_per_chunk = per;
  p.mchunks = cdiv(M, per);
  p.parts = (K <= 64 ? 2 : 1) * (N <= 64 ? 2 : 1);
  p.ws_bytes = align256((size_t)p.mchunks * p.parts * K * N * sizeof(float));
  p.small = update_is_small(M, K, N);
  return p;
}

hipError_t launch_vmm6(const VmmArgs& a, const VmmPlan& p, int terms, bool codes, hipStream_t st) {
  return terms == 5 ? launch_vmm_f6_b(a, p, terms, codes, st) : launch_vmm_f6_a(a, p, terms, codes, st);
}

hipError_t launch_vmm(const VmmArgs& a, const VmmPlan& p, int terms, bool codes, hipStream_t st) {
  return p.g.ks <= 8 ? launch_vmm_f16_a(a, p, terms, codes, st) : launch_vmm_f16_b(a, p, terms, codes, st);
}

int run_vmm(const xbar_config* cfg, const void* planes, const float* in, float* out, int M, int K, int N,
            float w_max, float in_scale, void* ws, size_t ws_bytes, int16_t* codes, void* stream, bool transposed,
            const ConvGeom* conv = nullptr, unsigned long long* hist = nullptr, const ConvGeom* scatter = nullptr) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(M, K, N))) return rc;
  if (!aligned16(planes) || !aligned16(in) || (!hist && !aligned16(out)) || !aligned16(ws)) return XBAR_EALIGN;
  if (codes && (reinterpret_cast<uintptr_t>(codes) & 1u)) return XBAR_EALIGN;
  if (!finite_pos(w_max) || !finite_pos(in_scale)) return XBAR_EINVAL;
  // DAC level table: with 1-bit cycles (the paper's streaming scheme) and a zero level at 0 V the
  // table is one factor on every current, which goes into the ADC gain.
  // Other tables run through the general kernel variants, one contraction per level.
  float dac_gain = 1.0f;
  bool level_table = false;
  if (cfg->flags & XBAR_DAC_LUT) {
    if (cfg->stream_bits == 1 && cfg->dac_lut[0] == 0.0f) dac_gain = cfg->dac_lut[1];
    else if (cfg->stream_bits <= 4) level_table = true;
    else return XBAR_ENOTSUP;                        // the table has 16 entries
  }
  const Derived d = derive(cfg);
  const VmmPlan p = plan_vmm(cfg, d, M, K, N, transposed, scatter != nullptr);
  // the statistics pass writes no partial sums: the staged input is all it needs
  if (ws_bytes < (hist ? p.a_bytes : p.ws_bytes)) return XBAR_EWORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const float adc_fs = transposed ? cfg->adc_fs_bwd : cfg->adc_fs_fwd;

  QuantArgs qa;
  qa.X = in;
  qa.A = reinterpret_cast<uint8_t*>(ws);
  qa.M = M; qa.L = p.Lin; qa.MP = p.MP; qa.T = p.g.T; qa.ks = p.ks16; qa.tile = p.g.tile; qa.P = p.P;
  qa.input_bits = cfg->input_bits;
  qa.offset = p.offset;
  qa.nibbles = d.fmt == kFmtF6 ? 1 : 0;
  qa.scale = in_scale;
  qa.inv_scale = in_scale > 1e-30f && in_scale < 1e30f ? 1.0f / in_scale : std::numeric_limits<float>::quiet_NaN();
  qa.pairs = (p.g.T - 1) * ((p.ks16 + 1) / 2) + cdiv(p.Lin - (p.g.T - 1) * p.g.tile, 32);
  qa.n_threads = (long long)p.MP * qa.pairs * 64;
  if (conv) qa.conv = *conv;
  const bool general = codes != nullptr || hist != nullptr || level_table || (cfg->flags & XBAR_ADC_CURVE) != 0;
  const bool small = p.small && !general;
  if (small) {
  } else if (conv) {
    hipLaunchKernelGGL(quantize_input_kernel<true>, dim3((unsigned)((qa.n_threads + 255) / 256)), dim3(256), 0, st, qa);
  } else {
    hipLaunchKernelGGL(quantize_input_kernel<false>, dim3((unsigned)((qa.n_threads + 255) / 256)), dim3(256), 0, st, qa);
  }
  if (!small && hipGetLastError() != hipSuccess) return XBAR_EHIP;

  const PlaneGeom gf = plane_geom(cfg, d, K, N, false);
  VmmArgs a;
  a.A = reinterpret_cast<const u32x2*>(ws);
  a.B = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(planes) + (transposed ? align256(gf.bytes) : 0));
  a.part = reinterpret_cast<char*>(ws) + p.a_bytes;
  a.codes = codes;
  a.hist = hist;
  a.adc_curve_on = (cfg->flags & XBAR_ADC_CURVE) ? 1 : 0;
  for (int i = 0; i < 17; ++i) a.adc_curve[i] = cfg->adc_curve[i];
  a.q_adc = (float)d.q_adc;
  a.inv_q_adc = 1.0f / (float)d.q_adc;
  a.dac_levels = level_table ? 1 << cfg->stream_bits : 0;
  // table entries are voltages over v_max; one input level is v_max / (2^stream_bits - 1)
  for (int i = 0; i < 16; ++i) a.dac_lut[i] = (float)((double)cfg->dac_lut[i] * (double)((1 << cfg->stream_bits) - 1));
  a.M = M; a.Lin = p.Lin; a.Lout = p.Lout; a.MP = p.MP; a.OP = p.g.OP; a.MB = p.MB; a.T = p.g.T; a.P = p.P;
  a.npol = d.npol; a.pol_stride = p.g.pol_bytes / 16;
  a.VT = p.VT; a.S_w = d.S_w; a.S_in = d.S_in; a.slice_bits = cfg->slice_bits; a.stream_bits = cfg->stream_bits;
  a.ks = p.g.ks; a.tile = p.g.tile; a.vt_per_chunk = p.vt_per_chunk; a.nchunk = p.nchunk; a.lds_kb = p.lds_kb;
  a.ks16 = p.ks16; a.sg = p.sg; a.row_waves = p.row_waves;
  a.scale_lo = a.scale_hi = 0;
  for (int j = 0; j < kMaxTermsF6; ++j) {
    const int byte = 127 + d.term_exp[j];
    if (j < 4) a.scale_lo |= byte << (8 * j);
    else a.scale_hi |= byte;
  }
  const bool split = p.wide == 2 && !general;
  a.split_sg = p.split_sg;
  a.flush_every = hist ? 0 : p.flush_every;            // the statistics pass keeps no sums
  a.direct = (p.nchunk == 1 && !p.offset && !scatter) ? 1 : 0;   // a scatter gathers from the partial sums
  a.total_wg = p.nchunk * p.g.OP * p.MB;
  a.per_xcd = cdiv(a.total_wg, 8);
  a.gain = (float)d.q_adc / adc_fs * dac_gain;
  a.clamp_lo = kMagic - (float)d.q_adc;
  a.clamp_hi = kMagic + (float)d.q_adc;
  a.bias_per_vt = split ? p.bias_split[0] : p.bias_per_vt;
  a.bias_high_per_vt = split ? p.bias_split[1] : 0;
  a.out = out;
  {
    const double lsb = (double)adc_fs / (double)d.q_adc;
    const double qa_max = (double)((1u << cfg->input_bits) - 1), qw_max = (double)((1u << cfg->weight_bits) - 1);
    a.scale = lsb * (double)in_scale * (double)w_max / (qa_max * qw_max);
    if (p.offset) a.scale = 2.0 * a.scale;           // coded value = (2 u - Qa) / Qa
  }
  hipEvent_t ev0 = g_trace_before, ev1 = g_trace_after;
  g_trace_before = g_trace_after = nullptr;
  const long long* wsum = nullptr;
  double half_range = 0.0;
  if (p.offset) {      // minus the half-range times the sum of the programmed weights of this output
    const long long* sums =
        reinterpret_cast<const long long*>(reinterpret_cast<const char*>(planes) + weight_sums_offset(cfg, d, K, N));
    wsum = transposed ? sums + N : sums;
    half_range = (double)in_scale * (double)w_max / (double)((1u << cfg->weight_bits) - 1);
  }
  if (ev0 && hipEventRecord(ev0, st) != hipSuccess) return XBAR_EHIP;
  void* small_part = nullptr;
  if (small) {
    SmallArgs sa;
    sa.v = a;
    sa.q = qa;
    sa.is_conv = conv ? 1 : 0;
    sa.narrow = p.narrow;
    sa.ws = ws;
    small_part = reinterpret_cast<char*>(ws) + align256(vmm_small_ws_bytes(p, d));
    sa.v.part = scatter ? small_part : nullptr;
    sa.wsum = wsum;
    sa.half_range = half_range;
    unsigned long long cycles = 0;
    // the 6-bit kernel takes cycles in pairs; one that is not there leaves the converter's constant
    for (int b = 0; b < (d.fmt == kFmtF6 ? (d.S_in + 1) / 2 * 2 : d.S_in); ++b) cycles += 1ull << (cfg->stream_bits * b);
    sa.bias_item = (uint32_t)((unsigned long long)kMagicBits * cycles);
    if (launch_vmm_small(sa, p, d, st) != hipSuccess) return XBAR_EHIP;
  } else if ((d.fmt == kFmtF6 ? launch_vmm6(a, p, d.terms, general, st) : launch_vmm(a, p, d.terms, general, st)) != hipSuccess)
    return XBAR_EHIP;
  if (ev1 && hipEventRecord(ev1, st) != hipSuccess) return XBAR_EHIP;
  if (hist) return XBAR_OK;

  if (small ? scatter != nullptr : !a.direct) {
    FinishArgs f;
    f.part = small ? small_part : a.part;
    f.out = out;
    f.n = (long long)M * p.Lout;
    f.nchunk = small ? 1 : p.nchunk;
    f.wide = small ? !p.narrow : p.wide != 0 || p.flush_every != 0;
    f.Lout = p.Lout;
    f.scale = a.scale;
    f.wsum = wsum;
    f.half_range = half_range;
    if (scatter) {     // backward convolution: out is the NHWC image of input errors
      FinishCol2imArgs fc;
      fc.f = f;
      fc.dX = out;
      fc.conv = *scatter;
      fc.K = p.Lout;
      fc.n_img = (long long)(M / (scatter->OH * scatter->OW)) * scatter->H * scatter->W * scatter->C;
      // 16-byte accesses: channels in fours (then K = kernel positions x channels is a multiple of 4 too)
      if (scatter->C % 4 == 0)
        hipLaunchKernelGGL(vmm_finish_col2im_kernel<4>, dim3((unsigned)((fc.n_img / 4 + 255) / 256)), dim3(256), 0, st, fc);
      else
        hipLaunchKernelGGL(vmm_finish_col2im_kernel<1>, dim3((unsigned)((fc.n_img + 255) / 256)), dim3(256), 0, st, fc);
    } else {
      if (f.n % 4 == 0)
        hipLaunchKernelGGL(vmm_finish_kernel<4>, dim3((unsigned)((f.n / 4 + 255) / 256)), dim3(256), 0, st, f);
      else
        hipLaunchKernelGGL(vmm_finish_kernel<1>, dim3((unsigned)((f.n + 255) / 256)), dim3(256), 0, st, f);
    }
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  }
  return XBAR_OK;
}


int run_update(const xbar_config* cfg, float* W, const float* X, const float* dY, int M, int K, int N, float w_max,
               float grad_scale, float lr, uint64_t step, void* ws, size_t ws_bytes, void* hip_stream, const ConvGeom* conv,
               float* Gp = nullptr, float* Gn = nullptr) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(M, K, N))) return rc;
  if (!aligned16(W) || !aligned16(X) || !aligned16(dY) || !aligned16(ws)) return XBAR_EALIGN;
  if ((Gp || Gn) && (!aligned16(Gp) || !aligned16(Gn))) return XBAR_EALIGN;
  if (!finite_pos(w_max) || !std::isfinite(grad_scale) || !std::isfinite(lr)) return XBAR_EINVAL;
  const UpdPlan p = plan_update(M, K, N);
  if (ws_bytes < p.ws_bytes) return XBAR_EWORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  GradArgs g;
  g.X = X; g.D = dY; g.part = reinterpret_cast<float*>(ws);
  g.M = M; g.K = K; g.N = N; g.KB = p.KB; g.NB = p.NB; g.m_per_chunk = p.m_per_chunk;
  WriteArgs w;
  w.W = W; w.Gp = Gp; w.Gn = Gn; w.part = g.part; w.n = (long long)K * N; w.mchunks = p.mchunks * p.parts; w.flags = cfg->flags;
  w.w_max = (double)w_max; w.grad_scale = (double)grad_scale; w.lr = (double)lr;
  w.v = (double)cfg->upd_nl_v; w.gamma = (double)cfg->upd_noise_gamma;
  w.seed = cfg->seed; w.step = step; w.step_add = current_step_source();
  if (!conv && p.small) {
    g.shares = p.parts > 1 ? 2 : 1;                  // a stage has two k-steps: of four shares two are empty
    g.partials = p.mchunks * g.shares;
    const dim3 grid((unsigned)cdiv(N, 32), (unsigned)cdiv(K, 32));
    // up to 256 blocks, one per compute unit, one weight per thread: sixteen waves share the latency (us, four weights / one:
    // 2400 x 40 weights, 150 blocks, batch 32: 6.1 / 5.9, 512: 13.5 / 9.0; 2400 x 96, 225 blocks: 6.0 / 6.2, 10.9 / 8.5; 2400 x 128,
    // 300 blocks: 7.1 / 8.7, 13.3 / 13.3)
    if (N % 4 == 0 && grid.x * grid.y > 256) {
      if (Gp) hipLaunchKernelGGL((update_small_kernel<4, true>), grid, dim3(256), 0, st, g, w);
      else hipLaunchKernelGGL((update_small_kernel<4, false>), grid, dim3(256), 0, st, g, w);
    } else {
      if (Gp) hipLaunchKernelGGL((update_small_kernel<1, true>), grid, dim3(1024), 0, st, g, w);
      else hipLaunchKernelGGL((update_small_kernel<1, false>), grid, dim3(1024), 0, st, g, w);
    }
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  if (N % 4 == 0 && (conv ? conv->C : K) % 4 == 0) {
    // Tiles of 128 columns also where one or two waves have rows of W to contract: us of a whole update, tiles of 128 / of 64 columns / the
    // kernel below, which shares the batch rows among the waves: 8 x 128 weights, 200704 rows 30.7 / 35.2 / 37.6, 32 x 128 33.7 / 38.0 / 39.3,
    // 16 x 256 x 12544 13.1 / 14.4 / 14.2, 64 x 256 x 200704 63 / 73 / 70, 64 x 4096 x 4096 29.9 / 33.7 / 32.5; the other way about 32 x 512 x 4096
    // 18.2 / 18.5 / 17.3, 32 x 1024 x 2048 18.6 / 19.0 / 17.8, 64 x 512 x 4096 23.8 / 24.3 / 22.8 (of 35 layers of up to 64 rows five, by 5 % at most)
    const bool wide = N > 64;
    const int tile_cols = wide ? 128 : 64;
    g.KB = cdiv(K, wide ? 128 : kQuadRows);
    g.NB = cdiv(N, tile_cols);
    g.tile_rows = cdiv(cdiv(K, g.KB), 32) * 32;
    g.shares = p.parts > 1 ? 2 : 1;                  // of four shares two are empty
    w.mchunks = p.mchunks * g.shares;
    g.total_wg = g.KB * g.NB * w.mchunks;
    g.per_xcd = cdiv(g.total_wg, 8);
    // stages of 64 rows where tiles are small and there are as many
    const int rows = g.m_per_chunk / g.shares, groups = (g.tile_rows + std::min(N, tile_cols)) / 4 <= 32 && rows % 64 == 0 ? 8 : 4;
    if (conv) g.conv = *conv;
    void (*k)(GradArgs);
    if (wide && groups == 8) k = conv ? grad_quads_kernel<1, 4, 8, true> : grad_quads_kernel<1, 4, 8, false>;
    else if (wide) k = conv ? grad_quads_kernel<1, 4, 4, true> : grad_quads_kernel<1, 4, 4, false>;
    else if (conv) k = N <= 32 ? (groups == 8 ? grad_quads_kernel<2, 1, 8, true> : grad_quads_kernel<2, 1, 4, true>)
                               : (groups == 8 ? grad_quads_kernel<2, 2, 8, true> : grad_quads_kernel<2, 2, 4, true>);
    else k = N <= 32 ? (groups == 8 ? grad_quads_kernel<2, 1, 8, false> : grad_quads_kernel<2, 1, 4, false>)
                     : (groups == 8 ? grad_quads_kernel<2, 2, 8, false> : grad_quads_kernel<2, 2, 4, false>);
    hipLaunchKernelGGL(k, dim3((unsigned)(g.per_xcd * 8)), dim3(256), 0, st, g);
  } else {
    g.total_wg = p.KB * p.NB * p.mchunks;
    g.per_xcd = cdiv(g.total_wg, 8);
    const dim3 grid((unsigned)(g.per_xcd * 8)), block(256);
    if (conv) {
      g.conv = *conv;
      if (K <= 64 && N <= 64) hipLaunchKernelGGL((grad_gemm_kernel<true, true, true>), grid, block, 0, st, g);
      else if (K <= 64) hipLaunchKernelGGL((grad_gemm_kernel<true, false, true>), grid, block, 0, st, g);
      else if (N <= 64) hipLaunchKernelGGL((grad_gemm_kernel<false, true, true>), grid, block, 0, st, g);
      else hipLaunchKernelGGL((grad_gemm_kernel<false, false, true>), grid, block, 0, st, g);
    } else {
      if (K <= 64 && N <= 64) hipLaunchKernelGGL((grad_gemm_kernel<true, true, false>), grid, block, 0, st, g);
      else if (K <= 64) hipLaunchKernelGGL((grad_gemm_kernel<true, false, false>), grid, block, 0, st, g);
      else if (N <= 64) hipLaunchKernelGGL((grad_gemm_kernel<false, true, false>), grid, block, 0, st, g);
      else hipLaunchKernelGGL((grad_gemm_kernel<false, false, false>), grid, block, 0, st, g);
    }
  }
  if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  if ((Gp ? launch_update_write<true>(w, st) : launch_update_write<false>(w, st)) != hipSuccess) return XBAR_EHIP;
  return XBAR_OK;
}

}  // namespace

namespace xbar_detail {
// Checks a convolution geometry and derives the layer's matrix shape: M = batch x output positions,
// K = kernel height x kernel width x input channels.
int conv_dims(const xbar_conv_geom* q, ConvGeom* g, int* M, int* K) {
  if (!q) return XBAR_EINVAL;
  if (q->batch <= 0 || q->in_h <= 0 || q->in_w <= 0 || q->in_c <= 0 || q->k_h <= 0 || q->k_w <= 0 || q->stride <= 0 ||
      q->pad < 0 || q->out_h <= 0 || q->out_w <= 0)
    return XBAR_ESHAPE;
  if (q->in_h + 2 * q->pad < q->k_h || q->in_w + 2 * q->pad < q->k_w) return XBAR_ESHAPE;
  if (q->out_h != (q->in_h + 2 * q->pad - q->k_h) / q->stride + 1 ||
      q->out_w != (q->in_w + 2 * q->pad - q->k_w) / q->stride + 1)
    return XBAR_ESHAPE;
  const long long m = (long long)q->batch * q->out_h * q->out_w, k = (long long)q->k_h * q->k_w * q->in_c;
  const long long pixels = (long long)q->batch * q->in_h * q->in_w * q->in_c;
  if (m >= (1ll << 31) || k >= (1ll << 31) || pixels >= (1ll << 38)) return XBAR_ESHAPE;
  g->H = q->in_h; g->W = q->in_w; g->C = q->in_c; g->KH = q->k_h; g->KW = q->k_w;
  g->stride = q->stride; g->pad = q->pad; g->OH = q->out_h; g->OW = q->out_w;
  *M = (int)m;
  *K = (int)k;
  return XBAR_OK;
}

const unsigned long long* current_step_source() { return g_step_source; }
}  // namespace xbar_detail

// ---------------------------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------------------------
extern "C" {

uint32_t xbar_abi_version(void) { return XBAR_ABI_VERSION; }

int xbar_probe_mfma_rate(int mode, int iters, void* out, size_t out_bytes, void* hip_stream) {
  if (mode < 0 || mode > 6 || iters <= 0 || iters > (1 << 24)) return XBAR_EINVAL;
  if (!aligned16(out)) return XBAR_EALIGN;
  if (out_bytes < (size_t)512 * 256 * sizeof(float)) return XBAR_EWORKSPACE;
  if (mode == 4) {
    hipLaunchKernelGGL(mfma_probe_f6_kernel, dim3(512), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<float*>(out), iters);
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  if (mode >= 5) {
    const size_t lds_bytes = 4 * 4 * f6_term_stride(2);
    if (mode == 5)
      hipLaunchKernelGGL(contraction_loop_probe_kernel<false>, dim3(512), dim3(256), lds_bytes,
                         reinterpret_cast<hipStream_t>(hip_stream), reinterpret_cast<float*>(out), iters);
    else
      hipLaunchKernelGGL(contraction_loop_probe_kernel<true>, dim3(512), dim3(256), lds_bytes,
                         reinterpret_cast<hipStream_t>(hip_stream), reinterpret_cast<float*>(out), iters);
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  if (mode >= 2) {
    hipLaunchKernelGGL(mfma_probe_i8_kernel, dim3(512), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<int*>(out), iters, mode);
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  hipLaunchKernelGGL(mfma_probe_kernel, dim3(512), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream),
                     reinterpret_cast<float*>(out), iters, mode);
  return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
}

float xbar_adc_range_from_histogram(const unsigned long long* hist, int bins, float bin_width, double quantile) {
  if (!hist || bins <= 0 || !finite_pos(bin_width) || !(quantile > 0.0) || quantile > 1.0) return 0.0f;
  double total = 0.0;
  for (int b = 0; b < bins; ++b) total += (double)hist[b];
  double cum = 0.0;
  int b = 0;
  for (; b < bins - 1; ++b) {
    cum += (double)hist[b];
    if (cum >= quantile * total) break;
  }
  const double current = std::max(((double)b + 0.5) * (double)bin_width, (double)bin_width);
  return (float)std::exp2(std::ceil(std::log2(current)));
}

int xbar_plane_format(const xbar_config* cfg, int* terms) {
  const int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  const Derived d = derive(cfg);
  if (terms) *terms = d.terms;
  return d.fmt;
}

void xbar_set_step_source(const unsigned long long* device_step) { g_step_source = device_step; }

int xbar_step_advance(unsigned long long* device_step, void* hip_stream) {
  if (!device_step || (reinterpret_cast<uintptr_t>(device_step) & 7u)) return XBAR_EALIGN;
  hipLaunchKernelGGL(step_advance_kernel, dim3(1), dim3(1), 0, reinterpret_cast<hipStream_t>(hip_stream), device_step);
  return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
}

void xbar_trace_next_vmm(void* before, void* after) {
  g_trace_before = reinterpret_cast<hipEvent_t>(before);
  g_trace_after = reinterpret_cast<hipEvent_t>(after);
}

const char* xbar_strerror(int code) {
  switch (code) {
    case XBAR_OK: return "ok";
    case XBAR_EINVAL: return "invalid parameter struct or scalar argument";
    case XBAR_ESHAPE: return "M, K, N must be positive, K*N below 2^31 and M*K, M*N below 2^38 elements";
    case XBAR_EALIGN: return "null or misaligned pointer (16 bytes required)";
    case XBAR_EWORKSPACE: return "workspace or plane buffer too small";
    case XBAR_EHIP: return "HIP kernel launch failed";
    case XBAR_ENOTSUP: return "not supported by the GPU kernels";
    case XBAR_ESCRATCH: return "shape needs more scratch memory than the library's static array holds (XBAR_STATIC_SCRATCH_BYTES)";
    default: return "unknown xbar status";
  }
}

int xbar_config_validate(const xbar_config* c) {
  if (!c) return XBAR_EINVAL;
  if (c->struct_size != sizeof(xbar_config) || c->abi_version != XBAR_ABI_VERSION) return XBAR_EINVAL;
  if (c->xbar_rows < 16 || c->xbar_rows > 256 || c->xbar_rows % 16) return XBAR_EINVAL;
  if (c->xbar_cols < 16 || c->xbar_cols > 256 || c->xbar_cols % 16) return XBAR_EINVAL;
  if (c->slice_bits < 1 || c->slice_bits > 4) return XBAR_EINVAL;
  if (c->weight_bits < 1 || c->weight_bits > 16 || c->weight_bits % c->slice_bits) return XBAR_EINVAL;
  if (c->input_bits < 1 || c->input_bits > 8) return XBAR_EINVAL;
  if (c->stream_bits < 1 || c->stream_bits > c->input_bits || c->input_bits % c->stream_bits) return XBAR_EINVAL;
  if (c->adc_bits < 2 || c->adc_bits > 16) return XBAR_EINVAL;
  if (c->flags & ~0x1FFFu) return XBAR_EINVAL;
  if ((c->flags & XBAR_PULSE_CODED) && (c->flags & XBAR_PULSE_MAGNITUDE)) return XBAR_EINVAL;   // one pulse coding
  if (c->flags & XBAR_ADC_PER_ARRAY) {
    if (c->flags & XBAR_ADC_CURVE) return XBAR_EINVAL;     // the curve is that of a signed converter
    if (c->adc_bits > 15) return XBAR_EINVAL;              // unsigned codes are reported as int16
  }
  if (c->flags & XBAR_ADC_CURVE)
    for (int i = 0; i < 17; ++i) {
      if (!std::isfinite(c->adc_curve[i]) || c->adc_curve[i] < -1.0f || c->adc_curve[i] > 1.0f) return XBAR_EINVAL;
      if (i && c->adc_curve[i] < c->adc_curve[i - 1]) return XBAR_EINVAL;     // a converter is monotone
    }
  {  // at most one wire model
    const uint32_t w = c->flags & (XBAR_NI_WIRE_AAM | XBAR_NI_WIRE_PROFILE | XBAR_NI_WIRE_AAM2);
    if (w & (w - 1)) return XBAR_EINVAL;
  }
  if (!finite_pos(c->r_min) || !finite_pos(c->r_max) || !(c->r_max > c->r_min)) return XBAR_EINVAL;
  if (!finite_pos(c->v_max)) return XBAR_EINVAL;
  if (!finite_nonneg(c->r_row) || !finite_nonneg(c->r_col) || !finite_nonneg(c->r_source) ||
      !finite_nonneg(c->r_sense))
    return XBAR_EINVAL;
  if (!finite_nonneg(c->var_sigma) || !finite_nonneg(c->upd_nl_v) || !finite_nonneg(c->upd_noise_gamma))
    return XBAR_EINVAL;
  if (!finite_pos(c->adc_fs_fwd) || !finite_pos(c->adc_fs_bwd)) return XBAR_EINVAL;
  if (c->flags & XBAR_DAC_LUT)
    for (int i = 0; i < (1 << c->stream_bits) && i < 16; ++i)
      if (!std::isfinite(c->dac_lut[i])) return XBAR_EINVAL;
  return XBAR_OK;
}

size_t xbar_planes_bytes(const xbar_config* cfg, int K, int N) {
  if (xbar_config_validate(cfg) || check_shape(1, K, N)) return 0;
  const Derived d = derive(cfg);
  return device_words_offset(cfg, d, K, N) + device_words_bytes(cfg, d, K, N);
}

size_t xbar_workspace_bytes(const xbar_config* cfg, int op, int M, int K, int N) {
  if (xbar_config_validate(cfg) || check_shape(M, K, N)) return 0;
  const Derived d = derive(cfg);
  if (op == XBAR_OP_FWD) return plan_vmm(cfg, d, M, K, N, false).ws_bytes;
  if (op == XBAR_OP_BWD) return plan_vmm(cfg, d, M, K, N, true).ws_bytes;
  if (op == XBAR_OP_UPDATE) return plan_update(M, K, N).ws_bytes;
  if (op == XBAR_OP_FCM) return fcm_workspace_bytes(cfg, K, N);
  if (op == XBAR_OP_UPDATE_PULSED) return pulsed_workspace_bytes(M, K, N);
  return 0;
}

int xbar_tile(const xbar_config* cfg, const float* W, int K, int N, float w_max, uint64_t step, const float* profile,
              void* planes, size_t planes_bytes, void* hip_stream) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(1, K, N))) return rc;
  if (!aligned16(W) || !aligned16(planes)) return XBAR_EALIGN;
  if ((cfg->flags & XBAR_NI_WIRE_PROFILE) && !aligned16(profile)) return XBAR_EALIGN;
  if (!finite_pos(w_max)) return XBAR_EINVAL;
  if (planes_bytes < xbar_planes_bytes(cfg, K, N)) return XBAR_EWORKSPACE;
  const Derived d = derive(cfg);
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  double* wire_u = nullptr;
  if (cfg->flags & XBAR_NI_WIRE_AAM2) {
    wire_u = reinterpret_cast<double*>(reinterpret_cast<char*>(planes) + align256(plane_geom(cfg, d, K, N, false).bytes) +
                                       align256(plane_geom(cfg, d, K, N, true).bytes));
    if ((rc = launch_wire_model(cfg, W, K, N, w_max, step, wire_u, st))) return rc;
  }
  if (cfg->flags & XBAR_INPUT_OFFSET) {
    SumArgs sa;
    sa.W = W;
    sa.colsum = reinterpret_cast<long long*>(reinterpret_cast<char*>(planes) + weight_sums_offset(cfg, d, K, N));
    sa.rowsum = sa.colsum + N;
    sa.K = K; sa.N = N; sa.weight_bits = cfg->weight_bits; sa.w_max = w_max;
    hipLaunchKernelGGL(clear_sums_kernel, dim3((unsigned)cdiv(std::max(K, N), 256)), dim3(256), 0, st, sa);
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
    hipLaunchKernelGGL(weight_sums_kernel, dim3((unsigned)(cdiv(K, 64) * cdiv(N, 64))), dim3(256), 0, st, sa);
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  }
  TileArgs a;
  a.W = W;
  a.profile = profile;
  a.codes = nullptr;
  a.wire_u = wire_u;
  a.K = K; a.N = N; a.R = cfg->xbar_rows; a.C = cfg->xbar_cols; a.S_w = d.S_w;
  a.slice_bits = cfg->slice_bits; a.terms = d.terms;
  a.flags = cfg->flags;
  a.g_min = 1.0 / (double)cfg->r_max;
  a.dg = (1.0 / (double)cfg->r_min - a.g_min) / (double)((1 << cfg->slice_bits) - 1);
  a.inv_dg = 1.0 / a.dg;
  a.var_sigma = (double)cfg->var_sigma;
  a.r_row = (double)cfg->r_row;
  a.r_col = (double)cfg->r_col;
  a.r_source = (double)cfg->r_source;
  a.r_sense = (double)cfg->r_sense;
  {  // |U| < 2^slice_bits: fp16 holds multiples of 2^-(11 - slice_bits) below that bound exactly; one
     // array alone adds the off-state conductance (below the full range for on/off ratios from 2): one bit less
    const int hi_frac = (d.npol == 2 ? 10 : 11) - cfg->slice_bits;
    a.hi_scale = std::ldexp(1.0, hi_frac);
    a.hi_inv_scale = std::ldexp(1.0, -hi_frac);
  }
  a.w_max = w_max;
  a.qw = (double)((1u << cfg->weight_bits) - 1);
  a.q_per_w = a.qw / (double)w_max;
  a.seed = cfg->seed;
  a.step = step;
  a.step_add = current_step_source();
  for (int j = 0; j < kMaxTermsF6; ++j) a.term_exp[j] = d.term_exp[j];

  uint8_t* at = reinterpret_cast<uint8_t*>(planes);
  PlaneGeom g[2] = {plane_geom(cfg, d, K, N, false), plane_geom(cfg, d, K, N, true)};
  BothCopies b;
  for (int dir = 0; dir < 2; ++dir) {
    b.base[dir] = at + (dir ? align256(g[0].bytes) : 0);
    b.OP[dir] = g[dir].OP; b.ks[dir] = g[dir].ks; b.tile[dir] = g[dir].tile; b.pol_bytes[dir] = g[dir].pol_bytes;
  }
  const int pairs = cdiv(d.S_w, 2);
  if (d.fmt == kFmtF16) {
    b.a = a;
    b.nb = cdiv(N, 32);
    const dim3 grid((unsigned)(cdiv(K, 32) * b.nb), (unsigned)pairs);
    // 1024 threads while all blocks fit the chip at once, two to a compute unit (us, 1024 / 256 threads: 256 x 256 weights,
    // 4 slices, 128 blocks: 5.6 / 8.5; 784 x 500, 800 blocks: 16.4 / 15.6)
    const bool few = grid.x * grid.y <= 512;
    if (d.npol == 2 && few) hipLaunchKernelGGL((tile_f16_kernel<2, 1024>), grid, dim3(1024), 0, st, b);
    else if (d.npol == 2) hipLaunchKernelGGL((tile_f16_kernel<2, 256>), grid, dim3(256), 0, st, b);
    else if (few) hipLaunchKernelGGL((tile_f16_kernel<1, 1024>), grid, dim3(1024), 0, st, b);
    else hipLaunchKernelGGL((tile_f16_kernel<1, 256>), grid, dim3(256), 0, st, b);
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  uint32_t* table = nullptr;
  if (uses_code_table(d)) {
    table = reinterpret_cast<uint32_t*>(at + code_table_offset(cfg, d, K, N));
    const int entries = ((1 << cfg->slice_bits) - 1) * cfg->xbar_rows * cfg->xbar_cols;
    hipLaunchKernelGGL(code_table_kernel, dim3((unsigned)cdiv(entries, 256)), dim3(256), 0, st, a, table, whole_steps(cfg) ? 0 : 1);
    if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
    a.codes = table;
  }
  if (whole_steps(cfg)) {
    b.a = a;
    b.nb = cdiv(N, 64);
    const unsigned patches = (unsigned)(cdiv(K, 64) * b.nb);
    // one slice pair per block, in 16 waves where the layer has few patches (a wave then has four weights to work
    // through); the cheap sources take all the slices of a patch in one block once that leaves 4 blocks per compute unit
    if (uses_device_words(d)) {
      const dim3 grid(patches, (unsigned)pairs);
      const bool few = patches * (unsigned)pairs < 1024;
      if (d.npol == 2) hipLaunchKernelGGL((tile_f6_kernel<kFromDevices, 2, 512>), dim3(patches, (unsigned)d.S_w), dim3(512), 0, st, b, 1);
      else if (few) hipLaunchKernelGGL((tile_f6_kernel<kFromDevices, 1, 1024>), grid, dim3(1024), 0, st, b, 1);
      else hipLaunchKernelGGL((tile_f6_kernel<kFromDevices, 1, 512>), grid, dim3(512), 0, st, b, 1);
    } else {
      const int per = (int)std::min<unsigned>((unsigned)pairs, std::max(1u, patches * (unsigned)pairs / 1024u));
      const dim3 grid(patches, (unsigned)cdiv(pairs, per));
      if (table) hipLaunchKernelGGL((tile_f6_kernel<kFromTable, 1, 512>), grid, dim3(512), 0, st, b, per);
      else hipLaunchKernelGGL((tile_f6_kernel<kFromDigits, 1, 512>), grid, dim3(512), 0, st, b, per);
    }
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  }
  // arrays whose rows or columns are no whole steps of 64: the two copies group the devices differently, each is
  // written on its own
  for (int dir = 0; dir < 2; ++dir)
    for (int pol = 0; pol < d.npol; ++pol) {
      a.planes = reinterpret_cast<uint16_t*>(b.base[dir] + (size_t)pol * g[dir].pol_bytes);
      a.tile = g[dir].tile; a.ks = g[dir].ks; a.T = g[dir].T; a.OP = g[dir].OP;
      // every k-step that the contraction reads is written whole, padding included
      a.n_threads = (long long)a.T * a.ks * 8 * a.OP * 32;
      const unsigned blocks = (unsigned)((a.n_threads + 255) / 256);
      if (table) {
        a.codes = table + (dir == 1 ? code_table_words(cfg) : 0);
        // a thread quantises its weights once for all the slices it covers: as many slices per thread as
        // still leave about four waves for every SIMD of the chip
        a.spt = (int)std::min<long long>(d.S_w, std::max<long long>(1, a.n_threads * d.S_w / 262144));
        const dim3 grid(blocks, (unsigned)cdiv(d.S_w, a.spt));
        if (dir == 0) hipLaunchKernelGGL(tile_planes_f6_table_kernel<false>, grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(tile_planes_f6_table_kernel<true>, grid, dim3(256), 0, st, a);
      } else if (uses_device_words(d)) {
        uint32_t* words = reinterpret_cast<uint32_t*>(at + device_words_offset(cfg, d, K, N));
        if (dir == 0 && pol == 0) {                  // every device once, for both copies and both arrays
          const dim3 wgrid((unsigned)(((long long)K * N + 255) / 256), (unsigned)d.S_w);
          if (d.npol == 2) hipLaunchKernelGGL(device_words_kernel<2>, wgrid, dim3(256), 0, st, a, words);
          else hipLaunchKernelGGL(device_words_kernel<1>, wgrid, dim3(256), 0, st, a, words);
          if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
        }
        a.codes = words + (size_t)pol * d.S_w * K * N;
        a.n_threads = (long long)a.T * a.OP * a.ks * 64;   // one wave per fragment group
        const dim3 pgrid((unsigned)((a.n_threads + 255) / 256), (unsigned)d.S_w);
        if (dir == 0) hipLaunchKernelGGL(tile_planes_f6_words_kernel<false>, pgrid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL(tile_planes_f6_words_kernel<true>, pgrid, dim3(256), 0, st, a);
      } else if (dir == 0) hipLaunchKernelGGL(tile_planes_f6_kernel<false>, dim3(blocks, (unsigned)d.S_w), dim3(256), 0, st, a);
      else hipLaunchKernelGGL(tile_planes_f6_kernel<true>, dim3(blocks, (unsigned)d.S_w), dim3(256), 0, st, a);
      if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
    }
  return XBAR_OK;
}

int xbar_fwd(const xbar_config* cfg, const void* planes, const float* X, float* Y, int M, int K, int N, float w_max,
             float x_scale, void* ws, size_t ws_bytes, int16_t* codes, void* hip_stream) {
  return run_vmm(cfg, planes, X, Y, M, K, N, w_max, x_scale, ws, ws_bytes, codes, hip_stream, false);
}

int xbar_fwd_static(const xbar_config* cfg, const void* planes, const float* X, float* Y, int M, int K, int N, float w_max,
                    float x_scale, void* hip_stream) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(M, K, N))) return rc;
  const size_t need = plan_vmm(cfg, derive(cfg), M, K, N, false).ws_bytes;
  if (need > (size_t)XBAR_STATIC_SCRATCH_BYTES) return XBAR_ESCRATCH;
  void* ws = nullptr;
  if ((rc = static_scratch(&ws))) return rc;
  return run_vmm(cfg, planes, X, Y, M, K, N, w_max, x_scale, ws, (size_t)XBAR_STATIC_SCRATCH_BYTES, nullptr, hip_stream, false);
}

int xbar_bwd(const xbar_config* cfg, const void* planes, const float* dY, float* dX, int M, int K, int N, float w_max,
             float g_scale, void* ws, size_t ws_bytes, int16_t* codes, void* hip_stream) {
  return run_vmm(cfg, planes, dY, dX, M, K, N, w_max, g_scale, ws, ws_bytes, codes, hip_stream, true);
}

int xbar_update(const xbar_config* cfg, float* W, const float* X, const float* dY, int M, int K, int N, float w_max,
                float grad_scale, float lr, uint64_t step, void* ws, size_t ws_bytes, void* hip_stream) {
  return run_update(cfg, W, X, dY, M, K, N, w_max, grad_scale, lr, step, ws, ws_bytes, hip_stream, nullptr);
}

int xbar_pair_init(const float* W, float* Gp, float* Gn, int K, int N, float w_max, void* hip_stream) {
  const int rc = check_shape(1, K, N);
  if (rc) return rc;
  if (!aligned16(W) || !aligned16(Gp) || !aligned16(Gn)) return XBAR_EALIGN;
  if (!finite_pos(w_max)) return XBAR_EINVAL;
  PairInitArgs a;
  a.W = W; a.Gp = Gp; a.Gn = Gn; a.n = (long long)K * N; a.w_max = (double)w_max;
  hipLaunchKernelGGL(pair_init_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream), a);
  return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
}

int xbar_update_pair(const xbar_config* cfg, float* Gp, float* Gn, float* W, const float* X, const float* dY, int M, int K,
                     int N, float w_max, float grad_scale, float lr, uint64_t step, void* ws, size_t ws_bytes, void* hip_stream) {
  if (!Gp || !Gn) return XBAR_EALIGN;
  return run_update(cfg, W, X, dY, M, K, N, w_max, grad_scale, lr, step, ws, ws_bytes, hip_stream, nullptr, Gp, Gn);
}

int xbar_conv_update_pair(const xbar_config* cfg, float* Gp, float* Gn, float* W, const float* X, const float* dY,
                          const xbar_conv_geom* geom, int N, float w_max, float grad_scale, float lr, uint64_t step, void* ws,
                          size_t ws_bytes, void* hip_stream) {
  if (!Gp || !Gn) return XBAR_EALIGN;
  ConvGeom g;
  int M, K;
  const int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  return run_update(cfg, W, X, dY, M, K, N, w_max, grad_scale, lr, step, ws, ws_bytes, hip_stream,
                    conv_is_dense(geom) ? nullptr : &g, Gp, Gn);
}

size_t xbar_conv_workspace_bytes(const xbar_config* cfg, int op, const xbar_conv_geom* geom, int N) {
  ConvGeom g;
  int M, K;
  if (xbar_config_validate(cfg) || conv_dims(geom, &g, &M, &K) || check_shape(M, K, N)) return 0;
  const Derived d = derive(cfg);
  if (op == XBAR_OP_FWD) return plan_vmm(cfg, d, M, K, N, false).ws_bytes;
  if (op == XBAR_OP_BWD) return plan_vmm(cfg, d, M, K, N, true, !conv_is_dense(geom)).ws_bytes;
  if (op == XBAR_OP_UPDATE) return plan_update(M, K, N).ws_bytes;
  if (op == XBAR_OP_UPDATE_PULSED) return pulsed_workspace_bytes(M, K, N);
  return 0;
}

int xbar_conv_fwd(const xbar_config* cfg, const void* planes, const float* X, float* Y, const xbar_conv_geom* geom,
                  int N, float w_max, float x_scale, void* ws, size_t ws_bytes, int16_t* codes, void* hip_stream) {
  ConvGeom g;
  int M, K;
  const int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  return run_vmm(cfg, planes, X, Y, M, K, N, w_max, x_scale, ws, ws_bytes, codes, hip_stream, false,
                 conv_is_dense(geom) ? nullptr : &g);
}

int xbar_conv_bwd(const xbar_config* cfg, const void* planes, const float* dY, float* dX, const xbar_conv_geom* geom,
                  int N, float w_max, float g_scale, void* ws, size_t ws_bytes, void* hip_stream) {
  ConvGeom g;
  int M, K;
  int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  if ((rc = xbar_config_validate(cfg))) return rc;
  if ((rc = check_shape(M, K, N))) return rc;
  if (!aligned16(dX) || !aligned16(ws)) return XBAR_EALIGN;
  const size_t need = xbar_conv_workspace_bytes(cfg, XBAR_OP_BWD, geom, N);
  if (ws_bytes < need) return XBAR_EWORKSPACE;
  if (conv_is_dense(geom))       // every pixel is its own patch: the crossbar output is the result
    return run_vmm(cfg, planes, dY, dX, M, K, N, w_max, g_scale, ws, ws_bytes, nullptr, hip_stream, true);
  // the adding-up pass gathers every input pixel's patch errors from the partial sums
  return run_vmm(cfg, planes, dY, dX, M, K, N, w_max, g_scale, ws, ws_bytes, nullptr, hip_stream, true, nullptr, nullptr, &g);
}

int xbar_conv_update(const xbar_config* cfg, float* W, const float* X, const float* dY, const xbar_conv_geom* geom, int N,
                     float w_max, float grad_scale, float lr, uint64_t step, void* ws, size_t ws_bytes, void* hip_stream) {
  ConvGeom g;
  int M, K;
  const int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  return run_update(cfg, W, X, dY, M, K, N, w_max, grad_scale, lr, step, ws, ws_bytes, hip_stream,
                    conv_is_dense(geom) ? nullptr : &g);
}

namespace {
int run_histogram(const xbar_config* cfg, const void* planes, const float* in, int M, int K, int N, float in_scale, int op,
                  float bin_width, unsigned long long* hist, void* ws, size_t ws_bytes, void* hip_stream, const ConvGeom* conv);
}

int xbar_adc_histogram(const xbar_config* cfg, const void* planes, const float* in, int M, int K, int N, float in_scale,
                       int op, float bin_width, unsigned long long* hist, void* ws, size_t ws_bytes, void* hip_stream) {
  return run_histogram(cfg, planes, in, M, K, N, in_scale, op, bin_width, hist, ws, ws_bytes, hip_stream, nullptr);
}

int xbar_conv_adc_histogram(const xbar_config* cfg, const void* planes, const float* in, const xbar_conv_geom* geom, int N,
                            float in_scale, int op, float bin_width, unsigned long long* hist, void* ws, size_t ws_bytes,
                            void* hip_stream) {
  ConvGeom g;
  int M, K;
  const int rc = conv_dims(geom, &g, &M, &K);
  if (rc) return rc;
  // forward: the patches are gathered from the image; backward: the errors are a plain [M][N] matrix
  const bool gather = op == XBAR_OP_FWD && !conv_is_dense(geom);
  return run_histogram(cfg, planes, in, M, K, N, in_scale, op, bin_width, hist, ws, ws_bytes, hip_stream, gather ? &g : nullptr);
}

namespace {
int run_histogram(const xbar_config* cfg, const void* planes, const float* in, int M, int K, int N, float in_scale, int op,
                  float bin_width, unsigned long long* hist, void* ws, size_t ws_bytes, void* hip_stream, const ConvGeom* conv) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if (op != XBAR_OP_FWD && op != XBAR_OP_BWD) return XBAR_EINVAL;
  if (!finite_pos(bin_width)) return XBAR_EINVAL;
  if (!aligned16(hist)) return XBAR_EALIGN;
  // a converter with one code per bin: code = rne(I / bin_width), clamped to the last bin
  xbar_config c = *cfg;
  c.flags &= ~XBAR_ADC_CURVE;                        // the statistics are of the currents themselves
  c.adc_bits = (c.flags & XBAR_ADC_PER_ARRAY) ? 12 : 13;   // 4095 codes on the side(s) the converter has
  c.adc_fs_fwd = c.adc_fs_bwd = (float)(kStatBins - 1) * bin_width;
  if (!finite_pos(c.adc_fs_fwd)) return XBAR_EINVAL;
  return run_vmm(&c, planes, in, nullptr, M, K, N, 1.0f, in_scale, ws, ws_bytes, nullptr, hip_stream, op == XBAR_OP_BWD,
                 conv, hist);
}
}  // namespace

}  // extern "C"
