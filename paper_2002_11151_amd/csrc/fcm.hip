// Circuit-level crossbar model (Sec. IV-A) producing the stored distortion profile of Sec. IV-D:
// kernels and xbar_fcm_profile.
#include "xbar_common.h"
#include <type_traits>

using namespace xbar_detail;

namespace {

// ---------------------------------------------------------------------------------------------
// circuit-level crossbar model (Sec. IV-A: solve Ohm's and Kirchhoff's laws per crossbar instance;
// Sec. IV-D: the distortion profile D = (G_ideal - G_nonideal) / G_ideal that is stored and reused)
//
// Per crossbar, slice and array, with x_ij the device currents for the row voltages v:
//   x_ij / G_ij + sum_j' x_ij' wr(j,j') + sum_i' x_i'j wc(i,i') = v_i          (D + L) x = P v
//   wr(j,j') = r_source + (min(j,j') + 1) r_row,   wc(i,i') = (R - max(i,i')) r_col + r_sense
// L is the resistance matrix of the wires: symmetric, positive semidefinite, and applied in O(R C)
// by row and column prefix sums.  With x = s y, s = sqrt(G), the system (I + S L S) y = s v is
// symmetric positive definite with all eigenvalues >= 1 and a small condition number; conjugate
// gradients solve it for one unit row voltage at a time, and row i of the non-ideal conductance
// matrix is the column sums of x.  Devices that do not exist have s = 0 and drop out.
// ---------------------------------------------------------------------------------------------
struct FcmArgs {
  const float* W;
  float* profile;        // [S_w][2][K][N]
  double* scratch;       // per resident block: s, y, r, p, q of R C doubles each; state on chip: `far` pairs of coefficients
  int K, N, R, C, S_w, slice_bits, weight_bits, tiles_c;
  int groups, rhs_per_group, n_items, max_iter, far;
  uint32_t flags;
  double g_min, dg, var_sigma, r_row, r_col, r_source, r_sense, tol2;
  float w_max;
  uint64_t seed, step;
  const unsigned long long* step_add;   // optional device counter added to step
};

// Sum over the 256 threads of the block, returned to all of them; fixed order.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int d = 32; d; d >>= 1) v += __shfl_xor(v, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void fcm_kernel(FcmArgs a) {
  __shared__ double red[4];
  __shared__ double tot[2][4][64];                  // column pass: quarter totals per column of a strip
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int R = a.R, C = a.C;
  const int cpl = (C + 63) >> 6, strips = (C + 63) >> 6;
  const size_t rc = (size_t)R * C;
  double* sg = a.scratch + (size_t)blockIdx.x * 5 * rc;
  double* y = sg + rc;
  double* r = y + rc;
  double* p = r + rc;
  double* q = p + rc;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));

  for (int item = blockIdx.x; item < a.n_items; item += gridDim.x) {
    const int group = item % a.groups;
    const int t1 = item / a.groups;
    const int pol = t1 & 1;
    const int s = (t1 >> 1) % a.S_w;
    const int tile = (t1 >> 1) / a.S_w;
    const int k0 = (tile / a.tiles_c) * R, n0 = (tile % a.tiles_c) * C;
    const int rows = min(R, a.K - k0), cols = min(C, a.N - n0);
    const int i_begin = wave * (R / 4), i_end = min(rows, i_begin + R / 4);   // this wave's quarter (column pass)

    __syncthreads();                                 // the previous item is done with the scratch
    for (int i = wave; i < rows; i += 4)
      for (int j = lane; j < cols; j += 64) {
        const double qw = (double)((1u << a.weight_bits) - 1);
        const double wq = ::rint(clampd((double)a.W[(size_t)(k0 + i) * a.N + n0 + j] / (double)a.w_max, -1.0, 1.0) * qw);
        const int digit = (int)(((uint32_t)::fabs(wq) >> (a.slice_bits * s)) & ((1u << a.slice_bits) - 1));
        const bool mine = pol == 0 ? wq > 0.0 : wq < 0.0;
        double g = a.g_min + (mine ? digit * a.dg : 0.0);
        if (a.flags & XBAR_NI_VARIATION) {
          const uint64_t dev =
              (((uint64_t)(k0 + i) * (uint64_t)a.N + (uint64_t)(n0 + j)) * (uint64_t)a.S_w + (uint64_t)s) * 2 + pol;
          g *= 1.0 + a.var_sigma * rng.get(dev);
        }
        sg[(size_t)i * C + j] = ::sqrt(::fmax(g, 0.0));
      }
    __syncthreads();

    const int rhs_end = min(rows, (group + 1) * a.rhs_per_group);
    for (int rhs = group * a.rhs_per_group; rhs < rhs_end; ++rhs) {
      // y = 0, r = b = s on the driven row, p = 0 (the first direction is r)
      double part = 0.0;
      for (int i = wave; i < rows; i += 4)
        for (int j = lane; j < cols; j += 64) {
          const size_t at = (size_t)i * C + j;
          const double b = i == rhs ? sg[at] : 0.0;
          y[at] = 0.0;
          r[at] = b;
          p[at] = 0.0;
          part += b * b;
        }
      double rr = block_sum(part, red);              // also orders the stores above before the reads below
      const double stop = a.tol2 * rr;
      double beta = 0.0;
      for (int it = 0; it < a.max_iter && rr > stop; ++it) {
        // rows: p <- r + beta p;  q <- p + s Lr(s p)
        for (int i = wave; i < rows; i += 4) {
          const size_t base = (size_t)i * C;
          double pv[4], sv[4], l0[4], l1[4];
          double run0 = 0.0, run1 = 0.0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (u >= cpl) break;
            const int j = lane * cpl + u;
            pv[u] = sv[u] = 0.0;
            if (j < cols) {
              pv[u] = r[base + j] + beta * p[base + j];
              sv[u] = sg[base + j];
              p[base + j] = pv[u];
            }
            const double cur = sv[u] * pv[u];
            run0 += cur;
            run1 += (double)(j + 1) * cur;
            l0[u] = run0;
            l1[u] = run1;
          }
          const double inc0 = wave_inclusive_scan(run0, lane), inc1 = wave_inclusive_scan(run1, lane);
          const double total = __shfl(inc0, 63, 64);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (u >= cpl) break;
            const int j = lane * cpl + u;
            if (j < cols) {
              const double p0 = inc0 - run0 + l0[u], p1 = inc1 - run1 + l1[u];
              const double lr = a.r_source * total + a.r_row * (p1 + (double)(j + 1) * (total - p0));
              q[base + j] = pv[u] + sv[u] * lr;
            }
          }
        }
        __syncthreads();
        // columns: q <- q + s Lc(s p);  p.q
        double pq = 0.0;
        for (int strip = 0; strip < strips; ++strip) {
          const int j = strip * 64 + lane;
          const bool active = j < cols;
          double t0 = 0.0, t1s = 0.0;
          if (active)
            for (int i = i_begin; i < i_end; ++i) {
              const size_t at = (size_t)i * C + j;
              const double cur = sg[at] * p[at];
              t0 += cur;
              t1s += (double)(R - i) * cur;
            }
          tot[0][wave][lane] = t0;
          tot[1][wave][lane] = t1s;
          __syncthreads();
          if (active) {
            double above = 0.0, below = t1s, total = 0.0;
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
              const double x0 = tot[0][g4][lane];
              total += x0;
              if (g4 < wave) above += x0;
              if (g4 > wave) below += tot[1][g4][lane];
            }
            for (int ib = i_begin; ib < i_end; ib += 4) {
              double sv[4], pv[4], qv[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) {            // loads first: they do not wait for the stores below
                const size_t at = (size_t)min(ib + u, i_end - 1) * C + j;
                sv[u] = sg[at];
                pv[u] = p[at];
                qv[u] = q[at];
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const int i = ib + u;
                if (i < i_end) {
                  const double cur = sv[u] * pv[u];
                  above += cur;
                  below -= (double)(R - i) * cur;
                  const double lc = a.r_col * ((double)(R - i) * above + below) + a.r_sense * total;
                  const double qn = qv[u] + sv[u] * lc;
                  q[(size_t)i * C + j] = qn;
                  pq += pv[u] * qn;
                }
              }
            }
          }
          __syncthreads();                             // tot is reused by the next strip
        }
        pq = block_sum(pq, red);
        const double alpha = rr / pq;
        // y <- y + alpha p;  r <- r - alpha q
        part = 0.0;
        for (int i = wave; i < rows; i += 4)
          for (int j = lane; j < cols; j += 64) {
            const size_t at = (size_t)i * C + j;
            y[at] += alpha * p[at];
            const double rn = r[at] - alpha * q[at];
            r[at] = rn;
            part += rn * rn;
          }
        const double rr_new = block_sum(part, red);
        beta = rr_new / rr;
        rr = rr_new;
      }
      // row rhs of the non-ideal conductance matrix: column sums of x = s y
      for (int strip = 0; strip < strips; ++strip) {
        const int j = strip * 64 + lane;
        double e = 0.0;
        if (j < cols)
          for (int i = i_begin; i < i_end; ++i) e += sg[(size_t)i * C + j] * y[(size_t)i * C + j];
        tot[0][wave][lane] = e;
        __syncthreads();
        if (wave == 0 && j < cols) {
          const double e_all = (tot[0][0][lane] + tot[0][1][lane]) + (tot[0][2][lane] + tot[0][3][lane]);
          const double sv = sg[(size_t)rhs * C + j];
          const double g = sv * sv;
          a.profile[((size_t)(2 * s + pol) * a.K + k0 + rhs) * a.N + n0 + j] = g > 0.0 ? (float)((g - e_all) / g) : 0.0f;
        }
        __syncthreads();
      }
    }
  }
}

// Same solve for 64 x 64 and 128 x 128 crossbars with the whole state on chip, in device currents: with u = S r and w = S p
// (S = sqrt(G)) an iteration is  w <- u + beta w;  u <- u - alpha (w + G L w),  and x, whose column sums are wanted, grows by
// alpha w.  NT threads form a (NT / 16) x 16 grid; thread (ty, tx) owns the SR x SC devices at rows SR ty.., columns SC tx..; u and
// w live in its registers (two waves per SIMD: one alone leaves the double-precision pipe waiting for its own results), G in LDS.
// With S_k the sum of a row's w from column k on and P_k that of a column's w down to row k,
//   (Lr w)_j = r_source S_0 + r_row sum_{k <= j} S_k,     w.Lr w = r_source S_0^2 + r_row sum_k S_k^2,
//   (Lc w)_i = r_sense P_last + r_col sum_{k >= i} P_k,   w.Lc w = r_sense P_last^2 + r_col sum_k P_k^2.
// Sums along a row run over the 16 consecutive lanes that share ty (DPP row shifts), along a column over the 4 lane groups of
// a wave (row swaps) and over the waves (LDS, one thread per column and kind of sum).
// The driven rows of a crossbar differ in the right-hand side alone and excite much the same part of the spectrum, so only a
// block's first solve works out alpha and beta (conjugate gradients, stopped at half the tolerance); the others run the same
// coefficients -- a fixed polynomial in the matrix -- without the scalar products and their barriers, and measure the residual
// once at the end.  Conjugate gradients run on the voltages u / G and w / G, which makes w.w / G and u.u / G products of the two: full
// precision and no reciprocal per device (with the instruction's 24 bits instead, on currents: 784 x 500 weights at 100 Ohm, when
// no solve of so many iterations shared, 98.3 ms against 81.0).
// One that misses the tolerance is finished by conjugate gradients, and the next starts anew.  (On the CPU,
// 128 x 128 devices at 1e-11: as many iterations as conjugate gradients of its own or one more, for Rmin of 1e3 .. 1e5 Ohm, 10 %
// variation, ragged tiles.)
// The polynomial is small on what the first solve drives and nowhere else.  Where the rows see little of each other (no column wires,
// say) and the first one is all off, it multiplies the others' residuals by up to 1e20, and since the residual is the recurrence's own,
// which does not see what was rounded on the way, a solve that went through such values must not be finished, whatever it ends at.  So
// every solve watches how far its voltages swing (`swing`), and one beyond kMaxSwing is thrown away, as is one that hardly shrank its
// residual: conjugate gradients of its own then give the next rows' coefficients.  After the second a block shares nothing any more.
// What bounds it: the issue of vector instructions, 770 per thread and iteration of 32 devices (353 the recurrences at 11 per
// device, the rest sums across lanes and waves), some 70 % of the time.  784 x 500 layer of the 784-500-10 perceptron (128 x 128
// arrays, 4 slices): 5.1 -> 3.4 ms against scalar products in every iteration (1130 instructions, four barriers for two, 15 of
// them spills); 256 x 256 weights on 64 x 64 arrays 345 -> 258 us, 64 x 10 61 -> 35.
template <int CTRL>
__device__ __forceinline__ double dpp_row_f64(double x) {   // lanes whose source lies outside the row of 16 get 0
  union { double d; int i[2]; } v, o;
  v.d = x;
  o.i[0] = __builtin_amdgcn_update_dpp(0, v.i[0], CTRL, 0xF, 0xF, true);
  o.i[1] = __builtin_amdgcn_update_dpp(0, v.i[1], CTRL, 0xF, 0xF, true);
  return o.d;
}

__device__ __forceinline__ double row16_inclusive_scan(double x) {
  x += dpp_row_f64<0x111>(x);                        // row_shr:1
  x += dpp_row_f64<0x112>(x);                        // row_shr:2
  x += dpp_row_f64<0x114>(x);                        // row_shr:4
  x += dpp_row_f64<0x118>(x);                        // row_shr:8
  return x;
}

// Inclusive sums of two values over the four groups (rows) of 16 lanes of a wave, lane by lane.  Row swaps between the two values
// line both up for one addition; upper: 1.0 in rows 2 and 3, else 0.0.
__device__ __forceinline__ void group16_inclusive_scans(double& x, double& y, double upper) {
  union Word { double d; uint32_t i[2]; } a, b, t, u, v;
  auto swap16 = [](Word& p, Word& q) __attribute__((always_inline)) {   // the odd rows of p with the even rows of q
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const auto s = __builtin_amdgcn_permlane16_swap(p.i[h], q.i[h], false, false);
      p.i[h] = s[0];
      q.i[h] = s[1];
    }
  };
  a.d = x;
  b.d = y;
  swap16(a, b);                                      // a: x0 y0 x2 y2, b: x1 y1 x3 y3
  t.d = a.d + b.d;                                   // x0 + x1, y0 + y1, x2 + x3, y2 + y3
#pragma unroll
  for (int h = 0; h < 2; ++h) u.i[h] = __builtin_amdgcn_permlane32_swap(t.i[h], t.i[h], false, false)[0];   // rows 0, 1, 0, 1 of t
  v = u;
  swap16(u, v);                                      // x0 + x1 in every row of u, y0 + y1 in every row of v
  swap16(a, t);                                      // a: x0, x0 + x1, x2, x2 + x3; t: the same of y
  x = __builtin_fma(upper, u.d, a.d);
  y = __builtin_fma(upper, v.d, t.d);
}

// Sum over the block, returned to every thread, in a fixed order: rows of 16 lanes by DPP, the four rows of a wave by
// lane reads, the waves through LDS.  `red`: one of two sets of slots used in turn, so that one barrier is enough.
template <int NW>
__device__ __forceinline__ double block_sum_n(double v, double* red) {
  v = row16_inclusive_scan(v);
  union { double d; int i[2]; } x;
  x.d = v;
  double row[4];
#pragma unroll
  for (int g = 0; g < 4; ++g)
    row[g] = __hiloint2double(__builtin_amdgcn_readlane(x.i[1], 16 * g + 15), __builtin_amdgcn_readlane(x.i[0], 16 * g + 15));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = (row[0] + row[1]) + (row[2] + row[3]);
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += red[w];
  return t;
}

// The driven row is at 1 V, and wires take no more than that off it: solves that share well swing by 0.1 .. 30 V (128 x 128 and
// 64 x 64 devices of 100 Ohm .. 100 kOhm, on the CPU), those that must not by 1e2 .. 1e20.  A thousand cost the result 1e-13 of the
// conductances around the row.
constexpr double kMaxSwing = 1e3;

template <int SR, int SC, int NT>
struct FcmShape {
  static constexpr int NW = NT / 64;                 // waves; 4 thread rows (ty) per wave
  static constexpr int R = (NT / 16) * SR, C = 16 * SC;          // == a.R, a.C
  static constexpr int kSums = 2 * NW * C;
  // G, a wave's column sums, what lies before / behind a wave; the last wave has nothing behind it: that line holds the slots
  // of the block sums and the coefficients
  static constexpr size_t kLdsBytes = (size_t)(R * C + 2 * kSums) * sizeof(double);
  static constexpr int kSteps = (C - 2 * NW) / 2;    // pairs of coefficients kept there; those of later steps in the workspace
};

template <int SR, int SC, int NT>
__global__ __launch_bounds__(NT, 2) void fcm_onchip_kernel(FcmArgs a) {
  extern __shared__ double fcm_lds[];
  using Shape = FcmShape<SR, SC, NT>;
  constexpr int NW = Shape::NW, R = Shape::R, C = Shape::C, kSteps = Shape::kSteps;
  double* g_lds = fcm_lds;                           // [SR * SC][NT]: element (ar, bc) of thread tid
  double* sums = g_lds + SR * SC * NT;               // [2][NW][C]: a wave's column sums; column SC tx + bc at 16 bc + tx (no bank
                                                     //   conflicts).  Written before the first barrier of an iteration, read before the second, but
                                                     //   for a wave's own
  double* rest = sums + Shape::kSums;                // [2][NW][C]: of the waves above (of the first wave: all), of those below.  Written
                                                     //   between the barriers, read behind the second
  double* total = rest;                              // [C] column totals
  double* red = rest + (2 * NW - 1) * C;             // [2][NW]
  double* coef = red + 2 * NW;                       // [2][kSteps]: alpha, beta
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int tx = tid & 15, ty = tid >> 4;
  const int i0 = ty * SR, j0 = tx * SC;
  // Places in LDS as an opaque start plus constants, which the instructions hold; taken apart by the compiler they are an address
  // register for each.  G reaches beyond what an instruction holds: two starts.
  constexpr int kHalf = SR * SC / 2;
  int at_g0 = tid, at_g1 = kHalf * NT + tid, at_wave = wave * C + tx, at_column = tx;
  asm("" : "+v"(at_g0), "+v"(at_g1), "+v"(at_wave), "+v"(at_column));
  auto g_of = [&](int e) __attribute__((always_inline)) -> double& { return g_lds[e < kHalf ? at_g0 + e * NT : at_g1 + (e - kHalf) * NT]; };
  const double upper = lane >= 32 ? 1.0 : 0.0;

  const int group = blockIdx.x % a.groups;
  const int t1 = blockIdx.x / a.groups;
  const int pol = t1 & 1;
  const int s = (t1 >> 1) % a.S_w;
  const int tile = (t1 >> 1) / a.S_w;
  const int k0 = (tile / a.tiles_c) * R, n0 = (tile % a.tiles_c) * C;
  const int rows = min(R, a.K - k0), cols = min(C, a.N - n0);
  const int rhs_begin = group * a.rhs_per_group, rhs_end = min(rows, rhs_begin + a.rhs_per_group);
  if (rhs_begin >= rhs_end) return;                  // a ragged tile: no row left for this block

  // every thread reads back only what it wrote itself: no barrier needed for g_lds.  Weights first, all loads side by side
#pragma unroll
  for (int ar = 0; ar < SR; ++ar)
#pragma unroll
    for (int bc = 0; bc < SC; ++bc) {
      const int i = min(i0 + ar, rows - 1), j = min(j0 + bc, cols - 1);
      g_lds[(ar * SC + bc) * NT + tid] = (double)a.W[(size_t)(k0 + i) * a.N + n0 + j];
    }
  {
    const double qw = (double)((1u << a.weight_bits) - 1), w_max = (double)a.w_max;
    NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));
#pragma unroll 1
    for (int e = 0; e < SR * SC; ++e) {
      const int i = i0 + e / SC, j = j0 + e % SC;
      double g = 0.0;
      if (i < rows && j < cols) {
        const int wq = quantized_weight((float)g_lds[e * NT + tid], w_max, qw, qw / w_max);
        const int digit = (int)(((uint32_t)abs(wq) >> (a.slice_bits * s)) & ((1u << a.slice_bits) - 1));
        const bool mine = pol == 0 ? wq > 0 : wq < 0;
        g = a.g_min + (mine ? digit * a.dg : 0.0);
        if (a.flags & XBAR_NI_VARIATION) {
          const uint64_t dev = (((uint64_t)(k0 + i) * (uint64_t)a.N + (uint64_t)(n0 + j)) * (uint64_t)a.S_w + (uint64_t)s) * 2 + pol;
          g *= 1.0 + a.var_sigma * rng.get(dev);
        }
      }
      g_lds[e * NT + tid] = ::fmax(g, 0.0);
    }
  }

  int steps = 0, discarded = 0;                      // coefficients known; solves that they did not fit
  double2* far = reinterpret_cast<double2*>(a.scratch) + (size_t)blockIdx.x * a.far - kSteps;
  for (int rhs = rhs_begin; rhs < rhs_end; ++rhs) {
    double u[SR][SC], w[SR][SC], e = 0.0;            // e: solution summed over column tid % C
    double beta = 0.0, alpha = 0.0, part = 0.0, swing = 0.0;
    // Computed here: left alone, the compiler moves the arithmetic behind the next branch and keeps all that it waits for
    auto pin = [](double& x, double& y, double& z) __attribute__((always_inline)) { asm volatile("" : "+v"(x), "+v"(y), "+v"(z)); };
    // One iteration; CG: on u / G and w / G, alpha from w.A w and, in `part`, the square of what is left.  `first`: w is 0 outside
    // the driven row.
    auto iterate = [&](auto is_cg, bool first, double rr) __attribute__((always_inline)) {
      constexpr bool CG = decltype(is_cg)::value;
      // Column by column in both passes: two running sums per row, those of one column at a time.  (Row by row the running sums
      // of all columns are alive beside u and w, and the registers spill.)
      double row0[SR], row1[SR], col0[SC], col1[SC], cross[SC] = {};   // row0: sum of w from the column on; row1: sum of those sums
      double pq = 0.0, energy = 0.0, row_sq = 0.0, col_sq = 0.0;
      if (CG || !first || (rhs >= 4 * SR * wave && rhs < 4 * SR * (wave + 1))) {
        // w <- u + beta w: sums, sums of the sums (and their squares) inside this thread's patch, rows from the right, columns
        // from above
#pragma unroll
        for (int bc = SC - 1; bc >= 0; --bc) {
          double run = 0.0, runs = 0.0;
#pragma unroll
          for (int ar = 0; ar < SR; ++ar) {
            w[ar][bc] = __builtin_fma(beta, w[ar][bc], u[ar][bc]);
            const double current = CG ? g_of(ar * SC + bc) * w[ar][bc] : w[ar][bc];
            row0[ar] = bc == SC - 1 ? current : row0[ar] + current;       // no sums that begin with 0: they are not free
            row1[ar] = bc == SC - 1 ? row0[ar] : row1[ar] + row0[ar];
            run = ar == 0 ? current : run + current;
            runs = ar == 0 ? run : runs + run;
            if constexpr (CG) {
              pq = __builtin_fma(current, w[ar][bc], pq);
              row_sq = __builtin_fma(row0[ar], row0[ar], row_sq);
              col_sq = __builtin_fma(run, run, col_sq);
              pin(pq, row_sq, col_sq);
            }
          }
          // sums over the lane groups above inside the wave.  Kept per column: the sum and the sum of (R - i) w down to and
          // with this thread inside the wave, and what multiplies the sum above the wave in the squares of P
          col0[bc] = run;
          col1[bc] = __builtin_fma((double)(R - SR - i0), run, runs);
          group16_inclusive_scans(col0[bc], col1[bc], upper);
          if constexpr (CG) {
            const double in0 = col0[bc] - run;       // above this thread, inside the wave
            col_sq = __builtin_fma(in0, __builtin_fma((double)SR, in0, 2.0 * runs), col_sq);
            cross[bc] = 2.0 * __builtin_fma((double)SR, in0, runs);
          }
          pin(col0[bc], col1[bc], cross[bc]);
#pragma unroll
          for (int ar = 0; ar < SR; ++ar) pin(w[ar][bc], row0[ar], row1[ar]);
        }
        energy = a.r_row * row_sq;
      } else {
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) col0[bc] = col1[bc] = 0.0;
#pragma unroll
        for (int ar = 0; ar < SR; ++ar) row0[ar] = row1[ar] = 0.0;
      }
      if (lane >= 48) {                              // last group of the wave holds the wave's sums
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          sums[at_wave + 16 * bc] = col0[bc];
          sums[at_wave + NW * C + 16 * bc] = col1[bc];
        }
      }
      __syncthreads();
      if (tid < 2 * C) {                             // one thread per column and kind of sum: prefix / suffix over the waves
        const int kind = tid / C, j = tid % C;
        const double* from = sums + kind * NW * C + j;
        double* to = rest + kind * NW * C + j;
        double v[NW], run = 0.0;
#pragma unroll
        for (int x = 0; x < NW; ++x) v[x] = from[x * C];
        if (kind == 0) {
#pragma unroll
          for (int x = 0; x < NW; ++x) {
            if (x > 0) to[x * C] = run;
            run += v[x];
          }
          to[0] = run;
        } else {
#pragma unroll
          for (int x = NW - 1; x > 0; --x) {
            run += v[x];
            to[(x - 1) * C] = run;
          }
        }
      }
      // rows: what lies outside the patch, and w.A w's row part.  From here on row0 is S at the patch's first column, row1
      // the drop up to it.  (Between the barriers: half of the waves have nothing else to do there)
#pragma unroll
      for (int ar = 0; ar < SR; ++ar) {
        const double full1 = __builtin_fma((double)j0, row0[ar], row1[ar]);   // sum of (j + 1) w
        const double inc0 = row16_inclusive_scan(row0[ar]), inc1 = row16_inclusive_scan(full1);
        const double all = dpp_row_f64<0x15F>(inc0);   // row_newbcast:15
        const double right = all - inc0;           // sum of w to the right of the patch
        if constexpr (CG) {                        // the driver's share
          energy = __builtin_fma(a.r_row * right, __builtin_fma((double)SC, right, 2.0 * row1[ar]), energy);
          energy = __builtin_fma(tx == 0 ? a.r_source * all : 0.0, all, energy);
        }
        row1[ar] = __builtin_fma(a.r_row, __builtin_fma((double)j0, all - (inc0 - row0[ar]), inc1 - full1), a.r_source * all);
        row0[ar] = a.r_row * (right + row0[ar]);
        pin(row0[ar], row1[ar], energy);
      }
      __syncthreads();
      auto outside = [&](int bc, double& above, double& below1, double& all) __attribute__((always_inline)) {
        const double in_above = rest[at_wave + 16 * bc], in_below = rest[at_wave + NW * C + 16 * bc];
        all = total[at_column + 16 * bc];
        above = wave == 0 ? 0.0 : in_above;
        below1 = (wave == NW - 1 ? 0.0 : in_below) + (sums[at_wave + NW * C + 16 * bc] - col1[bc]);
      };
      if constexpr (CG) {
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          double above, below1, all;
          outside(bc, above, below1, all);
          col_sq = __builtin_fma(above, __builtin_fma((double)SR, above, cross[bc]), col_sq);
          energy = __builtin_fma(ty == 0 ? a.r_sense * all : 0.0, all, energy);
          pin(col_sq, energy, cross[bc]);
        }
        pq += __builtin_fma(a.r_col, col_sq, energy);
        alpha = rr / block_sum_n<NW>(pq, red + NW);
        part = 0.0;
      }
      // u <- u - alpha A w
      double high = 0.0;
#pragma unroll
      for (int bc = 0; bc < SC; ++bc) {
        double above, below1, all;
        outside(bc, above, below1, all);
        // from the row below the patch up: the drop; P at the patch's last row (both in Ohm units)
        const double last = above + col0[bc];
        double pre = a.r_col * last, lc = __builtin_fma(a.r_col, __builtin_fma((double)(R - SR - i0), last, below1), a.r_sense * all);
#pragma unroll
        for (int ar = SR - 1; ar >= 0; --ar) {
          const double g = g_of(ar * SC + bc), current = CG ? g * w[ar][bc] : w[ar][bc];
          row1[ar] += row0[ar];
          row0[ar] = __builtin_fma(-a.r_row, current, row0[ar]);
          lc += pre;
          pre = __builtin_fma(-a.r_col, current, pre);
          const double drop = row1[ar] + lc, q = CG ? w[ar][bc] + drop : __builtin_fma(g, drop, w[ar][bc]);
          u[ar][bc] = __builtin_fma(-alpha, q, u[ar][bc]);
          // What a solve amplifies is smooth along the wires, so one device of a patch per column is looked at, which are one
          // or two per row.  All of them: 4 % of the instructions, not 1
          if constexpr (!CG) {
            if (bc * SR / SC == ar) high = ::fmax(high, ::fabs(drop));
          }
          if constexpr (CG) part = __builtin_fma(g * u[ar][bc], u[ar][bc], part);
          pin(u[ar][bc], row0[ar], row1[ar]);
          if constexpr (CG) pin(part, lc, pre);
        }
      }
      e = __builtin_fma(alpha, total[tid & (C - 1)], e);   // column sum of x = sum alpha w
      if constexpr (!CG) swing = ::fmax(swing, ::fabs(alpha) * high);
    };

    double b2 = 0.0;                                 // square of the right-hand side S v
#pragma unroll
    for (int ar = 0; ar < SR; ++ar)
#pragma unroll
      for (int bc = 0; bc < SC; ++bc) {
        u[ar][bc] = (i0 + ar == rhs) ? g_of(ar * SC + bc) : 0.0;
        w[ar][bc] = 0.0;
        b2 += u[ar][bc];
      }
    b2 = block_sum_n<NW>(b2, red + NW);
    const double stop = a.tol2 * b2;
    double rr = b2;
    bool known = steps > 0;
    if (known) {
      for (int it = 0; it < steps; ++it) {
        if (it < kSteps) {
          alpha = coef[it];
          beta = coef[kSteps + it];
        } else {
          const double2 both = far[it];
          alpha = both.x;
          beta = both.y;
        }
        iterate(std::false_type{}, it == 0, 0.0);
      }
      // An upper bound of the residual first: the instruction's reciprocal is good to 2^29 units in the last place by the documents of
      // the instruction set, 2^-23 (2^-24.4 measured), and only what it clears is done.  (By division 4 % of a solve of eight iterations.)
      part = swing <= kMaxSwing ? 0.0 : INFINITY;    // (a NaN in the voltages is one in u)
#pragma unroll
      for (int ar = 0; ar < SR; ++ar)
#pragma unroll
        for (int bc = 0; bc < SC; ++bc)              // a device that is not there has u = 0
          part = __builtin_fma(u[ar][bc] * __builtin_amdgcn_rcp(::fmax(g_of(ar * SC + bc), 1e-300)), u[ar][bc], part);
      rr = (1.0 + 0x1p-20) * block_sum_n<NW>(part, red);
      if (!(rr <= 1e-6 * b2)) {                      // also an infinity or a NaN
        known = false;
        ++discarded;
      } else if (rr > stop) {                        // conjugate gradients from here, on u / G (w counts for nothing: beta is 0)
        part = 0.0;
#pragma unroll
        for (int ar = 0; ar < SR; ++ar)
#pragma unroll
          for (int bc = 0; bc < SC; ++bc) {
            const double g = g_of(ar * SC + bc), left = g > 0.0 ? u[ar][bc] / g : 0.0;
            part = __builtin_fma(left, u[ar][bc], part);
            u[ar][bc] = left;
          }
        rr = block_sum_n<NW>(part, red + NW);
        beta = 0.0;
      }
    }
    if (!known) {                                    // from the start: u / G is v
#pragma unroll
      for (int ar = 0; ar < SR; ++ar)
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          u[ar][bc] = (i0 + ar == rhs) ? 1.0 : 0.0;
          w[ar][bc] = 0.0;
        }
      beta = e = 0.0;
      rr = b2;
    }
    // conjugate gradients: all of a solve of its own, what the coefficients may have left of another
    const double goal = known ? stop : 0.25 * stop;
    int it = 0;
    for (; it < a.max_iter && rr > goal; ++it) {
      iterate(std::true_type{}, false, rr);
      if (!known && tid == 0) {                      // the solves after this one read them behind a barrier
        if (it < kSteps) {
          coef[it] = alpha;
          coef[kSteps + it] = beta;
        } else if (it < kSteps + a.far) {
          far[it] = double2{alpha, beta};
        }
      }
      const double rr_new = block_sum_n<NW>(part, red);
      beta = rr_new / rr;
      rr = rr_new;
    }
    // a solve that missed the tolerance drives what the first one hardly did (a row of off-state devices, say): the next starts anew
    steps = known ? (it > 0 ? 0 : steps) : it <= kSteps + a.far && discarded < 2 ? it : 0;
    if (tid < C) sums[tid] = e;                      // the sums of the last iteration have been read: two barriers ago at least
    __syncthreads();
    if (rhs >= i0 && rhs < i0 + SR) {
#pragma unroll
      for (int bc = 0; bc < SC; ++bc) {
        const int j = j0 + bc;
        if (j < cols) {
          const double g = g_lds[((rhs - i0) * SC + bc) * NT + tid];
          a.profile[((size_t)(2 * s + pol) * a.K + k0 + rhs) * a.N + n0 + j] = g > 0.0 ? (float)((g - sums[at_column + 16 * bc]) / g) : 0.0f;
        }
      }
    }
    // the next solve writes these sums only behind the barrier of its first block sum
  }
}

// The driven rows of a crossbar are split over several blocks, as many as fill the chip (`slots` blocks at a time) evenly: every block
// sets its devices up and has one solve without known coefficients, together worth about kSetupRows rows.
constexpr double kSetupRows = 1.2;
int rows_per_block(const FcmArgs& a, int slots) {
  // Whole tiles' blocks come first and take so many rounds over the chip; the last tile row's rows fill the last round's gaps
  const int tiles_r = cdiv(a.K, a.R), sets = a.tiles_c * a.S_w * 2, last = a.K - (tiles_r - 1) * a.R;
  double best = 0.0;
  int rows = 1;
  for (int g = 1; g <= a.R; ++g) {
    const int per = cdiv(a.R, g);
    const double whole = kSetupRows + per, part = kSetupRows + std::min(per, last);
    const long long n_whole = (long long)sets * (tiles_r - 1) * cdiv(a.R, per), n_part = (long long)sets * cdiv(last, per);
    const long long rounds = n_whole / slots, rest = n_whole % slots, gaps = rest ? slots - rest : 0;
    const long long more = std::max(0ll, n_part - gaps);
    const double cost = (rounds + (rest ? 1 : 0)) * whole + (double)((more + slots - 1) / slots) * part;
    if (g == 1 || cost < best) {
      best = cost;
      rows = per;
    }
  }
  return rows;
}
constexpr int kSlots128 = 256, kSlots64 = 256 * 3;   // blocks that the chip holds

// False: no such LDS size on this device.
template <int SR, int SC, int NT>
bool launch_onchip(FcmArgs a, int slots, size_t ws_bytes, hipStream_t st) {
  constexpr int lds_bytes = (int)FcmShape<SR, SC, NT>::kLdsBytes;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&fcm_onchip_kernel<SR, SC, NT>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          lds_bytes) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  a.rhs_per_group = rows_per_block(a, slots);
  a.groups = cdiv(a.R, a.rhs_per_group);
  const unsigned blocks = (unsigned)(cdiv(a.K, a.R) * a.tiles_c * a.S_w * 2 * a.groups);
  // The workspace, which the general kernel needs, has room for 256 pairs per block but for the very largest layers.  784 x 500
  // weights, 128 x 128 arrays, ms with the pairs in LDS alone and with these, against scalar products in every iteration: 100
  // Ohm (some 130 iterations) 81.0, 63.2, 74.6, 300 Ohm 48.3, 35.3, 44.9; 256 x 256 on 64 x 64 arrays, 100 Ohm 3.73, 3.01, 3.20
  a.far = (int)std::min<size_t>(256, ws_bytes / sizeof(double2) / blocks);
  hipLaunchKernelGGL((fcm_onchip_kernel<SR, SC, NT>), dim3(blocks), dim3(NT), lds_bytes, st, a);
  return true;
}

struct FcmPlan {
  int n_items, groups, rhs_per_group, blocks;
  int onchip;            // 0: state in the workspace; 64 / 128: square crossbars of that size, state on chip
  size_t ws_bytes;
};

FcmPlan plan_fcm(const xbar_config* c, const Derived& d, int K, int N) {
  FcmPlan p;
  const int per_drive_sets = cdiv(K, c->xbar_rows) * cdiv(N, c->xbar_cols) * d.S_w * 2;   // (tile, slice, array)
  // split the driven rows of a crossbar over several blocks when there are few crossbars
  p.groups = std::min(c->xbar_rows / 4, std::max(1, cdiv(2048, per_drive_sets)));
  p.rhs_per_group = cdiv(c->xbar_rows, p.groups);
  p.groups = cdiv(c->xbar_rows, p.rhs_per_group);
  p.n_items = per_drive_sets * p.groups;
  p.onchip = (c->xbar_rows == c->xbar_cols && (c->xbar_rows == 64 || c->xbar_rows == 128)) ? c->xbar_rows : 0;
  // the workspace is sized for the general kernel in every case (it is the fallback)
  const size_t slot = (size_t)5 * c->xbar_rows * c->xbar_cols * sizeof(double);
  p.blocks = std::min(p.n_items, slot > (size_t)1 << 20 ? 1024 : 2048);
  p.ws_bytes = align256((size_t)p.blocks * slot);
  return p;
}

}  // namespace

namespace xbar_detail {
size_t fcm_workspace_bytes(const xbar_config* cfg, int K, int N) { return plan_fcm(cfg, derive(cfg), K, N).ws_bytes; }
}  // namespace xbar_detail

extern "C" {

int xbar_fcm_profile(const xbar_config* cfg, const float* W, int K, int N, float w_max, uint64_t step, float* profile,
                     void* ws, size_t ws_bytes, void* hip_stream) {
  int rc = xbar_config_validate(cfg);
  if (rc) return rc;
  if ((rc = check_shape(1, K, N))) return rc;
  if (!aligned16(W) || !aligned16(profile) || !aligned16(ws)) return XBAR_EALIGN;
  if (!finite_pos(w_max)) return XBAR_EINVAL;
  const Derived d = derive(cfg);
  const FcmPlan p = plan_fcm(cfg, d, K, N);
  if (ws_bytes < p.ws_bytes) return XBAR_EWORKSPACE;
  FcmArgs a;
  a.W = W; a.profile = profile; a.scratch = reinterpret_cast<double*>(ws);
  a.K = K; a.N = N; a.R = cfg->xbar_rows; a.C = cfg->xbar_cols; a.S_w = d.S_w;
  a.slice_bits = cfg->slice_bits; a.weight_bits = cfg->weight_bits; a.tiles_c = cdiv(N, cfg->xbar_cols);
  a.groups = p.groups; a.rhs_per_group = p.rhs_per_group; a.n_items = p.n_items;
  a.max_iter = 500;
  a.flags = cfg->flags;
  a.g_min = 1.0 / (double)cfg->r_max;
  a.dg = (1.0 / (double)cfg->r_min - a.g_min) / (double)((1 << cfg->slice_bits) - 1);
  a.var_sigma = (double)cfg->var_sigma;
  a.r_row = (double)cfg->r_row; a.r_col = (double)cfg->r_col;
  a.r_source = (double)cfg->r_source; a.r_sense = (double)cfg->r_sense;
  a.tol2 = 1e-22;                                   // relative residual 1e-11
  a.w_max = w_max; a.seed = cfg->seed; a.step = step; a.step_add = current_step_source();
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  if (p.onchip == 128 ? launch_onchip<4, 8, 512>(a, kSlots128, ws_bytes, st) : p.onchip == 64 && launch_onchip<4, 4, 256>(a, kSlots64, ws_bytes, st))
    return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
  hipLaunchKernelGGL(fcm_kernel, dim3((unsigned)p.blocks), dim3(256), 0, st, a);
  if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  return XBAR_OK;
}

int xbar_fcm_rows_per_block(const xbar_config* cfg, int K, int N) {
  if (xbar_config_validate(cfg) || check_shape(1, K, N)) return 0;
  const Derived d = derive(cfg);
  const int onchip = plan_fcm(cfg, d, K, N).onchip;
  FcmArgs a = {};
  a.K = K; a.R = cfg->xbar_rows; a.S_w = d.S_w; a.tiles_c = cdiv(N, cfg->xbar_cols);
  return onchip ? rows_per_block(a, onchip == 128 ? kSlots128 : kSlots64) : 0;
}

}  // extern "C"
