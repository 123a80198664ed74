// Circuit-level crossbar model (Sec. IV-A) producing the stored distortion profile of Sec. IV-D:
// kernels and xbar_fcm_profile.
#include "xbar_common.h"

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
  double* scratch;       // per resident block: s, y, r, p, q of R C doubles each
  int K, N, R, C, S_w, slice_bits, weight_bits, tiles_c;
  int groups, rhs_per_group, n_items, max_iter;
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

// Same solve for 64 x 64 and 128 x 128 crossbars with the whole state on chip.  NT threads form a (NT / 16) x 16 grid;
// thread (ty, tx) owns the SR x SC devices at rows SR ty.., columns SC tx..; residual and search direction live in its
// registers (two waves per SIMD: one alone leaves the double-precision pipe waiting for its own results), sqrt(G) in
// LDS.  With u = s p, S_k the sum of a row's u from column k on and P_k that of a column's u down to row k,
//   (Lr u)_j = r_source S_0 + r_row sum_{k <= j} S_k,     u.Lr u = r_source S_0^2 + r_row sum_k S_k^2,
//   (Lc u)_i = r_sense P_last + r_col sum_{k >= i} P_k,   u.Lc u = r_sense P_last^2 + r_col sum_k P_k^2,
// so p.Ap comes out of the pass that forms p and its sums (9 operations per device: squares of the sums inside the
// thread's patch, completed with what lies outside it after the scans), and the residual pass rebuilds A p from
// running sums (9 more); A p is never stored.  Sums along a row run over the 16 consecutive lanes that share ty (DPP row
// shifts), along a column over the 4 lane groups of a wave (shuffles) and over the waves (LDS, one thread per column).
// Measured on the 784 x 500 layer of the 784-500-10 perceptron (128 x 128 arrays, 4 slices): 12.4 -> 5.0 ms against
// 8 x 8 devices per thread, one wave per SIMD and A p evaluated twice (40 operations per device and iteration).
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

// Inclusive sum over the four groups of 16 lanes of a wave (lane by lane), by row swaps: even and odd rows, then halves.
__device__ __forceinline__ double group16_inclusive_scan(double x, int lane) {
  union { double d; uint32_t i[2]; } v, even, odd, t, low;
  v.d = x;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto s = __builtin_amdgcn_permlane16_swap(v.i[h], v.i[h], false, false);
    even.i[h] = s[0];                               // rows 0, 0, 2, 2
    odd.i[h] = s[1];                                // rows 1, 1, 3, 3
  }
  t.d = even.d + odd.d;
#pragma unroll
  for (int h = 0; h < 2; ++h) low.i[h] = __builtin_amdgcn_permlane32_swap(t.i[h], t.i[h], false, false)[0];   // rows 0 + 1
  return ((lane & 16) ? t.d : x) + (lane >= 32 ? low.d : 0.0);
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

template <int SR, int SC, int NT>
__global__ __launch_bounds__(NT, 2) void fcm_onchip_kernel(FcmArgs a) {
  extern __shared__ double fcm_lds[];
  constexpr int NW = NT / 64;                        // waves; 4 thread rows (ty) per wave
  constexpr int R = (NT / 16) * SR, C = 16 * SC;     // == a.R, a.C
  double* s_lds = fcm_lds;                           // [SR * SC][NT]: element (ar, bc) of thread tid
  double* xch = s_lds + SR * SC * NT;                // [2][NW][C]: a wave's column sums, then what the waves before / behind it
                                                     //   hold; column SC tx + bc at 16 bc + tx (no bank conflicts)
  double* tot = xch + 2 * NW * C;                    // [C] column totals
  double* red = tot + C;                             // [2][NW]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int tx = tid & 15, ty = tid >> 4;
  const int i0 = ty * SR, j0 = tx * SC;
  NormalStream rng(a.seed, kStreamVariation, effective_step(a.step, a.step_add));

  {
    const int item = blockIdx.x;
    const int group = item % a.groups;
    const int t1 = item / a.groups;
    const int pol = t1 & 1;
    const int s = (t1 >> 1) % a.S_w;
    const int tile = (t1 >> 1) / a.S_w;
    const int k0 = (tile / a.tiles_c) * R, n0 = (tile % a.tiles_c) * C;
    const int rows = min(R, a.K - k0), cols = min(C, a.N - n0);

#pragma unroll 1
    for (int ar = 0; ar < SR; ++ar)
#pragma unroll 1
      for (int bc = 0; bc < SC; ++bc) {
        const int i = i0 + ar, j = j0 + bc;
        double g = 0.0;
        if (i < rows && j < cols) {
          const double qw = (double)((1u << a.weight_bits) - 1);
          const double wq =
              ::rint(clampd((double)a.W[(size_t)(k0 + i) * a.N + n0 + j] / (double)a.w_max, -1.0, 1.0) * qw);
          const int digit = (int)(((uint32_t)::fabs(wq) >> (a.slice_bits * s)) & ((1u << a.slice_bits) - 1));
          const bool mine = pol == 0 ? wq > 0.0 : wq < 0.0;
          g = a.g_min + (mine ? digit * a.dg : 0.0);
          if (a.flags & XBAR_NI_VARIATION) {
            const uint64_t dev =
                (((uint64_t)(k0 + i) * (uint64_t)a.N + (uint64_t)(n0 + j)) * (uint64_t)a.S_w + (uint64_t)s) * 2 + pol;
            g *= 1.0 + a.var_sigma * rng.get(dev);
          }
        }
        s_lds[(ar * SC + bc) * NT + tid] = ::sqrt(::fmax(g, 0.0));
      }
    // every thread reads back only what it wrote itself: no barrier needed for s_lds

    const int rhs_end = min(rows, (group + 1) * a.rhs_per_group);
    for (int rhs = group * a.rhs_per_group; rhs < rhs_end; ++rhs) {
      double r[SR][SC], p[SR][SC], e = 0.0;          // e: solution summed over column tid
      double part = 0.0;
#pragma unroll
      for (int ar = 0; ar < SR; ++ar)
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          r[ar][bc] = (i0 + ar == rhs) ? s_lds[(ar * SC + bc) * NT + tid] : 0.0;
          p[ar][bc] = 0.0;
          part += r[ar][bc] * r[ar][bc];
        }
      double rr = block_sum_n<NW>(part, red);
      const double stop = a.tol2 * rr;
      double beta = 0.0;
      for (int it = 0; it < a.max_iter && rr > stop; ++it) {
        // p <- r + beta p; u = s p: sums, sums of the sums and their squares inside this thread's patch, rows from the
        // right, columns from above
        double row0[SR], row1[SR], col0[SC], col1[SC];
        double pq = 0.0, row_sq = 0.0, col_sq = 0.0;
#pragma unroll
        for (int x = 0; x < SC; ++x) col0[x] = col1[x] = 0.0;
#pragma unroll
        for (int ar = 0; ar < SR; ++ar) {
          double run = 0.0, runs = 0.0;
#pragma unroll
          for (int bc = SC - 1; bc >= 0; --bc) {
            p[ar][bc] = __builtin_fma(beta, p[ar][bc], r[ar][bc]);
            const double u = s_lds[(ar * SC + bc) * NT + tid] * p[ar][bc];
            pq = __builtin_fma(p[ar][bc], p[ar][bc], pq);
            run += u;
            runs += run;
            row_sq = __builtin_fma(run, run, row_sq);
            col0[bc] += u;
            col1[bc] += col0[bc];
            col_sq = __builtin_fma(col0[bc], col0[bc], col_sq);
          }
          row0[ar] = run;                            // sum of u
          row1[ar] = runs;                           // sum of (j - j0 + 1) u
          // a row at a time: left alone, the compiler sets the chains of squares aside and spills what they wait for
          asm volatile("" : "+v"(pq), "+v"(row_sq), "+v"(col_sq));
        }
        // rows: what lies outside the patch, and p.Ap's row part
        double suffix[SR], left1[SR], energy = a.r_row * row_sq;
#pragma unroll
        for (int ar = 0; ar < SR; ++ar) {
          const double full1 = __builtin_fma((double)j0, row0[ar], row1[ar]);   // sum of (j + 1) u
          const double inc0 = row16_inclusive_scan(row0[ar]), inc1 = row16_inclusive_scan(full1);
          const double total = dpp_row_f64<0x15F>(inc0);   // row_newbcast:15
          const double right = total - inc0;         // sum of u to the right of the patch
          suffix[ar] = a.r_row * (right + row0[ar]); // S at the patch's first column; then the sum over k < j0 of S_k with
          left1[ar] = __builtin_fma(a.r_row, __builtin_fma((double)j0, total - (inc0 - row0[ar]), inc1 - full1), a.r_source * total);
          energy = __builtin_fma(a.r_row * right, __builtin_fma((double)SC, right, 2.0 * row1[ar]), energy);   // the driver's share
          if (tx == 0) energy = __builtin_fma(a.r_source * total, total, energy);
          if (ar & 1) asm volatile("" : "+v"(suffix[ar]), "+v"(left1[ar]), "+v"(energy));
        }
        // columns: sums over the lane groups above inside the wave.  Kept per column: the sum and the sum of (R - i) u down
        // to and with this thread inside the wave, and what multiplies the sum above the wave in the squares of P
        double cross[SC];
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          double inc0 = col0[bc], inc1 = __builtin_fma((double)(R - SR - i0), col0[bc], col1[bc]);
          inc0 = group16_inclusive_scan(inc0, lane);
          inc1 = group16_inclusive_scan(inc1, lane);
          const double in0 = inc0 - col0[bc];        // above this thread, inside the wave
          col_sq = __builtin_fma(in0, __builtin_fma((double)SR, in0, 2.0 * col1[bc]), col_sq);
          cross[bc] = 2.0 * __builtin_fma((double)SR, in0, col1[bc]);
          col0[bc] = inc0;
          col1[bc] = inc1;
          if (bc & 1) asm volatile("" : "+v"(col0[bc]), "+v"(col1[bc]), "+v"(cross[bc]), "+v"(col_sq));
        }
        if (lane >= 48) {                            // last group of the wave holds the wave's sums
#pragma unroll
          for (int bc = 0; bc < SC; ++bc) {
            xch[(0 * NW + wave) * C + 16 * bc + tx] = col0[bc];
            xch[(1 * NW + wave) * C + 16 * bc + tx] = col1[bc];
          }
        }
        __syncthreads();
        if (tid < 2 * C) {                           // one thread per column and kind of sum: prefix / suffix over the waves
          const int kind = tid / C, j = tid % C;
          double* line = xch + kind * NW * C + j;
          double v[NW], run = 0.0;
#pragma unroll
          for (int w = 0; w < NW; ++w) v[w] = line[w * C];
          if (kind == 0) {
#pragma unroll
            for (int w = 0; w < NW; ++w) { line[w * C] = run; run += v[w]; }   // above this wave
            tot[j] = run;
          } else {
#pragma unroll
            for (int w = NW - 1; w >= 0; --w) { run += v[w]; line[w * C] = run; }   // this wave and below
          }
        }
        __syncthreads();
        double lc[SC], pre[SC];                      // from the row below the patch up; P at the patch's last row (both in Ohm units)
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          const double total = tot[16 * bc + tx], above = xch[(0 * NW + wave) * C + 16 * bc + tx];
          const double below1 = xch[(1 * NW + wave) * C + 16 * bc + tx] - col1[bc];
          col_sq = __builtin_fma(above, __builtin_fma((double)SR, above, cross[bc]), col_sq);
          if (ty == 0) energy = __builtin_fma(a.r_sense * total, total, energy);
          const double last = above + col0[bc];
          pre[bc] = a.r_col * last;
          lc[bc] = __builtin_fma(a.r_col, __builtin_fma((double)(R - SR - i0), last, below1), a.r_sense * total);
          if (bc & 1) asm volatile("" : "+v"(pre[bc]), "+v"(lc[bc]), "+v"(col_sq), "+v"(energy));
        }
        pq += __builtin_fma(a.r_col, col_sq, energy);
        pq = block_sum_n<NW>(pq, red + NW);
        const double alpha = rr / pq;
        // r <- r - alpha A p, walking up the rows
        part = 0.0;
#pragma unroll
        for (int ar = SR - 1; ar >= 0; --ar) {
          double suf = suffix[ar], lr = left1[ar];
#pragma unroll
          for (int bc = 0; bc < SC; ++bc) {
            const double sv = s_lds[(ar * SC + bc) * NT + tid];
            const double u = sv * p[ar][bc];
            lr += suf;
            suf = __builtin_fma(-a.r_row, u, suf);
            lc[bc] += pre[bc];
            pre[bc] = __builtin_fma(-a.r_col, u, pre[bc]);
            const double q = __builtin_fma(sv, lr + lc[bc], p[ar][bc]);
            const double rn = __builtin_fma(-alpha, q, r[ar][bc]);
            r[ar][bc] = rn;
            part = __builtin_fma(rn, rn, part);
          }
          asm volatile("" : "+v"(part));
        }
        if (tid < C) e = __builtin_fma(alpha, tot[tid], e);   // column sum of x = s y, y = sum alpha p
        const double rr_new = block_sum_n<NW>(part, red);
        beta = rr_new / rr;
        rr = rr_new;
      }
      if (tid < C) tot[tid] = e;                     // everyone has read the totals: the reduction of rr came after
      __syncthreads();
      if (rhs >= i0 && rhs < i0 + SR) {
#pragma unroll
        for (int bc = 0; bc < SC; ++bc) {
          const int j = j0 + bc;
          if (j < cols) {
            const double sv = s_lds[((rhs - i0) * SC + bc) * NT + tid];
            const double g = sv * sv;
            a.profile[((size_t)(2 * s + pol) * a.K + k0 + rhs) * a.N + n0 + j] =
                g > 0.0 ? (float)((g - tot[16 * bc + tx]) / g) : 0.0f;
          }
        }
      }
      // the next solve writes the totals only behind the barriers of its first reduction
    }
  }
}

constexpr int kFcmThreads128 = 512, kFcmThreads64 = 256;   // fcm_onchip_kernel: 4 x 8 and 4 x 4 devices per thread

struct FcmPlan {
  int n_items, groups, rhs_per_group, blocks;
  int onchip;            // 0: state in the workspace; 64 / 128: square crossbars of that size, state on chip
  size_t lds_bytes, ws_bytes;
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
  {  // s, the column exchange area [2][waves][C], the column totals and two sets of reduction slots
    const int waves = (p.onchip == 128 ? kFcmThreads128 : kFcmThreads64) / 64;
    p.lds_bytes = ((size_t)p.onchip * p.onchip + 2 * waves * p.onchip + p.onchip + 2 * waves) * sizeof(double);
  }
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
  if (p.onchip) {
    const void* fn = p.onchip == 128 ? reinterpret_cast<const void*>(&fcm_onchip_kernel<4, 8, kFcmThreads128>)
                                     : reinterpret_cast<const void*>(&fcm_onchip_kernel<4, 4, kFcmThreads64>);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes) == hipSuccess) {
      if (p.onchip == 128)
        hipLaunchKernelGGL((fcm_onchip_kernel<4, 8, kFcmThreads128>), dim3((unsigned)p.n_items), dim3(kFcmThreads128), p.lds_bytes, st, a);
      else
        hipLaunchKernelGGL((fcm_onchip_kernel<4, 4, kFcmThreads64>), dim3((unsigned)p.n_items), dim3(kFcmThreads64), p.lds_bytes, st, a);
      return hipGetLastError() == hipSuccess ? XBAR_OK : XBAR_EHIP;
    }
    (void)hipGetLastError();                         // no such LDS size on this device: general kernel
  }
  hipLaunchKernelGGL(fcm_kernel, dim3((unsigned)p.blocks), dim3(256), 0, st, a);
  if (hipGetLastError() != hipSuccess) return XBAR_EHIP;
  return XBAR_OK;
}

}  // extern "C"
