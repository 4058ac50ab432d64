// Top-r eigen-subspace of the token Gram matrix by block subspace iteration
// (the rank-r truncated SVD of paper Sec. III-A.3 only needs V_r and Sigma_r).
//
// Only the r dominant eigenpairs of G = Z_M^T Z_M enter the energies, so instead of
// diagonalising all of G, a block of P > r vectors is iterated:
//     Y <- G Y,  Y <- orthonormalise(Y)          (P = r + 64..127; error shrinks by lambda_{P+1}/lambda_r per step)
// and the P x P projection Q^T G Q is split at its r-th eigenvalue (split.hip): U = Pi Q^T spans the dominant subspace and
// c_i = (U (Q^T G))_ii.  All products are fp64 MFMA GEMMs; the cost scales with r, not with M.
//
// Storage is transposed (vectors are rows, Yt is P x nP) so that every product is in the
// K-contiguous "NT" form of the GEMM kernel: (G Y)^T = Yt G^T = Yt G.
// Orthonormalisation is Cholesky-QR: S = Yt Yt^T = L L^T (blocked right-looking Cholesky, 64-wide
// panels, trailing update on the MFMA), Yt <- L^-1 Yt (blocked forward substitution).
// The start block is Omega G with a fixed +-1 pattern Omega, so exact duplicate tokens (equal rows of
// G) cannot make it rank deficient.
// The residual of the dominant subspace, Pi Q^T G - H U, is checked; images that fail (slow decay, P too small, no gap
// at the cut) take four more steps and, if they fail again, the full block Jacobi solve of G.
#include "common.h"
#include "host_cache.h"
#include "kernels.h"

namespace covspec {

namespace {

constexpr int NB = 64;        // panel width of Cholesky / substitution
constexpr int NBP = NB + 1;   // LDS pitch
// Relative residual accepted for the dominant subspace, row by row (split_finish_kernel).  It perturbs an energy by at
// most 1e-9 / (relative gap at r) relative.  A block that took the steps planned for it sits at 2e-10 (kPlanTol) or below,
// one that took all of the first pass at 1e-11..1e-13, unconverged ones orders above.  (Energies as returned, in fp32, are
// 2.6e-8 off their 64-bit values with either, the rounding to fp32.)
constexpr double kRitzTol = 1e-9;
// see the end of chol_kernel
constexpr double kPivotNear = 0.25;   // smallest scaled pivot above this: rows nearly orthogonal, blocks of three steps
constexpr double kPivotFar = 1e-3;    // above this: blocks of two steps
constexpr double kGradeDigits = 14.0; // decimal digits a block's grading (lambda_1 / lambda_P)^steps may use up
constexpr int kMaxBlockSteps = 3;
constexpr double kPlanTol = 2e-10;     // residual that the planned number of steps has to promise (checked: kRitzTol)
constexpr double kPivotOnePass = 0.01; // final step: above this one Cholesky-QR pass leaves the rows orthonormal to ~1e-14
constexpr size_t kCholLdsFixed = (size_t)(2 * NB * NBP + NB) * sizeof(double);   // plus P doubles: the diagonal of S

__global__ void omega_kernel(double* __restrict__ om, int P, int n, int nP) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)P * nP) return;
  const int r = (int)(i / nP), c = (int)(i - (long)r * nP);
  uint32_t h = (uint32_t)r * 0x9E3779B1u ^ ((uint32_t)c + 0x7F4A7C15u) * 0x85EBCA77u;
  h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 12; h *= 0x297A2D39u; h ^= h >> 15;
  om[i] = (c < n) ? ((h & 1u) ? 1.0 : -1.0) : 0.0;
}

// value of `v` in lane `l` (compile-time lane), uniform across the wave
__device__ __forceinline__ double lane_value(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l), hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

// Everything a wave has written to LDS before is read back by it after (its LDS accesses complete in order; this only
// keeps the compiler from moving one across the other).
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Factors the 64 x 64 block `a` (LDS, pitch NBP, lower triangle: a = L L^T) and inverts the factor, in one wave: inv(L) goes
// to `inv` (its tiles above the diagonal are zero already), the diagonal of L to dl.  Pivots are floored at `floor_`.
// By 16 x 16 tiles.  A diagonal tile is eliminated together with a unit matrix, lane = column (lanes 0..15 the tile,
// 16..31 the unit matrix): step k subtracts a_ik / a_kk times row k from row i, the a_ik being the scalars of lane k, and
// leaves the inverse of the unit-diagonal factor in the right half, no exchange through LDS and no column to wait for.  The
// tiles below and the rest of the block follow on the MFMA, then the inverse tile by tile, inv_ts = -inv_tt sum L_tu inv_us:
// the sum comes out of the MFMA in the layout its B operand wants.  A column by column factorisation by one wave with the
// inversion after it by the workgroup took 23 + 14 us of a panel, this takes 11.
__device__ __noinline__ void factor_invert_wave(double* a, double* inv, double* dl, double floor_) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4, c = lane & 31;
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    double x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int hi = i > i16 ? i : i16, lo = i > i16 ? i16 : i;
      const double v = a[(16 * s + hi) * NBP + 16 * s + lo];
      x[i] = c < 16 ? v : (c - 16 == i ? 1.0 : 0.0);
    }
    double mine = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const double piv = fmax(lane_value(x[k], k), floor_);
      double rp = __builtin_amdgcn_rcp(piv);
      rp = fma(rp, fma(-piv, rp, 1.0), rp);
      rp = fma(rp, fma(-piv, rp, 1.0), rp);
      const double row = x[k] * rp;
#pragma unroll
      for (int i = k + 1; i < 16; ++i) x[i] = fma(-lane_value(x[i], k), row, x[i]);
      double rs = __builtin_amdgcn_rsq(piv);
      rs = rs * fma(-0.5 * piv, rs * rs, 1.5);
      rs = rs * fma(-0.5 * piv, rs * rs, 1.5);
      x[k] *= rs;                                  // lanes 16..31: row k of inv(L_ss)
      if (lane == k) mine = piv * rs;
    }
    if (lane < 16) dl[16 * s + lane] = mine;
    if (lane >= 16 && lane < 32) {
#pragma unroll
      for (int k = 0; k < 16; ++k) inv[(16 * s + k) * NBP + 16 * s + i16] = i16 <= k ? x[k] : 0.0;
    }
    wave_lds_fence();
    double wf[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) wf[j] = inv[(16 * s + i16) * NBP + 16 * s + 4 * j + kq];
#pragma unroll 1
    for (int t = s + 1; t < 4; ++t) {              // L_ts = A_ts inv(L_ss)^T
      f64x4_t o = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(16 * t + i16) * NBP + 16 * s + 4 * j + kq], wf[j], o, 0, 0, 0);
      wave_lds_fence();
#pragma unroll
      for (int v = 0; v < 4; ++v) a[(16 * t + 4 * v + kq) * NBP + 16 * s + i16] = o[v];
    }
    wave_lds_fence();
#pragma unroll 1
    for (int t = s + 1; t < 4; ++t)                // A_tu -= L_ts L_us^T
#pragma unroll 1
      for (int u = s + 1; u <= t; ++u) {
        f64x4_t o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = a[(16 * t + 4 * v + kq) * NBP + 16 * u + i16];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          o = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[(16 * t + i16) * NBP + 16 * s + 4 * j + kq], a[(16 * u + i16) * NBP + 16 * s + 4 * j + kq], o, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) a[(16 * t + 4 * v + kq) * NBP + 16 * u + i16] = o[v];
      }
    wave_lds_fence();
  }
#pragma unroll 1
  for (int d = 1; d < 4; ++d) {
#pragma unroll 1
    for (int t = d; t < 4; ++t) {
      const int s = t - d;
      f64x4_t sum = (f64x4_t){0.0, 0.0, 0.0, 0.0}, o = sum;
#pragma unroll 1
      for (int u = s; u < t; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          sum = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(16 * t + i16) * NBP + 16 * u + 4 * j + kq], inv[(16 * u + 4 * j + kq) * NBP + 16 * s + i16], sum, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(-inv[(16 * t + i16) * NBP + 16 * t + 4 * j + kq], sum[j], o, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) inv[(16 * t + 4 * v + kq) * NBP + 16 * s + i16] = o[v];
    }
    wave_lds_fence();
  }
}

// Cholesky factorisation S[b] = L L^T (P x P, P % 64 == 0, [P/16][P/16] tiles in fragment order, those on and below the
// diagonal), one 512-thread workgroup per image, right-looking over 64-wide panels:
//   diagonal block: factored and inverted by one wave (factor_invert_wave); the inverse goes to Dinv[b][J] (its 16 tiles);
//   panel below:    X = S[I,J] inv(L_JJ)^T on the MFMA, in place (these blocks are L[I,J]);
//   next diagonal block: updated by all waves, into LDS; then one wave factors it while the others do the
//   trailing part:  S[I,I'] -= X_I X_I'^T for I' <= I on the MFMA, units of 16 x 32.
// Every product is formed transposed, so that its result is the fragment of the tile it goes to.
// On return the strictly-lower blocks of S hold L; its diagonal blocks are represented by their inverses.
// Pivots are floored at 1e-28 * trace(first block) so that a numerically rank-deficient block cannot
// produce NaNs (the residual check afterwards decides whether the result is usable).
// Bound by the chain of panels (and, from order 384 on, by one compute unit's MFMA rate in the trailing part).  One image of
// order 192 / eight of 384 / sixty-four of 256, us: 168 / 448 / 257 with the block factored column by column, its inverse
// formed by the workgroup and the next diagonal block updated by the wave that factors it; 76 / 220 / 115 without; 69 / 172 / 107
// with the tiles in fragment order.  (256 registers; five are spilled, read back once a panel, outside the loops.)
// Dynamic LDS: 2 * 64 * 65 + 64 + P doubles.
__global__ __launch_bounds__(512) void chol_kernel(double* S, double* __restrict__ Dinv, int P, int* skip_until, int* last_orth, int step,
                                                   int last_free_step, int next_weight, int r, int n_sq, int* hold, int* slow) {
  extern __shared__ double lds[];
  double* a = lds;                  // [64][65] diagonal block, its factor after factor_invert_wave (tiles below the diagonal)
  double* inv = lds + NB * NBP;     // [64][65] the inverse of the factor
  double* dl = lds + 2 * NB * NBP;  // [64] diagonal of the factor
  double* diag0 = dl + NB;          // [P] the diagonal of S before any update: squared row lengths
  const int b = blockIdx.x;
  if (skip_until && skip_until[b] > step) return;   // this image does not orthonormalise at this step
  double* Sb = S + (long)b * P * P;
  double dmin = 1e300, dmax = 0.0, pmin = 1.0;   // extremes of the factor's diagonal, smallest scaled pivot (wave 0, by lane)
  double d0 = 0.0, dr = 0.0, dP = 0.0;           // diagonal of the factor at rows 0, r - 1 and P - 1 (wave 0)
  const int nblk = P / NB, per16 = P / 16;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  auto tile = [&](int rt, int ct) -> double* { return Sb + ((long)rt * per16 + ct) * kFragTile; };
  for (int k = tid; k < P; k += 512) diag0[k] = tile(k >> 4, k >> 4)[frag_at(k & 15, k & 15)];
  for (int e = tid; e < NB * NB; e += 512) inv[(e >> 6) * NBP + (e & 63)] = 0.0;
  for (int t = w; t < 10; t += 8) {                     // t-th tile of a block on or below its diagonal
    const int x = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, y = t - x * (x + 1) / 2;
    const f64x4_t c = frag_load(tile(x, y), lane);
#pragma unroll
    for (int v = 0; v < 4; ++v) a[(16 * x + i16) * NBP + 16 * y + 4 * v + kq] = c[v];
  }
  __syncthreads();
  double floor_ = 0.0;
  for (int i = 0; i < NB; ++i) floor_ += diag0[i];       // the same value in every thread
  floor_ = 1e-300 + 1e-28 * floor_;
  if (w == 0) factor_invert_wave(a, inv, dl, floor_);
  __syncthreads();

  for (int J = 0; J < nblk; ++J) {
    const int j0 = J * NB, jt = 4 * J;
    // here `inv` holds the inverse of the factor of diagonal block J
    if (w == 0) {
      const double d = dl[lane], s0 = diag0[j0 + lane];
      dmin = fmin(dmin, d);
      dmax = fmax(dmax, d);
      if (s0 > 0.0) pmin = fmin(pmin, d * d / s0);
      if (J == (r - 1) / NB) dr = __shfl(d, (r - 1) % NB, 64);
      if (J == 0) d0 = __shfl(d, 0, 64);
      if (J == nblk - 1) dP = __shfl(d, NB - 1, 64);
    }
    for (int t = w; t < 10; t += 8) {
      const int x = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, y = t - x * (x + 1) / 2;
      f64x4_t c;
#pragma unroll
      for (int v = 0; v < 4; ++v) c[v] = inv[(16 * x + i16) * NBP + 16 * y + 4 * v + kq];
      frag_store(Dinv + ((long)b * nblk + J) * NB * NB + (4 * x + y) * kFragTile, lane, c);
    }
    // ---- panel: X = S[I,J] inv^T, 16-row tiles dealt to the waves; inv is lower triangular
    const int below = (P - j0 - NB) / 16;
    for (int t = w; t < below; t += 8) {
      const int rt = jt + 4 + t;
      f64x4_t f[4], out[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) f[c] = frag_load(tile(rt, jt + c), lane);
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        out[y] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c <= y; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            out[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(inv[(16 * y + i16) * NBP + 16 * c + 4 * v + kq], f[c][v], out[y], 0, 0, 0);
      }
#pragma unroll
      for (int y = 0; y < 4; ++y) frag_store(tile(rt, jt + y), lane, out[y]);
    }
    __syncthreads();     // the panel is complete in global memory and `a`, `inv` are free
    if (below == 0) break;
    // ---- the next diagonal block, into LDS: its ten 16 x 16 tiles on and below the diagonal
    for (int t = w; t < 10; t += 8) {
      const int x = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, y = t - x * (x + 1) / 2;
      const int rt = jt + 4 + x, ct = jt + 4 + y;
      f64x4_t fr[4], fc[4], acc = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        fr[c] = frag_load(tile(rt, jt + c), lane);
        fc[c] = frag_load(tile(ct, jt + c), lane);
      }
      const f64x4_t cc = frag_load(tile(rt, ct), lane);
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fc[c][v], fr[c][v], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) a[(16 * x + i16) * NBP + 16 * y + 4 * v + kq] = cc[v] - acc[v];
    }
    __syncthreads();
    // ---- trailing update by waves 1..7, unit = 16 rows of block I x 32 columns of block I' <= I, in contiguous
    //      ranges, so that consecutive units mostly share the columns and their fragments stay in registers (64 columns
    //      would not fit the registers).  Wave 0 factors the next diagonal block meanwhile.
    if (w == 0) {
      factor_invert_wave(a, inv, dl, floor_);
    } else {
      const int nb = below / 4;
      const int units = 4 * nb * (nb + 1);            // 8 * nb (nb + 1) / 2; units 0..7 are the next diagonal block
      const int u0 = 8 + (int)((long)(units - 8) * (w - 1) / 7), u1 = 8 + (int)((long)(units - 8) * w / 7);
      // unit u -> pair index u / 8 -> (I, I2) with I (I + 1) / 2 + I2 = pair index
      int I = 0, I2 = 0;
      {
        int pi = u0 >> 3;
        while ((I + 1) * (I + 2) / 2 <= pi) ++I;
        I2 = pi - I * (I + 1) / 2;
      }
      f64x4_t fb[2][4];
      int have = -1;
#pragma unroll 1
      for (int u = u0; u < u1; ++u) {
        const int q = u & 3, h = (u >> 2) & 1;
        const int rt = jt + 4 + 4 * I + q, ct = jt + 4 + 4 * I2 + 2 * h;
        if (ct <= rt) {                               // a diagonal block: no tile above the diagonal
          f64x4_t fa[4], cc[2];
#pragma unroll
          for (int c = 0; c < 4; ++c) fa[c] = frag_load(tile(rt, jt + c), lane);
          if (have != ct) {
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
              for (int c = 0; c < 4; ++c) fb[y][c] = frag_load(tile(ct + y, jt + c), lane);
            have = ct;
          }
          cc[0] = frag_load(tile(rt, ct), lane);
          if (ct < rt) cc[1] = frag_load(tile(rt, ct + 1), lane);
#pragma unroll
          for (int y = 0; y < 2; ++y) {
            if (ct + y <= rt) {
              f64x4_t acc = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
              for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[y][c][v], fa[c][v], acc, 0, 0, 0);
              frag_store(tile(rt, ct + y), lane, cc[y] - acc);
            }
          }
        }
        if ((u & 7) == 7) {   // next pair
          if (I2 == I) { ++I; I2 = 0; } else ++I2;
        }
      }
    }
    __syncthreads();
  }
  if (w == 0) {
    dmin = wave_min(dmin);
    dmax = wave_max(dmax);
    pmin = wave_min(pmin);
  }
  // How many steps (products with G) the image may take before it orthonormalises again.  Two things limit a
  // block of m steps.  (1) Cholesky-QR needs the SCALED Gram matrix (unit diagonal) to be well conditioned; the raw
  // grading lambda_1 / lambda_P of the rows is harmless.  The scaled pivots L_kk^2 / S_kk (squared sine of the
  // angle between row k and the rows before it) say how close to orthogonal the rows were: the iteration orders
  // the rows like the eigenvectors, and once it has, they stay nearly orthogonal over several steps.  (2) Within a
  // row the wanted direction must not drown in rounding noise along the dominant one: (lambda_1 / lambda_P)^m has
  // to stay well inside the 16 digits; the diagonal of L spans that ratio for the steps of the block just closed.
  if (tid == 0) {
    int m = 1;
    const int begun = hold[b] > last_orth[b] ? hold[b] : last_orth[b];    // first product of the block just factored
    if (step >= 1 && dmin > 0.0) {
      const int closed = step - begun;                              // steps in the block just factored (>= 1)
      const double digits_per_step = log10(fmax(dmax / dmin, 10.0)) / (double)(closed < 1 ? 1 : closed);
      const int by_grade = (int)(kGradeDigits / digits_per_step);
      const int by_pivot = pmin > kPivotNear ? kMaxBlockSteps : (pmin > kPivotFar ? 2 : 1);
      // by_pivot counts products with G; the products that follow multiply by G^next_weight.  by_grade is in
      // products of the block just closed, whose weight is never below that of the next ones.
      const int by_pivot_products = by_pivot / next_weight;
      m = by_pivot_products < by_grade ? by_pivot_products : by_grade;
      if (m < 1) m = 1;
    }
    int next = step + m;                      // the next step that orthonormalises
    if (next > last_free_step) next = last_free_step;     // the final step always does
    // The final step is followed by a second pass (step + 1) that makes the rows orthonormal to rounding; the
    // error of one pass is about 1e-16 times the scaled condition number, so with large pivots it is not needed.
    if (step == last_free_step) next = pmin > kPivotOnePass ? step + 2 : step + 1;
    // How many steps are needed.  The block just closed multiplied orthonormal rows by G^(2 closed), and the rows are
    // ordered: the diagonal of L holds lambda_k^(2 closed), which gives the contraction rho = lambda_P / lambda_r and the
    // grading lambda_1 / lambda_r (within a quarter of the true rho at step 2 on all workloads).  A first pass of s steps
    // leaves a residual of about 2 rho^s; what the G^2 as formed is off by, 1e-16 (lambda_1 / lambda_r)^2, is contracted by
    // the g steps with G itself behind it.  With the rows orthonormal an image may wait out an even number of products (the
    // two blocks swap roles per product) and go on where the pass ends: a decay of 0.01 per step needs 6 steps of the 12.
    if (n_sq > 0 && step >= 2 && step <= n_sq && last_orth[b] >= 1 && hold[b] < 0) {
      const double per = 0.5 / (double)(step - begun);
      const double est = pow(fmax(dP, 1e-300) / fmax(dr, 1e-300), per), grade = pow(d0 / fmax(dr, 1e-300), per);
      const double rho = fmin(1.25 * est, 1.0);
      const int total = last_free_step + 1;
      for (int t = (last_free_step - step) / 2 * 2 + step; t > step; t -= 2) {    // resume at product t
        const int with_sq = n_sq - t > 0 ? n_sq - t : 0, g = total - (t > n_sq ? t : n_sq);
        const int steps = 2 * (step + with_sq) + g;
        if (2.0 * pow(rho, (double)steps) + 1e-16 * grade * grade * pow(rho, (double)g) < kPlanTol) {
          hold[b] = t;
          next = t + 1 < last_free_step ? t + 1 : last_free_step;
          break;
        }
      }
      // an image that this pass cannot bring down to the tolerance skips the split and goes on in the second pass
      if (2.0 * pow(est, (double)(2 * n_sq + total - n_sq)) > 4.0 * kRitzTol) slow[b] = 1;
    }
    skip_until[b] = next;
    last_orth[b] = step;
  }
}

// Yt[b] <- L^-1 Yt[b] (P x nP, pitch nP) by blocked forward substitution with the factor chol_kernel left
// in S (strictly-lower blocks) and Dinv (inverted diagonal blocks), both tiles in fragment order.  Columns are independent: each wave
// owns 16 of them and never reads what another wave writes, so the whole solve is one launch.
//   for block row bi:  T = Yt[bi] - sum_{K<bi} L[bi,K] Yt[K];   Yt[bi] = inv(L_bibi) T
// What the MFMA returns (lane = column, register = k) is exactly the layout its B operand wants, so the solved blocks are
// kept in registers and are the B operands of the following rows as they are; the A operands are a stream that is known in
// advance, four groups of 16 k of it in flight.  Nothing waits for memory but the first group: the chain is MFMAs.
// Written back to memory and read again block by block, with the loads of a block in front of its MFMAs, the solve took,
// us: 192 x 320 29, 192 x 1280 batch 4 33, 384 x 1152 batch 8 91, 256 x 640 batch 64 145; in registers 26, 30, 83, 127; with
// the factor in fragment order (row-major, a load touched 64 cache lines) 15, 19, 45, 76.
// Instantiated for up to six blocks (rank 320); larger factors go through trsm_any_kernel.  us, trsm_any_kernel / here: 192 x 320
// batch 8 37 / 17, 256 x 640 54 / 23, 384 x 1152 99 / 45; seven blocks measured 124 / 57 and eight 151 / 72 (448 x 704, 512 x 832).
template <int N>
struct TrsmAt {          // group N of the A stream: block row bi takes 4 bi groups of L and 4 of its inverted diagonal block
  static constexpr int row() { int bi = 0; while (2 * (bi + 1) * (bi + 2) <= N) ++bi; return bi; }
  static constexpr int bi = row(), at = N - 2 * bi * (bi + 1), K = at >> 2, q = at & 3;
};

struct TrsmPtr { const double *L, *D; double* Y; long nP; };      // lane offsets included

template <int NBLK, int N>
__device__ __forceinline__ void trsm_fetch(const TrsmPtr& p, f64x4_t (&f)[4]) {
  if constexpr (N < 2 * NBLK * (NBLK + 1)) {
    typedef TrsmAt<N> A;
#pragma unroll
    for (int x = A::K < A::bi ? 0 : A::q; x < 4; ++x)     // the inverted block is lower triangular
      f[x] = A::K < A::bi ? frag_load(p.L + ((long)(4 * A::bi + x) * (4 * NBLK) + 4 * A::K + A::q) * kFragTile, 0)
                          : frag_load(p.D + (16 * A::bi + 4 * x + A::q) * kFragTile, 0);
  }
}

template <int NBLK, int N>
__device__ __forceinline__ void trsm_steps(const TrsmPtr& p, f64x4_t (&y)[NBLK][4], f64x4_t (&f)[4][4], f64x4_t (&acc)[4], f64x4_t (&rhs)[4]) {
  if constexpr (N < 2 * NBLK * (NBLK + 1)) {
    typedef TrsmAt<N> A;
    if constexpr (A::at == 0) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        acc[x] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) rhs[x][v] = p.Y[(long)(A::bi * NB + 16 * x + 4 * v) * p.nP];
      }
    }
    if constexpr (A::K == A::bi && A::q == 0) {         // T is complete; the inverted block takes it as its B operand
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        rhs[x] = rhs[x] - acc[x];
        acc[x] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double bv = A::K < A::bi ? y[A::K][A::q][v] : rhs[A::q][v];
#pragma unroll
      for (int x = A::K < A::bi ? 0 : A::q; x < 4; ++x) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[N & 3][x][v], bv, acc[x], 0, 0, 0);
    }
    trsm_fetch<NBLK, N + 4>(p, f[N & 3]);
    __builtin_amdgcn_sched_barrier(0);                  // the loads stay four groups ahead of their use
    if constexpr (A::K == A::bi && A::q == 3) {
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        y[A::bi][x] = acc[x];
#pragma unroll
        for (int v = 0; v < 4; ++v) p.Y[(long)(A::bi * NB + 16 * x + 4 * v) * p.nP] = acc[x][v];
      }
    }
    trsm_steps<NBLK, N + 1>(p, y, f, acc, rhs);
  }
}

template <int NBLK>
__global__ __launch_bounds__(256, 1) void trsm_kernel(double* Yt, const double* __restrict__ S, const double* __restrict__ Dinv, int nP,
                                                      int wg_per_image, const int* __restrict__ last_orth, int step) {
  const int b = blockIdx.x / wg_per_image, cw = blockIdx.x - b * wg_per_image;
  if (last_orth && last_orth[b] != step) return;    // the factorisation of this step did not run for this image
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  constexpr int P = NBLK * NB;
  TrsmPtr p;
  p.L = S + (long)b * P * P + 2 * lane;
  p.D = Dinv + (long)b * NBLK * NB * NB + 2 * lane;
  p.Y = Yt + (long)b * P * nP + (long)kq * nP + cw * 64 + w * 16 + i16;     // nP % 64 == 0, so every column exists
  p.nP = nP;
  f64x4_t y[NBLK][4], f[4][4], acc[4], rhs[4];
  trsm_fetch<NBLK, 0>(p, f[0]);
  trsm_fetch<NBLK, 1>(p, f[1]);
  trsm_fetch<NBLK, 2>(p, f[2]);
  trsm_fetch<NBLK, 3>(p, f[3]);
  trsm_steps<NBLK, 0>(p, y, f, acc, rhs);
}

// The same for any number of blocks: the solved blocks go through memory.
__global__ __launch_bounds__(256) void trsm_any_kernel(double* Yt, const double* __restrict__ S, const double* __restrict__ Dinv,
                                                        int P, int nP, int wg_per_image, const int* __restrict__ last_orth, int step) {
  const int b = blockIdx.x / wg_per_image, cw = blockIdx.x - b * wg_per_image;
  if (last_orth && last_orth[b] != step) return;    // the factorisation of this step did not run for this image
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  const int col = cw * 64 + w * 16 + i16;    // nP % 64 == 0, so every column exists
  const int nblk = P / NB;
  double* Yb = Yt + (long)b * P * nP;
  const double* Lb = S + (long)b * P * P;
  for (int bi = 0; bi < nblk; ++bi) {
    f64x4_t acc[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[x] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    for (int kk = 0; kk < bi * NB; kk += 16) {
      f64x4_t fa[4];
      double fb[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) fa[x] = frag_load(Lb + ((long)(4 * bi + x) * (P / 16) + kk / 16) * kFragTile, lane);
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) fb[jj] = Yb[(long)(kk + 4 * jj + kq) * nP + col];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[x][jj], fb[jj], acc[x], 0, 0, 0);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[x][v] = Yb[(long)(bi * NB + 16 * x + 4 * v + kq) * nP + col] - acc[x][v];
    const double* Db = Dinv + ((long)b * nblk + bi) * NB * NB;
    f64x4_t out[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) out[a] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    // step (x, v) contracts k = 16x + 4v + kq, the row acc[x][v] holds in this lane; the inverse is lower triangular
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int a = x; a < 4; ++a) {
        const f64x4_t da = frag_load(Db + (4 * a + x) * kFragTile, lane);
#pragma unroll
        for (int v = 0; v < 4; ++v) out[a] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[v], acc[x][v], out[a], 0, 0, 0);
      }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) Yb[(long)(bi * NB + 16 * a + 4 * v + kq) * nP + col] = out[a][v];
    __threadfence_block();   // the rows just written are B operands of the next block rows
  }
}

// skip_until[b] = ok[b] ? INT_MAX : -1 (images that passed take no further part), last_orth[b] = hold[b] = -1, slow[b] = 0
__global__ void mask_passed_kernel(const int* __restrict__ ok, int* __restrict__ skip_until, int* __restrict__ last_orth, int* __restrict__ hold,
                                   int* __restrict__ slow, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  skip_until[b] = ok[b] ? 0x7fffffff : -1;
  last_orth[b] = -1;
  hold[b] = -1;
  slow[b] = 0;
}

}  // namespace

int subspace_block(int n, int r) {
  // P = r + 64 rounded up to the panel width: the split costs P^3 per step and each iteration P^2 n, while a wider
  // block only buys a better contraction factor lambda_{P+1}/lambda_r per step, so the narrow block with a
  // few more steps is the cheaper trade.  0 = not worthwhile (P would be most of n).
  int P = (r + 64 + NB - 1) / NB * NB;
  return (4 * P <= 3 * n) ? P : 0;
}

size_t subspace_workspace_bytes(int B, int n, int nP, int P) {
  if (P <= 0) return split_direct(nP) ? 3 * (size_t)B * nP * nP * 8 + split_scratch_bytes(B, nP) + 256 : 0;
  const size_t blk = (size_t)B * P * nP * 8;
  return 2 * blk + (size_t)P * nP * 8 + 3 * (size_t)B * P * P * 8 + (size_t)B * P * NB * 8 + split_scratch_bytes(B, P) + 256 + 4 * (size_t)B * 4 + 256 + (size_t)B * nP * nP * 8 /* G^2 */ + 256;
}

// The first pass makes iters steps of the iteration as iters / 3 products with G^2 followed by iters / 3 with G.
// Launches of the probed shape: start block and the products of the first pass.
int subspace_product_launches(int iters) { return 2 * (iters / 3) + 1; }

hipError_t launch_subspace_eigen(const double* G, int B, int n, int nP, int r, int P, int iters, int more_iters, void* ws_, int* ok,
                                 float* c, int* img_status, hipEvent_t probe_begin, hipEvent_t probe_end, hipStream_t st) {
  if (P == 0) {
    // the whole matrix is the window
    if (!split_direct(nP)) return hipErrorInvalidValue;
    const size_t sq = (size_t)B * nP * nP;
    double* X0 = (double*)ws_;
    double *Y = X0 + sq, *X1 = Y + sq;
    void* scratch = (void*)(((uintptr_t)(X1 + sq) + 255) & ~(uintptr_t)255);
    const hipError_t ed = launch_spectral_split(G, B, nP, r, false, X0, Y, X1, scratch, nullptr, img_status, st);
    return ed != hipSuccess ? ed : launch_direct_energy(G, Y, B, n, nP, r, scratch, ok, c, st);
  }
  hipError_t e0;
  if (P <= 0 || P % NB != 0 || P > n || P > 4096 || nP % NB != 0) return hipErrorInvalidValue;
  if (iters < 3 || iters % 3 != 0 || more_iters < 1) return hipErrorInvalidValue;
  {
    static PerDeviceInt raised;
    if ((e0 = ensure_dynamic_lds(raised, (const void*)chol_kernel, kCholLdsFixed + 4096 * sizeof(double))) != hipSuccess) return e0;
  }
  char* ws = (char*)ws_;
  const size_t blk = (size_t)B * P * nP * 8;
  double* Yt = (double*)ws;
  double* Zt = (double*)(ws + blk);
  double* Om = (double*)(ws + 2 * blk);
  double* S = (double*)(ws + 2 * blk + (size_t)P * nP * 8);
  double* H = S + (size_t)B * P * P;
  double* D = H + (size_t)B * P * P;
  double* Pi = D + (size_t)B * P * NB;                                                      // [B][P][P] the projector
  void* scratch = (void*)(((uintptr_t)(Pi + (size_t)B * P * P) + 255) & ~(uintptr_t)255);
  int* skip_until = (int*)((char*)scratch + split_scratch_bytes(B, P));                     // [B] next step that orthonormalises
  int* last_orth = skip_until + B;                                                          // [B] step of the last one
  int* hold = last_orth + B;                                                                // [B] products before this one are left out
  int* slow = hold + B;                                                                     // [B] no split at the end of the first pass
  double* G2 = (double*)(((uintptr_t)(slow + B) + 255) & ~(uintptr_t)255);             // [B][nP][nP] G squared
  // after the products with G^2 its place is free: one of the iterates of the split (P <= nP), then U, its partial energies
  // and the partial row lengths of the residual: nP (P + P / 32 + P / 32) <= nP^2 doubles per image, as P <= 3/4 n
  double* U = G2;
  double* cpart = U + (size_t)B * P * nP;                                                   // [B][P / 32][nP]
  double* rnorm = cpart + (size_t)B * (P / kSymTile) * nP;                                       // [B][P][nP / 32]
  hipError_t e;

  // Second pass: images that passed the first check take no further part; the kernels see them as skip_until ==
  // INT_MAX (never reached by a step counter), which is what `masked` switches on for the plain products.
  bool masked = false;
  auto mask = [&](GemmArgs& g) {
    if (masked) { g.skip = skip_until; g.skip_if = 0x7ffffffe; }
    else { g.skip = slow; g.skip_if = 0; }
  };
  auto gemm_yt_g = [&](const double* X, double* out, const double* Gop, int it) {   // out = X Gop  (P x nP), Gop = G or G^2; product `it`
    GemmArgs g;
    g.A = X; g.B = Gop; g.C = out; g.M = P; g.N = nP; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = nP;
    g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)nP * nP; g.strideC = (long)P * nP;
    g.epilogue = EPI_STORE_F64;
    if (masked) mask(g);
    else { g.skip = hold; g.skip_if = it; }
    return launch_gemm64_nt(g, true, true, st);
  };
  // X <- L^-1 X with X X^T = L L^T.  Images with skip_until[b] > step leave X alone, and the factorisation decides
  // how many steps the image takes before the next one (never beyond last_free_step).
  const size_t chol_lds = kCholLdsFixed + (size_t)P * sizeof(double);
  auto cholqr = [&](double* X, int step, int last_free_step, int next_weight, int n_sq) -> hipError_t {
    GemmArgs g;
    g.A = X; g.B = X; g.C = S; g.M = P; g.N = P; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = P;
    g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)P * nP; g.strideC = (long)P * P;
    g.epilogue = EPI_STORE_F64;
    g.frag = true;
    g.skip = skip_until;
    g.skip_if = step;
    if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(chol_kernel, dim3((unsigned)B), dim3(512), chol_lds, st, S, D, P, skip_until, last_orth, step, last_free_step,
                       next_weight, r, n_sq, hold, slow);
    const dim3 tg((unsigned)(B * (nP / NB)));
    const double *cS = S, *cD = D;
    const int* orth = last_orth;
    switch (P / NB) {
#define COVSPEC_TRSM(n) \
  case n: hipLaunchKernelGGL(trsm_kernel<n>, tg, dim3(256), 0, st, X, cS, cD, nP, nP / NB, orth, step); break;
      COVSPEC_TRSM(2)
      COVSPEC_TRSM(3)
      COVSPEC_TRSM(4)
      COVSPEC_TRSM(5)
      COVSPEC_TRSM(6)
#undef COVSPEC_TRSM
      default: hipLaunchKernelGGL(trsm_any_kernel, tg, dim3(256), 0, st, X, cS, cD, P, nP, nP / NB, orth, step);
    }
    return hipGetLastError();
  };
  double* cur = Yt;
  double* oth = Zt;
  // `steps` products from the block in `cur` (each preceded by an orthonormalisation where the image's schedule
  // asks for one), then the split, the residual check and the energies.
  // The first n_sq products multiply by G^2: two steps of the iteration at the cost of one (the same subspace as
  // two products with G and an orthonormalisation between them).  G^2 as formed is off by about 1e-16 |G|^2, which
  // is a fixed perturbation of the operator of relative size 1e-16 (lambda_1 / lambda_r)^2 at the r-th eigenvalue
  // (1e-8 for a spectrum that falls by 1e4 down to r); the products with G itself that follow contract that error
  // like any other, and a CPU model of the workloads' matrices needs three to four of them.  The last product
  // feeds the split and the residual check and is with G in any case.
  auto pass = [&](int n_sq, int n_plain, int pass_no) -> hipError_t {
    const int steps = n_sq + n_plain;
    for (int it = 0; it < steps; ++it) {
      // the block of step 0 is not (orthonormal) x G, so its factor says nothing about the next step (the kernel
      // takes one step after it); the last step always orthonormalises, twice where its pivots ask for it
      const int w = it < n_sq ? 2 : 1;
      if ((e = cholqr(cur, it, steps - 1, w, n_sq)) != hipSuccess) return e;
      if (it + 1 == steps && (e = cholqr(cur, it + 1, steps - 1, 1, 0)) != hipSuccess) return e;
      if ((e = gemm_yt_g(cur, oth, w == 2 ? G2 : G, it)) != hipSuccess) return e;   // last: oth = Q^T G
      double* t = cur; cur = oth; oth = t;
    }
    // now oth = Q^T (orthonormal rows), cur = Q^T G.  H = (Q^T G) Q
    {
      GemmArgs g;
      g.A = cur; g.B = oth; g.C = H; g.M = P; g.N = P; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = P;
      g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)P * nP; g.strideC = (long)P * P;
      g.epilogue = EPI_STORE_F64;
      g.lower_only = true;      // H is symmetric: the tiles below the diagonal are mirrored
      g.mirror = true;
      mask(g);
      if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
    }
    if ((e = launch_spectral_split(H, B, P, r, true, S, Pi, G2, scratch, masked ? (const int*)ok : (const int*)slow, img_status, st)) != hipSuccess) return e;
    // U = Pi Q^T, and the energies (U Q^T G)_ii
    {
      GemmArgs g;
      g.A = Pi; g.B = oth; g.C = U; g.D = cur; g.dots = cpart; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * nP;
      mask(g);
      if ((e = launch_gemm64_store_dot(g, st)) != hipSuccess) return e;
    }
    // row lengths of the residual Pi Q^T G - H U
    {
      GemmArgs g;
      g.A = Pi; g.B = cur; g.A2 = H; g.B2 = U; g.C = rnorm; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP / kSymTile;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * (nP / kSymTile);
      mask(g);
      if ((e = launch_gemm64_rownorm_dual(g, st)) != hipSuccess) return e;
    }
    return launch_split_finish(H, Pi, rnorm, nP / kSymTile, cpart, P / kSymTile, B, P, n, nP, r, kRitzTol, scratch, slow, ok, pass_no, c, st);
  };

  // G^2 (symmetric: tiles on and below the diagonal, mirrored)
  {
    GemmArgs g;
    g.A = G; g.B = G; g.C = G2; g.M = nP; g.N = nP; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = nP;
    g.batch = B; g.strideA = (long)nP * nP; g.strideB = (long)nP * nP; g.strideC = (long)nP * nP;
    g.epilogue = EPI_STORE_F64;
    g.lower_only = true;
    g.mirror = true;
    if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
  }
  // start block: Omega G
  hipLaunchKernelGGL(omega_kernel, dim3((unsigned)(((long)P * nP + 255) / 256)), dim3(256), 0, st, Om, P, n, nP);
  if (probe_begin && (e = hipEventRecord(probe_begin, st)) != hipSuccess) return e;
  {
    GemmArgs g;
    g.A = Om; g.B = G; g.C = Yt; g.M = P; g.N = nP; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = nP;
    g.batch = B; g.strideA = 0; g.strideB = (long)nP * nP; g.strideC = (long)P * nP;
    g.epilogue = EPI_STORE_F64;
    if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
  }
  if (probe_end && (e = hipEventRecord(probe_end, st)) != hipSuccess) return e;
  if ((e = launch_fill_int(skip_until, 3 * B, -1, st)) != hipSuccess) return e;
  if ((e = launch_fill_int(slow, B, 0, st)) != hipSuccess) return e;
  if ((e = pass(iters / 3, iters / 3, 1)) != hipSuccess) return e;
  // images whose subspace is not there yet (slower spectral decay than the first pass allows for) go on from Q^T G
  // for a few more steps; for the others every kernel of this pass returns at once
  masked = true;
  hipLaunchKernelGGL(mask_passed_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, st, (const int*)ok, skip_until, last_orth, hold, slow, B);
  return pass(0, more_iters, 2);
}

}  // namespace covspec
