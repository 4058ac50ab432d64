// Top-r eigen-subspace of the token Gram matrix by block subspace iteration
// (the rank-r truncated SVD of paper Sec. III-A.3 only needs V_r and Sigma_r).
//
// Only the r dominant eigenpairs of G = Z_M^T Z_M enter the energies, so instead of
// diagonalising all of G, a block of P > r vectors is iterated:
//     Y <- p(G) Y,  Y <- orthonormalise(Y)       (P = r + 64..127)
// with p the Chebyshev polynomial of [0, lambda_P]: of all polynomials of m products it grows fastest beyond that interval, so
// that m products shrink the error by T_m(2 lambda_r / lambda_P - 1), about (4 lambda_r / lambda_P)^m / 2 for a fast decay and
// 2.4^m where lambda_r is only 1.2 lambda_P, against (lambda_r / lambda_P)^m for m products with G itself.  How many products a
// block takes and how many blocks there are is decided per image from the factor's diagonal (plan_block).
// Before: 12 or 16 steps with G or G^2 (formed once per call) and an orthonormalisation after one to three of them.  G^2 costs n / 2P
// products and loses (lambda_1 / lambda_r)^2 of the 1e-16, which products with G behind it had to contract again.
// us per covspec_select: four of n = 1638, P = 192 (9 products, G^2, 7 factorisations -> 10 and 4) 2890 -> 2140; a frame of four
// videos, n = 1280 (second pass, 11 factorisations -> 5) 2590 -> 1800; sixty-four of 640, P = 256 (7 -> 4) 7.0 -> 6.1 ms.
// The P x P projection Q^T G Q is split at its r-th eigenvalue (split.hip): U = Pi Q^T spans the dominant subspace and
// c_i = (U (Q^T G))_ii.  All products are fp64 MFMA GEMMs; the cost scales with r, not with M.
//
// Storage is transposed (vectors are rows, Yt is P x nP) so that every product is in the
// K-contiguous "NT" form of the GEMM kernel: (G Y)^T = Yt G^T = Yt G.
// Orthonormalisation is Cholesky-QR: S = Yt Yt^T = L L^T (by block rows of 64, a workgroup each), Yt <- L^-1 Yt (blocked forward
// substitution).
// The start block is Omega G with a fixed +-1 pattern Omega, so exact duplicate tokens (equal rows of
// G) cannot make it rank deficient.
// The residual of the dominant subspace, Pi Q^T G - H U, is checked; images that fail (slow decay, P too small, no gap
// at the cut) take up to two further blocks and, if they fail again, the full block Jacobi solve of G.
#include "common.h"
#include "host_cache.h"
#include "kernels.h"

namespace covspec {

namespace {

constexpr int NB = 64;        // panel width of Cholesky / substitution
constexpr int NBP = NB + 1;   // LDS pitch
// Relative residual accepted for the dominant subspace, row by row (split_finish_kernel).  It perturbs an energy by at
// most 1e-9 / (relative gap at r) relative.  Blocks are planned to a residual of 2e-10 (plan_block: to 4e-10 where the first pass ends,
// 8e-10 to 2e-9 where a steep image's second does) and sit at 1e-14 to 4e-10, unconverged ones orders above.  (Energies as returned, in
// fp32, are 2.6e-8 off their 64-bit values with either, the rounding to fp32.)
constexpr double kRitzTol = 1e-9;
// A last factorisation leaves rows with inner products of about 1e-16 over its smallest scaled pivot, up to 1e-6 at this line, typically
// 1e-9 and less.  They enter the residual of the check in full (Q G - H Q is H times them), which refuses what exceeds it; below the line
// the image is not split and goes on in the second pass.
constexpr double kPivotOnePass = 1e-10;
constexpr double kPivotFloor = 1e-14;  // see chol_kernel
constexpr double kLn10 = 2.302585092994046;
constexpr float kSteep = 9.0f;         // ln(lambda_1 / lambda_P) from which growth and not launches limit a block of three products

constexpr size_t kCholLds = (size_t)2 * NB * NBP * sizeof(double);
constexpr int kMaxBlocks = 64;         // block rows: P <= 4096

__global__ void omega_kernel(double* __restrict__ om, int P, int n, int nP) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)P * nP) return;
  const int r = (int)(i / nP), c = (int)(i - (long)r * nP);
  uint32_t h = (uint32_t)r * 0x9E3779B1u ^ ((uint32_t)c + 0x7F4A7C15u) * 0x85EBCA77u;
  h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 12; h *= 0x297A2D39u; h ^= h >> 15;
  om[i] = (c < n) ? ((h & 1u) ? 1.0 : -1.0) : 0.0;
}

// ---- The schedule of an image.  Orthonormalisations are numbered; before orthonormalisation k the kernels read state k of the
// image, the factorisation writes state k + 1, the products behind it read that.  Four integers per image and state:
//   ST_REST  0: takes part in the next orthonormalisation, 1: in the last one of the pass only, 2: in none of this pass
//   ST_IDLE  minus the number of products of the block that follows
//   ST_SEL, ST_END  the buffer its first operand is in, and the one its result is in (products alternate between the two)
enum { ST_REST, ST_IDLE, ST_SEL, ST_END, ST_FIELDS };
constexpr int kMaxDegrees = 6;
struct IterPlan {
  double tb;      // 2 / beta, beta = the upper end of the damped interval; 0: the block's products are with G itself
  float l1, s;    // ln(lambda_1 / beta); how far the rows are separated from the leading ones, ln of the growth so far
  float y;        // what lies beyond beta grows like cosh(m y) over m products: acosh(2 lambda_P / beta - 1), 0 where beta is above lambda_P
  int pw, n, m[kMaxDegrees]; // products with G up to the first estimate; Chebyshev blocks so far and their degrees
  int redo;       // failed the check: the last product was with G, from orthonormal rows
  int there;      // second pass: with the block under way, by its estimate, the image is there
};
struct PlanArgs {
  const int* in;  // states of this orthonormalisation and of the next, [ST_FIELDS][B] each
  int* out;
  IterPlan* plan;
  int* left;      // [B] nothing left to do for the image in this pass
  int B, r;
  int slots;      // products that may follow; 0: the last orthonormalisation of the pass, Q G follows
  int first;      // the very first: nothing is known about the spectrum yet
  int pass;
  int closing;    // the last block of the pass follows
};
// Products that may follow: two between the first two orthonormalisations (the spectrum is not known yet), then as
// many as tell the rows apart, three or four at most (plan_block; a launch that no image needs costs 2 us); kSlots2: the second pass.
constexpr int kBlocks = 3, kSlots[kBlocks] = {2, 3, 4}, kBlocks2 = 2, kSlots2[kBlocks2] = {3, 2};
constexpr int kStates1 = kBlocks + 2, kStates = kStates1 + kBlocks2 + 2;       // the first pass's and all
constexpr int kOrths = kBlocks + 1;            // of the first pass; the second has fewer
static_assert(kBlocks2 <= kBlocks && kBlocks + kBlocks2 <= kMaxDegrees, "");


__device__ __forceinline__ float ln_cosh(float t) { return t + log1pf(expf(-2.0f * t)) - 0.6931472f; }
// acosh(e^v) for v >= 0
__device__ __forceinline__ float acosh_exp(float v) { return v + logf(1.0f + sqrtf(fmaxf(0.0f, 1.0f - expf(-2.0f * v)))); }
// ln(lambda / beta) where T_1 of lambda is cosh(t)
__device__ __forceinline__ float over_beta(float t) { return t > 10.0f ? t - 1.3862944f : logf(0.5f + 0.5f * coshf(t)); }

// Decides what follows an orthonormalisation from the diagonal of its factor (rows 0, r - 1 and P - 1: d1, dr, dP) and its smallest
// scaled pivot (L_kk^2 / S_kk, the squared sine between row k and the rows before it).  The rows are ordered like the
// eigenvectors, so after m products with G from orthonormal rows the diagonal holds lambda_k^m: within a quarter of lambda_P and a
// third of lambda_r after the first block on the token matrices of all workloads.  After a Chebyshev block it holds T_m.
//   products needed: the error, from x^-pw / T_m1 / T_m2 ... with x = lambda_r / beta, has to
//     come below 2e-10;
//   products possible in one block: with growth e^b between the first row and the last, a rounding error of the size eps in row
//     k along row 1 becomes eps e^b of it.  eps is e^-s while the rows are not yet separated any further, else what the
//     factorisation left: 1e-16 over the pivot for the row that has it, taken as 1e-19 over it for the last rows, for steep spectra as 3e-19
//     and in the second pass, behind which is only the full solve, as 1e-18 (1e-19 for these too: some run out of blocks; 1e-17: more need the
//     second pass).  Cholesky-QR stands eps e^b of 3e4 (a scaled pivot of 1e-9), and 1e3 (3e2) at the last one, which is not repeated.  A row whose pivot drowns all
//     the same starts again from what rounding left of it (kPivotFloor).
// A steep spectrum (kSteep) allows two or three products a block where the launches allow three or four, and needs more blocks than the
// first pass has.  Its image, if it is further from its end than a block of the second pass reaches, takes the last orthonormalisation of
// the first too, with one product of a block where the others form Q G, and may take two blocks in the second pass; others take one
// there.  (With four blocks in all lambda_k = 1 / k^3 of 512 rows, r = 64, ended in the full solve, 22 ms where 2 suffice, and so did one in
// some four hundred token matrices of 1152 rows, r = 288, 110 ms.)
// Modelled in fp64 on the token matrices and on spectra from x = 1.2 to 1e5, lambda_1 / lambda_P from 2 to 5e7.
__device__ __forceinline__ void plan_block(const PlanArgs& q, int b, double d1, double dr, double dP, double pmin) {
  IterPlan& p = q.plan[b];
  int* out = q.out + b;
  const int at = q.in[ST_END * q.B + b];          // the trsm works in place
  int m = 0, rest = 0;
  const bool sane = dP > 0.0 && d1 < 1e300 && dr > 0.0 && dr < 1e300 && pmin > 0.0;
  if (q.first) {
    // The diagonal of a random block's factor spans a tenth of lambda_1 / lambda_P or more, unless its first row happens to have little of
    // the first eigenvector, and its pivots are some (lambda_P / lambda_1)^2; two products while those that they leave stay above 1e-10.
    m = d1 <= 1e4 * dP && pmin > 3e-10 ? 2 : 1;
    p.tb = 0.0; p.l1 = p.s = p.y = 0.0f; p.pw = 1 + m; p.n = 0; p.redo = 0; p.there = 0;
  } else if (q.slots == 0 && !q.left[b]) {
    if (pmin > kPivotOnePass) {
      m = 1;                                      // Q G
      p.tb = 0.0;
    } else {
      q.left[b] = 1;
    }
  } else if (!sane) {
    q.left[b] = 1;
    rest = 2;
  } else {
    const int slots = q.slots == 0 ? 1 : q.slots;
    float a;                                      // ln(lambda_r / beta)
    if (p.n == 0 || p.redo) {
      const float per = p.redo ? 1.0f : 1.0f / (float)(p.pw - 1);
      const float lP = per * (float)log(dP) + 0.18232f;      // the estimate is up to a fifth low
      p.l1 = fmaxf(0.0f, per * (float)log(d1) - lP);
      if (!p.redo) p.s = (float)p.pw * p.l1;
      p.tb = 2.0 * exp(-(double)lP);
      p.y = 0.0f;
      a = per * (float)log(dr) - lP;
    } else {
      const float per = 1.0f / (float)p.m[p.n - 1];
      a = over_beta(acosh_exp(fmaxf(0.0f, (float)log(dr))) * per);
      if (dP > 1.0) p.y = fmaxf(p.y, acosh_exp((float)log(dP)) * per);
      p.l1 = fmaxf(p.l1, over_beta(acosh_exp(fmaxf(0.0f, (float)log(d1))) * per));    // row 1 of the first blocks may have little of its eigenvector
    }
    const float x = fmaxf(1.0f + 1e-6f, expf(a)), ax = acoshf(2.0f * x - 1.0f);
    const float a1 = p.l1 > 10.0f ? p.l1 + 1.3862944f : acoshf(fmaxf(1.0001f, 2.0f * expf(p.l1) - 1.0f));
    // what a block of m products contracts the error by, and the digits of the error so far, as natural logarithms
    auto gain = [&](int m) { return ln_cosh(ax * (float)m) - (p.y > 0.0f ? ln_cosh(p.y * (float)m) : 0.0f); };
    float e = (float)p.pw * (logf(x) - (p.y > 0.0f ? over_beta(p.y) : 0.0f)) - 0.7f;
    for (int k = 0; k < p.n; ++k) e += gain(p.m[k]);
    // At the end of a pass some of that is left to the residual check where an image would need another block otherwise: the estimate is mostly
    // on the safe side (modelled: 0.4 to 2.7 digits with lambda_1 / lambda_P below 6e4, -0.2 to 2 below 6e5), but not the first one, from
    // powers of G, which has been two digits off, nor those of steeper spectra, where rounding counts.
    const bool steep = p.l1 > kSteep;
    const double digits = !q.closing ? (q.pass == 2 && steep ? 10.0 : 9.7) : q.pass == 1 ? 9.4 : p.l1 < 13.3f ? 9.1 : 9.7;
    const float missing = (float)(digits * kLn10) - e;
    int need = missing <= 0.0f ? 0 : (int)fminf(40.0f, ceilf(acosh_exp(missing) / ax));
    while (p.y > 0.0f && need > 0 && need < 40 && gain(need) < missing) ++need;
    if (need == 0 && (!(pmin > kPivotOnePass) || (p.n == 0 && missing > (float)(-1.5 * kLn10)))) need = 1;
    if (p.redo) need = 40;
    if (p.there && pmin > kPivotOnePass) need = 0;
    p.there = 0;
    if (need == 0) {
      rest = 2;
      if (q.slots == 0) {                         // there after all
        q.left[b] = 0;
        m = 1;
        p.tb = 0.0;
      }
    } else {
      const float spare = (float)((steep && q.pass == 2 ? 2.5 : 3.0) * kLn10);
      const float apart = fmaxf(0.0f, fminf(p.s, (float)log(pmin) + (float)((!steep ? 19.0 : q.pass == 1 ? 18.5 : 18.0) * kLn10)));
      const int most = max(1, min(slots, (int)(acosh_exp(apart + (float)(4.5 * kLn10)) / a1)));
      const int last = max(1, min(slots, (int)(acosh_exp(apart + spare) / a1)));
      if (q.pass == 2) {
        // all images of the pass, done or not, meet at its second orthonormalisation, and the third is left out when all are
        m = min(need, last);
        rest = q.closing;
        p.there = need <= last || !steep;
      } else if (need <= last) {
        m = need;
        rest = 1;
      } else {
        const int blocks = 1 + (need - last + most - 1) / most;
        m = min(most, (need + blocks - 1) / blocks);
        if (q.closing) {                          // not there at the end of this pass: on to the second without a split
          q.left[b] = 1;
          // what a block there reaches from well separated rows; they are behind a block of less than the most
          const int reach = max(1, min(kSlots2[0], (int)(acosh_exp((float)(18.5 * kLn10)) / a1)));
          if (steep) m = min(m, max(need - reach, min(2, last)));
          if (!steep || need - m <= reach + 1) rest = 2;     // (the one more, by its estimate, is mostly not needed)
        }
      }
      p.s += ln_cosh(a1 * (float)m);
      if (p.n < kMaxDegrees) p.m[p.n++] = m;
    }
    p.redo = 0;
  }
  out[ST_REST * q.B] = rest;
  out[ST_IDLE * q.B] = -m;
  out[ST_SEL * q.B] = at;
  out[ST_END * q.B] = (at + m) & 1;
}

// An image that takes no part: its block stays as and where it is; at the end of a pass Q G is formed of one that is to be split.
__device__ __forceinline__ void rest_on(const PlanArgs& q, int b) {
  int* out = q.out + b;
  const int at = q.in[ST_END * q.B + b], m = q.slots == 0 && !q.left[b] ? 1 : 0;
  if (m) q.plan[b].tb = 0.0;
  out[ST_REST * q.B] = q.in[ST_REST * q.B + b];
  out[ST_IDLE * q.B] = -m;
  out[ST_SEL * q.B] = at;
  out[ST_END * q.B] = (at + m) & 1;
}

// Factors the 64 x 64 block `a` (LDS, pitch NBP, lower triangle: a = L L^T) and inverts the factor, by all eight waves: inv(L) goes
// to the tiles of `inv` on and below the diagonal, the diagonal of L to dl.  The pivot of row k is floored at
// kPivotFloor diag[k], diag the diagonal of S.  Ends with a barrier.
// By 16 x 16 tiles.  A diagonal tile is eliminated together with a unit matrix by wave 0, lane = column of both (the four rows of 16
// lanes do the same): step k subtracts a_ik / a_kk times row k from row i, the a_ik coming from lane k of the row in one move,
// and leaves the inverse of the unit-diagonal factor where the unit matrix was, no exchange through LDS and no column to wait for.
// (With the a_ik as two scalars from v_readlane and the unit matrix in other lanes a block took 13.4 us, so 11.4.)  The
// tiles below and the rest of the block follow on the MFMA, a wave per tile, and the inverse tile by tile,
// inv_ts = -inv_tt sum L_tu inv_us, while wave 0 eliminates the next diagonal tile: the sum comes out of the MFMA in the layout its
// B operand wants.  
// Pivot k and its reciprocal: an estimate good to 2^-24, r (1 + e + e^2).  The chain from one pivot to the next is what an elimination
// takes, so the floor is decided beside it.
template <int k>
__device__ __forceinline__ void pivot_of(const double (&x)[16], double floor_, double rfloor, double& piv, double& rp) {
  const double p = row_lane<k>(x[k]), f = row_lane<k>(floor_), rf = row_lane<k>(rfloor);
  const double r = __builtin_amdgcn_rcp(p), e = fma(-p, r, 1.0), good = fma(r, fma(e, e, e), r);
  const bool above = p > f;
  piv = above ? p : f;
  rp = above ? good : rf;
}
// Step k with its pivot and the reciprocal; the next pivot's is worked out beside the rest of the step.
template <int k>
__device__ __forceinline__ void eliminate_step(double (&x)[16], double (&u)[16], double floor_, double rfloor, double piv, double rp, double& mine) {
  if constexpr (k < 16) {
    const double row = x[k] * rp, urow = u[k] * rp;
    double next = 1.0, next_rp = 1.0;
    if constexpr (k < 15) {
      const double m = row_lane<k>(x[k + 1]);
      x[k + 1] = fma(-(m * x[k]), rp, x[k + 1]);
      u[k + 1] = fma(-m, urow, u[k + 1]);
      pivot_of<k + 1>(x, floor_, rfloor, next, next_rp);
    }
#pragma unroll
    for (int i = k + 2; i < 16; ++i) {
      const double m = row_lane<k>(x[i]);
      x[i] = fma(-m, row, x[i]);
      u[i] = fma(-m, urow, u[i]);
    }
    double rs = __builtin_amdgcn_rsq(piv);
    rs = rs * fma(-0.5 * piv, rs * rs, 1.5);
    rs = rs * fma(-0.5 * piv, rs * rs, 1.5);
    u[k] *= rs;                                  // row k of inv(L_ss)
    if ((threadIdx.x & 15) == k) mine = piv * rs;
#pragma unroll
    for (int i = k + 1; i < 16; ++i) asm volatile("" : "+v"(u[i]));   // or the updates of u pile up behind those of x, and spill
    eliminate_step<k + 1>(x, u, floor_, rfloor, next, next_rp, mine);
  }
}

__device__ __forceinline__ void eliminate_tile(double* a, double* inv, double* dl, const double* diag, int s) {
  const int lane = threadIdx.x & 63, i16 = lane & 15;
  double x[16], u[16], mine = 0.0, piv, rp;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int hi = i > i16 ? i : i16, lo = i > i16 ? i16 : i;
    x[i] = a[(16 * s + hi) * NBP + 16 * s + lo];
    u[i] = i16 == i ? 1.0 : 0.0;
  }
  const double floor_ = fma(kPivotFloor, diag[16 * s + i16], 1e-300);
  const double rfloor = 1.0 / floor_;
  pivot_of<0>(x, floor_, rfloor, piv, rp);
  eliminate_step<0>(x, u, floor_, rfloor, piv, rp, mine);
  if (lane < 16) {
    dl[16 * s + lane] = mine;
#pragma unroll
    for (int k = 0; k < 16; ++k) inv[(16 * s + k) * NBP + 16 * s + i16] = i16 <= k ? u[k] : 0.0;
  }
}

// inv_ts = -inv_tt sum over u of L_tu inv_us, one wave
__device__ __forceinline__ void invert_tile(const double* a, double* inv, int t, int s) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
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

__device__ __forceinline__ void factor_invert(double* a, double* inv, double* dl, const double* diag) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    if (w == 0) eliminate_tile(a, inv, dl, diag, s);
    else if (w < s) invert_tile(a, inv, s - 1, w - 1);   // row s - 1 of the inverse, tiles 0 .. s - 2
    __syncthreads();
    const int t = s + w;
    if (w > 0 && t < 4) {                          // L_ts = A_ts inv(L_ss)^T
      f64x4_t o = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(16 * t + i16) * NBP + 16 * s + 4 * j + kq], inv[(16 * s + i16) * NBP + 16 * s + 4 * j + kq], o, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) a[(16 * t + 4 * v + kq) * NBP + 16 * s + i16] = o[v];
    }
    __syncthreads();
    const int x = w < 1 ? 0 : w < 3 ? 1 : 2, y = w - x * (x + 1) / 2, r = s + 1 + x, c = s + 1 + y;
    if (w < 6 && r < 4) {                          // A_rc -= L_rs L_cs^T
      f64x4_t o;
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = a[(16 * r + 4 * v + kq) * NBP + 16 * c + i16];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[(16 * r + i16) * NBP + 16 * s + 4 * j + kq], a[(16 * c + i16) * NBP + 16 * s + 4 * j + kq], o, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) a[(16 * r + 4 * v + kq) * NBP + 16 * c + i16] = o[v];
    }
    __syncthreads();
  }
  if (w < 3) invert_tile(a, inv, 3, w);
  __syncthreads();
}

__device__ __forceinline__ void frag_store_through(double* tile, int lane, const f64x4_t& v) {
  double* t = tile + 2 * lane;
  store_through(t, v[0]);
  store_through(t + 1, v[1]);
  store_through(t + 128, v[2]);
  store_through(t + 129, v[3]);
}

// Progress of the factorisation of one image: written by the workgroup of a block row, polled by those of the rows after it.
// Cleared at the start of a pass.
struct CholFlags {
  unsigned int ticket;          // next block row to hand to a starting workgroup
  int failed;                   // a workgroup gave up waiting
  int cols[kMaxBlocks];         // per block row: columns of L that are in memory
  int done[kMaxBlocks];         // its diagonal block is factored, the inverse is in memory
};

// Waits until *flag >= value; false when the wait is over its limit or another workgroup has given up.  Everything the other
// workgroup stored through the L2 before it raised the flag is visible behind it.  Call uniformly.
__device__ __forceinline__ bool wait_flag(const int* flag, int value, CholFlags* f, int* s_flag, long long limit_ticks) {
  __syncthreads();                                 // the last wait's result has been read
  if (threadIdx.x == 0) {
    int ok = 1;
    const long long t0 = wall_clock64();
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < value) {
      if (__hip_atomic_load(&f->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > limit_ticks) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *s_flag = ok;
  }
  __syncthreads();
  return *s_flag != 0;
}

// Raises a flag when the stores of all waves have been acknowledged.  Call uniformly.
__device__ __forceinline__ void raise_flag(int* flag, int value) {
  __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0) lgkmcnt(0)
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Cholesky factorisation S[b] = L L^T (P x P, P % 64 == 0, [P/16][P/16] tiles in fragment order, those on and below the
// diagonal), one 512-thread workgroup per block row of 64 and image.  The workgroup of block row i:
//   for K < i:  T = S[i,K] - sum over K' < K of L[i,K'] L[K,K']^T;   L[i,K] = T inv(L_KK)^T, in place;   D += L[i,K] L[i,K]^T
//   factors and inverts S[i,i] - D (factor_invert); the inverse goes to Dinv[b][i] (its tiles).
// It waits for row K's columns before the sum and for row K's inverse before the product with it, so that the sum runs while
// row K is being factored; rows are taken in order (a ticket per image), so that a workgroup only waits for rows that have started
// before it, whatever else the device is doing; every wait is bounded.  What the rows hand one another is stored through the L2.
// Every product is formed transposed, so that its result is the fragment of the tile it goes to.
// On return the strictly-lower blocks of S hold L; its diagonal blocks are represented by their inverses.
// A pivot is floored relative to its own row's squared length (rows may differ in length by any number of digits: after a block of
// products they do, by the growth of the first row over the last), at the rounding of S: what is left of a row below that is noise, which
// the floor keeps shorter than the other rows, and the next factorisation makes a row of length one of it.  (At 1e-28 such a row came out
// up to 1e7 long, with as much of the other rows in it, and the image ended in the full solve.)
// Bound by the chain of diagonal blocks: factor, flag, product with the inverse, D.  One workgroup per image, which did the
// trailing updates itself beside the factorisation of the next block by one of its waves, took, us: one image of order 192 67,
// eight of 384 172, sixty-four of 256 98; this 55, 108 and 80 (eleven of the eighteen a row takes are the elimination).
// Dynamic LDS: 2 * 64 * 65 doubles.
__global__ __launch_bounds__(512) void chol_kernel(double* S, double* __restrict__ Dinv, double* __restrict__ diag, double* __restrict__ pivots, int P,
                                                   PlanArgs q, CholFlags* flags, long long limit_ticks) {
  extern __shared__ double lds[];
  double* a = lds;                  // [64][65] diagonal block, its factor after factor_invert (tiles below the diagonal)
  double* inv = lds + NB * NBP;     // [64][65] the inverse of the factor; before: T, then L[i,K]
  __shared__ double dl[NB], diag0[NB];
  __shared__ int s_flag;
  const int b = blockIdx.x % q.B;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  if (q.in[ST_REST * q.B + b] > (q.slots == 0 ? 1 : 0)) {      // no part in this orthonormalisation
    if (tid == 0 && blockIdx.x < (unsigned)q.B) rest_on(q, b);
    return;
  }
  CholFlags* f = flags + b;
  if (tid == 0) s_flag = (int)atomicAdd(&f->ticket, 1u);
  __syncthreads();
  const int row = s_flag, nblk = P / NB, per16 = P / 16;
  double* Sb = S + (long)b * P * P;
  double* Db = Dinv + (long)b * nblk * NB * NB;
  auto tile = [&](int rt, int ct) -> double* { return Sb + ((long)rt * per16 + ct) * kFragTile; };
  if (tid < NB) diag0[tid] = tile(4 * row + (tid >> 4), 4 * row + (tid >> 4))[frag_at(tid & 15, tid & 15)];
  // t-th tile of a block on or below its diagonal; wave w has the tiles w and, w < 2, w + 8
  auto low = [](int t, int& x, int& y) { x = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3; y = t - x * (x + 1) / 2; };
  f64x4_t dacc[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) dacc[e] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  const int rx = w >> 1;                                        // row tile of this wave, column tiles 2 (w & 1) + 0, 1 of the sum
  bool alive = true;
  for (int K = 0; K < row; ++K) {
    f64x4_t t[2];
    const int c0 = 2 * (w & 1);
#pragma unroll
    for (int y = 0; y < 2; ++y) t[y] = frag_load(tile(4 * row + rx, 4 * K + c0 + y), lane);
    if (K > 0) {
      if (!(alive = wait_flag(&f->cols[K], K, f, &s_flag, limit_ticks))) break;
      f64x4_t acc[2];
#pragma unroll
      for (int y = 0; y < 2; ++y) acc[y] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int k = 0; k < K; ++k) {
        f64x4_t fa[4], fb[2][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) fa[c] = frag_load(tile(4 * row + rx, 4 * k + c), lane);
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int c = 0; c < 4; ++c) fb[y][c] = frag_load(tile(4 * K + c0 + y, 4 * k + c), lane);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[y] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[y][c][v], fa[c][v], acc[y], 0, 0, 0);
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) t[y] = t[y] - acc[y];
    }
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) inv[(16 * rx + i16) * NBP + 16 * (c0 + y) + 4 * v + kq] = t[y][v];
    if (!(alive = wait_flag(&f->done[K], 1, f, &s_flag, limit_ticks))) break;
    // L[i,K]: this wave's column tiles are 0 and 3, or 1 and 2 (five products each)
    f64x4_t in[4], out[2];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) in[c][v] = inv[(16 * rx + i16) * NBP + 16 * c + 4 * v + kq];
    const int y0 = w & 1, y1 = 3 - (w & 1);
    {
      f64x4_t d0[2], d1[4];
#pragma unroll
      for (int c = 0; c < 2; ++c) if (c <= y0) d0[c] = frag_load(Db + (long)K * NB * NB + (4 * y0 + c) * kFragTile, lane);
#pragma unroll
      for (int c = 0; c < 4; ++c) if (c <= y1) d1[c] = frag_load(Db + (long)K * NB * NB + (4 * y1 + c) * kFragTile, lane);
      out[0] = out[1] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c <= y1) {
#pragma unroll
          for (int v = 0; v < 4; ++v) out[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d1[c][v], in[c][v], out[1], 0, 0, 0);
        }
#pragma unroll
      for (int c = 0; c < 2; ++c)
        if (c <= y0) {
#pragma unroll
          for (int v = 0; v < 4; ++v) out[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d0[c][v], in[c][v], out[0], 0, 0, 0);
        }
    }
    __syncthreads();                                            // T has been read
    frag_store_through(tile(4 * row + rx, 4 * K + y0), lane, out[0]);
    frag_store_through(tile(4 * row + rx, 4 * K + y1), lane, out[1]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      inv[(16 * rx + i16) * NBP + 16 * y0 + 4 * v + kq] = out[0][v];
      inv[(16 * rx + i16) * NBP + 16 * y1 + 4 * v + kq] = out[1][v];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int tt = w + 8 * e;
      if (tt < 10) {
        int x, y;
        low(tt, x, y);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            dacc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(inv[(16 * y + i16) * NBP + 16 * c + 4 * v + kq], inv[(16 * x + i16) * NBP + 16 * c + 4 * v + kq], dacc[e], 0, 0, 0);
      }
    }
    raise_flag(&f->cols[row], K + 1);                           // and L[i,K] in LDS has been read
  }
  if (alive) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int tt = w + 8 * e;
      if (tt < 10) {
        int x, y;
        low(tt, x, y);
        const f64x4_t c = frag_load(tile(4 * row + x, 4 * row + y), lane);
#pragma unroll
        for (int v = 0; v < 4; ++v) a[(16 * x + i16) * NBP + 16 * y + 4 * v + kq] = c[v] - dacc[e][v];
      }
    }
    __syncthreads();
    factor_invert(a, inv, dl, diag0);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int tt = w + 8 * e;
      if (tt < 10) {
        int x, y;
        low(tt, x, y);
        f64x4_t c;
#pragma unroll
        for (int v = 0; v < 4; ++v) c[v] = inv[(16 * x + i16) * NBP + 16 * y + 4 * v + kq];
        frag_store_through(Db + (long)row * NB * NB + (4 * x + y) * kFragTile, lane, c);
      }
    }
    if (w == 0) {
      const double d = dl[lane], s0 = diag0[lane];
      store_through(diag + (long)b * P + row * NB + lane, d);
      const double pm = wave_min(s0 > 0.0 ? fmin(1.0, d * d / s0) : 1.0);       // smallest scaled pivot of the rows
      if (lane == 0) store_through(pivots + (long)b * nblk + row, pm);
    }
    raise_flag(&f->done[row], 1);
  }
  if (row != nblk - 1) {
    if (!alive && tid == 0) __hip_atomic_store(&f->failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (tid != 0) return;
  if (alive) {                                                  // it has waited for all the other rows
    double pmin = 1.0;
    for (int k = 0; k < nblk; ++k) {
      const double pm = pivots[(long)b * nblk + k];
      pmin = pm < pmin || !(pm == pm) ? pm : pmin;
    }
    plan_block(q, b, diag[(long)b * P], diag[(long)b * P + q.r - 1], diag[(long)b * P + P - 1], pmin);
  } else {                                                      // no factor: nothing more for the image in this pass
    __hip_atomic_store(&f->failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    q.left[b] = 1;
    rest_on(q, b);
    q.out[ST_REST * q.B + b] = 2;
  }
}

// Y <- L^-1 Y (P x nP, pitch nP; Y is the image's block in Yt or `other` doubles behind it) by blocked forward substitution with the factor chol_kernel left
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
__global__ __launch_bounds__(256, 1) void trsm_kernel(double* Yt, long other, const double* __restrict__ S, const double* __restrict__ Dinv, int nP,
                                                      int wg_per_image, const int* __restrict__ state, int nimg, int rest_max) {
  const int b = blockIdx.x / wg_per_image, cw = blockIdx.x - b * wg_per_image;
  if (state[ST_REST * nimg + b] > rest_max) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  constexpr int P = NBLK * NB;
  TrsmPtr p;
  p.L = S + (long)b * P * P + 2 * lane;
  p.D = Dinv + (long)b * NBLK * NB * NB + 2 * lane;
  p.Y = Yt + (state[ST_END * nimg + b] ? other : 0) + (long)b * P * nP + (long)kq * nP + cw * 64 + w * 16 + i16;     // nP % 64 == 0, so every column exists
  p.nP = nP;
  f64x4_t y[NBLK][4], f[4][4], acc[4], rhs[4];
  trsm_fetch<NBLK, 0>(p, f[0]);
  trsm_fetch<NBLK, 1>(p, f[1]);
  trsm_fetch<NBLK, 2>(p, f[2]);
  trsm_fetch<NBLK, 3>(p, f[3]);
  trsm_steps<NBLK, 0>(p, y, f, acc, rhs);
}

// The same for any number of blocks: the solved blocks go through memory.
__global__ __launch_bounds__(256) void trsm_any_kernel(double* Yt, long other, const double* __restrict__ S, const double* __restrict__ Dinv,
                                                        int P, int nP, int wg_per_image, const int* __restrict__ state, int nimg, int rest_max) {
  const int b = blockIdx.x / wg_per_image, cw = blockIdx.x - b * wg_per_image;
  if (state[ST_REST * nimg + b] > rest_max) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  const int col = cw * 64 + w * 16 + i16;    // nP % 64 == 0, so every column exists
  const int nblk = P / NB;
  double* Yb = Yt + (state[ST_END * nimg + b] ? other : 0) + (long)b * P * nP;
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

// State 0 of a pass.  First: every block is in buffer 0.  Second: images that passed the check rest; one that was left out of the
// split goes on from its block, one that failed the check from the product with G that followed its last orthonormalisation.  And
// the flags of the pass's factorisations.
__global__ void begin_pass_kernel(int* __restrict__ out, const int* __restrict__ prev, const int* __restrict__ ok, IterPlan* __restrict__ plan,
                                  int* __restrict__ left, int* __restrict__ failed_before, int B, CholFlags* __restrict__ flags, int orths) {
  int* words = (int*)flags;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < orths * B * (int)(sizeof(CholFlags) / sizeof(int)); k += gridDim.x * blockDim.x) words[k] = 0;
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const bool passed = prev && ok[b] != 0, failed = prev && !passed && !left[b];
  const int at = prev ? prev[ST_END * B + b] : 0;
  out[ST_REST * B + b] = passed ? 2 : 0;
  out[ST_IDLE * B + b] = 0;
  out[ST_SEL * B + b] = at;
  out[ST_END * B + b] = at;
  plan[b].redo = failed;
  failed_before[b] = failed;
  left[b] = passed;
}

}  // namespace

inline size_t tail_doubles(int B, int P, int nP) {
  const size_t u = (size_t)nP * (P + 2 * (P / kSymTile)), x1 = (size_t)P * P;
  return (size_t)B * (u > x1 ? u : x1);
}

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
  return 2 * blk + (size_t)P * nP * 8 + 3 * (size_t)B * P * P * 8 + (size_t)B * P * NB * 8 + split_scratch_bytes(B, P) + 256 +
         (size_t)B * (sizeof(IterPlan) + (kStates * ST_FIELDS + 2) * sizeof(int) + kOrths * sizeof(CholFlags) + (P + P / NB) * 8) + 512 + tail_doubles(B, P, nP) * 8 + 256;
}

// Launches of the probed shape: start block and the products of the first pass (blocks that take fewer leave the rest out).
int subspace_product_launches() {
  int n = 2;
  for (int k = 0; k < kBlocks; ++k) n += kSlots[k];
  return n;
}

hipError_t launch_subspace_eigen(const double* G, int B, int n, int nP, int r, int P, void* ws_, int* ok,
                                 float* c, hipEvent_t probe_begin, hipEvent_t probe_end, hipStream_t st) {
  if (P == 0) {
    // the whole matrix is the window
    if (!split_direct(nP)) return hipErrorInvalidValue;
    const size_t sq = (size_t)B * nP * nP;
    double* X0 = (double*)ws_;
    double *Y = X0 + sq, *X1 = Y + sq;
    void* scratch = (void*)(((uintptr_t)(X1 + sq) + 255) & ~(uintptr_t)255);
    const hipError_t ed = launch_spectral_split(G, B, nP, r, false, X0, Y, X1, scratch, nullptr, nullptr, st);
    return ed != hipSuccess ? ed : launch_direct_energy(G, Y, B, n, nP, r, scratch, ok, c, st);
  }
  hipError_t e0;
  if (P <= 0 || P % NB != 0 || P > n || P > 4096 || nP % NB != 0) return hipErrorInvalidValue;
  {
    static PerDeviceInt raised;
    if ((e0 = ensure_dynamic_lds(raised, (const void*)chol_kernel, kCholLds)) != hipSuccess) return e0;
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
  IterPlan* plan = (IterPlan*)((char*)scratch + split_scratch_bytes(B, P));                  // [B]
  int* states = (int*)(plan + B);                                                           // [kStates][ST_FIELDS][B]
  int* left = states + (size_t)kStates * ST_FIELDS * B;                                     // [B] nothing left to do in this pass
  int* failed = left + B;                                                                   // [B] failed the check of the first pass
  CholFlags* flags = (CholFlags*)(failed + B);                                              // [kOrths][B]
  double* diag = (double*)(((uintptr_t)(flags + (size_t)kOrths * B) + 255) & ~(uintptr_t)255);   // [B][P] diagonal of the factor
  double* pivots = diag + (size_t)B * P;                                                    // [B][P / 64] smallest scaled pivots
  double* X1 = (double*)(((uintptr_t)(pivots + (size_t)B * (P / NB)) + 255) & ~(uintptr_t)255);  // an iterate of the split, then
  double* U = X1;                                                                           // [B][P][nP] Pi Q^T,
  double* cpart = U + (size_t)B * P * nP;                                                   // [B][P / 32][nP] partial energies
  double* rnorm = cpart + (size_t)B * (P / kSymTile) * nP;                                  // [B][P][nP / 32] of the residual's row lengths
  hipError_t e;

  const long other = (long)B * P * nP;       // from buffer 0 of the blocks to buffer 1
  auto state = [&](int k) { return states + (size_t)k * ST_FIELDS * B; };
  // out = X Gop (P x nP) with X in the buffer that state k names (flip: in the other one), out in the other
  auto gemm_yt_g = [&](int k, int flip, GemmArgs& g) {
    g.B = G; g.M = P; g.N = nP; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = nP;
    g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)nP * nP; g.strideC = (long)P * nP;
    g.epilogue = EPI_STORE_F64;
    g.A = flip ? Zt : Yt; g.C = flip ? Yt : Zt;
    g.sel = state(k) + ST_SEL * B; g.selA = flip ? -other : other; g.selC = -g.selA;
    return launch_gemm64_nt(g, true, true, st);
  };
  // X <- L^-1 X with X X^T = L L^T for the images that state k lets take part, and the plan of what follows
  auto cholqr = [&](int k, int slots, bool first, int pass, bool closing) -> hipError_t {
    const int rest_max = slots == 0 ? 1 : 0;
    GemmArgs g;
    g.A = Yt; g.B = Yt; g.C = S; g.M = P; g.N = P; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = P;
    g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)P * nP; g.strideC = (long)P * P;
    g.epilogue = EPI_STORE_F64;
    g.frag = true;
    g.sel = state(k) + ST_END * B; g.selA = g.selB = other;
    g.skip = state(k) + ST_REST * B; g.skip_if = rest_max;
    if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
    PlanArgs q;
    q.in = state(k); q.out = state(k + 1); q.plan = plan; q.left = left; q.B = B; q.r = r; q.slots = slots; q.first = first; q.pass = pass; q.closing = closing;
    const int orth = k < kStates1 ? k : k - kStates1;               // of its pass
    hipLaunchKernelGGL(chol_kernel, dim3((unsigned)(B * (P / NB))), dim3(512), kCholLds, st, S, D, diag, pivots, P, q, flags + (size_t)orth * B,
                       barrier_limit_ticks());
    const dim3 tg((unsigned)(B * (nP / NB)));
    const double *cS = S, *cD = D;
    const int* in = state(k);
    switch (P / NB) {
#define COVSPEC_TRSM(n) \
  case n: hipLaunchKernelGGL(trsm_kernel<n>, tg, dim3(256), 0, st, Yt, other, cS, cD, nP, nP / NB, in, B, rest_max); break;
      COVSPEC_TRSM(2)
      COVSPEC_TRSM(3)
      COVSPEC_TRSM(4)
      COVSPEC_TRSM(5)
      COVSPEC_TRSM(6)
#undef COVSPEC_TRSM
      default: hipLaunchKernelGGL(trsm_any_kernel, tg, dim3(256), 0, st, Yt, other, cS, cD, P, nP, nP / NB, in, B, rest_max);
    }
    return hipGetLastError();
  };
  // products of the block behind state k
  auto block = [&](int k, int slots) -> hipError_t {
    for (int i = 0; i < slots; ++i) {
      GemmArgs g;
      g.cheb = &plan->tb; g.cheb_stride = sizeof(IterPlan) / sizeof(double); g.cheb_step = i;
      g.skip = state(k) + ST_IDLE * B; g.skip_if = -(i + 1);
      if ((e = gemm_yt_g(k, i & 1, g)) != hipSuccess) return e;
    }
    return hipSuccess;
  };
  // the last orthonormalisation of a pass, the split, the residual check and the energies
  auto finish = [&](int k, int pass_no) -> hipError_t {
    if ((e = cholqr(k, 0, false, pass_no, false)) != hipSuccess) return e;
    const int* sel = state(k + 1) + ST_SEL * B;      // Q^T is there (orthonormal rows), Q^T G goes into the other buffer
    if ((e = block(k + 1, 1)) != hipSuccess) return e;
    {                                                // H = (Q^T G) Q
      GemmArgs g;
      g.A = Zt; g.B = Yt; g.C = H; g.M = P; g.N = P; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = P;
      g.batch = B; g.strideA = (long)P * nP; g.strideB = (long)P * nP; g.strideC = (long)P * P;
      g.sel = sel; g.selA = -other; g.selB = other;
      g.epilogue = EPI_STORE_F64;
      g.lower_only = true;      // H is symmetric: the tiles below the diagonal are mirrored
      g.mirror = true;
      g.skip = left; g.skip_if = 0;
      if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
    }
    if ((e = launch_spectral_split(H, B, P, r, true, S, Pi, X1, scratch, left, pass_no == 1 ? nullptr : failed, st)) != hipSuccess) return e;
    // U = Pi Q^T, and the energies (U Q^T G)_ii
    {
      GemmArgs g;
      g.A = Pi; g.B = Yt; g.C = U; g.D = Zt; g.dots = cpart; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * nP;
      g.sel = sel; g.selB = other; g.selD = -other;
      g.skip = left; g.skip_if = 0;
      if ((e = launch_gemm64_store_dot(g, st)) != hipSuccess) return e;
    }
    // row lengths of the residual Pi Q^T G - H U
    {
      GemmArgs g;
      g.A = Pi; g.B = Zt; g.A2 = H; g.B2 = U; g.C = rnorm; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP / kSymTile;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * (nP / kSymTile);
      g.sel = sel; g.selB = -other;
      g.skip = left; g.skip_if = 0;
      if ((e = launch_gemm64_rownorm_dual(g, st)) != hipSuccess) return e;
    }
    return launch_split_finish(H, Pi, rnorm, nP / kSymTile, cpart, P / kSymTile, B, P, n, nP, r, kRitzTol, scratch, left, ok, pass_no, c, st);
  };
  const dim3 ig((unsigned)((B + 3) / 4));          // 130 words of flags per image and factorisation

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
  hipLaunchKernelGGL(begin_pass_kernel, ig, dim3(256), 0, st, state(0), (const int*)nullptr, (const int*)ok, plan, left, failed, B, flags, kOrths);
  for (int k = 0; k < kBlocks; ++k) {
    if ((e = cholqr(k, kSlots[k], k == 0, 1, k == kBlocks - 1)) != hipSuccess) return e;
    if ((e = block(k + 1, kSlots[k])) != hipSuccess) return e;
  }
  if ((e = finish(kBlocks, 1)) != hipSuccess) return e;
  // images whose subspace is not there yet (slower decay of the spectrum than the blocks of the first pass allow for) take
  // one or two more; for the others every kernel of this pass returns at once
  hipLaunchKernelGGL(begin_pass_kernel, ig, dim3(256), 0, st, state(kStates1), (const int*)state(kStates1 - 1), (const int*)ok, plan, left, failed, B,
                     flags, kBlocks2 + 1);
  for (int k = 0; k < kBlocks2; ++k) {
    if ((e = cholqr(kStates1 + k, kSlots2[k], false, 2, k == kBlocks2 - 1)) != hipSuccess) return e;
    if ((e = block(kStates1 + k + 1, kSlots2[k])) != hipSuccess) return e;
  }
  return finish(kStates1 + kBlocks2, 2);
}

}  // namespace covspec
