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
#include <stddef.h>
#include <initializer_list>
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
constexpr double kPivotFloor = 1e-14;  // see chol_row
constexpr double kLn10 = 2.302585092994046;
constexpr float kSteep = 9.0f;         // ln(lambda_1 / lambda_P) from which growth and not launches limit a block of three products

constexpr size_t kCholLds = (size_t)2 * NB * NBP * sizeof(double);
constexpr int kMaxBlocks = 64;         // block rows: P <= 4096

// ---- The schedule of an image.  Orthonormalisations are numbered; before orthonormalisation k the kernels read state k of the
// image, the factorisation writes state k + 1, the products behind it read that.  Five integers per image and state:
//   ST_REST  0: takes part in the next orthonormalisation, 1: in the last one of the pass only, 2: in none of this pass
//   ST_IDLE  minus the number of products of the block that follows
//   ST_SEL, ST_END  the buffer its first operand is in, and the one its result is in (products alternate between the two)
//   ST_TURN  factorisations so far: its lowest bit says which of two buffers their inverted diagonal blocks go to
enum { ST_REST, ST_IDLE, ST_SEL, ST_END, ST_TURN, ST_FIELDS };
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
  const int at = q.in[ST_END * q.B + b];          // the substitution works in place
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
  out[ST_TURN * q.B] = q.in[ST_TURN * q.B + b] + 1;
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
  out[ST_TURN * q.B] = q.in[ST_TURN * q.B + b];
}

__device__ __forceinline__ void frag_store_through(double* tile, int lane, const f64x4_t& v) {
  double* t = tile + 2 * lane;
  store_through(t, v[0]);
  store_through(t + 1, v[1]);
  store_through(t + 128, v[2]);
  store_through(t + 129, v[3]);
}
__device__ __forceinline__ f64x4_t present(const f64x4_t& v) {
  return (f64x4_t){covspec::present(v[0]), covspec::present(v[1]), covspec::present(v[2]), covspec::present(v[3])};
}

// Factors a 64 x 64 block (a = L L^T) and inverts the factor, by all eight waves.  Wave 0 brings tile (0, 0) in registers, element
// (k, i) in lane (q = k % 4, i), register k / 4; the other tiles on and below the diagonal are in LDS (`a`, pitch NBP), a barrier before
// they are read.  inv(L) goes through the L2 to Db (its tiles on and below the diagonal, in fragment order), the diagonal of L to
// dl (valid in wave 0).  The pivot of row k is floored at floors[k].
// By 16 x 16 tiles.  A diagonal tile stays in the registers of wave 0 from the product that forms it to its inverse, four pivots at a
// time: the 4 x 4 block at the pivots is read into scalars and factored and inverted by every lane for itself (eliminate_panel), what it
// does to the other rows is a product of rank 4, one MFMA on the tile and one on the unit matrix that becomes the inverse.  The operand
// layouts meet: rows 4t .. 4t + 3 of the tile are its register t, which is the B operand of the product with the inverted 4 x 4 block,
// whose first result register is an operand of the update, and L_ts^T as the MFMA leaves it is both operands of A_tt - L_ts L_ts^T.
// The tiles below, the rest of the block and the inverse off its diagonal, inv_ts = -inv_tt sum L_tu inv_us, are the other waves', a wave
// per tile, while wave 0 is at the next diagonal tile; of the last row of the inverse only the products with inv_33 are left at the end.
// Bound by the chain of 64 pivots, a reciprocal and some five dependent operations each.  (One pivot at a time, the multipliers moved
// along the rows of 16 lanes, took 32 moves and 32 multiply-adds a pivot, all four rows the same: 11.4 us a block, bound by issue.)

// Pivots 4t .. 4t + 3 of the tile x (lane (q, i): rows 4v + q of column i) with the unit matrix u; floors of the tile's 16 pivots in LDS.
// piv: lane (q, i) gets the pivot of row 4t + q.
template <int t>
__device__ __forceinline__ void eliminate_panel(f64x4_t& x, f64x4_t& u, const double* floors, double& piv) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  auto at = [&](int i, int j) { return lane_value(x[t], 16 * i + 4 * t + j); };
  const double a00 = at(0, 0), a10 = at(1, 0), a20 = at(2, 0), a30 = at(3, 0);
  const double a11 = at(1, 1), a21 = at(2, 1), a31 = at(3, 1), a22 = at(2, 2), a32 = at(3, 2), a33 = at(3, 3);
  // L D L^T of the 4 x 4 block.  From one pivot to the next the chain is the reciprocal and one multiply-add.
  const double p0 = fmax(a00, floors[4 * t]), r0 = reciprocal(p0);
  const double b11 = fma(-(a10 * a10), r0, a11), b21 = fma(-(a20 * a10), r0, a21), b31 = fma(-(a30 * a10), r0, a31);
  const double b22 = fma(-(a20 * a20), r0, a22), b32 = fma(-(a30 * a20), r0, a32), b33 = fma(-(a30 * a30), r0, a33);
  const double p1 = fmax(b11, floors[4 * t + 1]), r1 = reciprocal(p1);
  const double c22 = fma(-(b21 * b21), r1, b22), c32 = fma(-(b31 * b21), r1, b32), c33 = fma(-(b31 * b31), r1, b33);
  const double p2 = fmax(c22, floors[4 * t + 2]), r2 = reciprocal(p2);
  const double p3 = fmax(fma(-(c32 * c32), r2, c33), floors[4 * t + 3]), r3 = reciprocal(p3);
  const double l10 = a10 * r0, l20 = a20 * r0, l30 = a30 * r0, l21 = b21 * r1, l31 = b31 * r1, l32 = c32 * r2;
  // the inverse of its unit-diagonal factor, as the A operand of a product that leaves its rows in the first register
  const double n20 = fma(l21, l10, -l20), n31 = fma(l32, l21, -l31), n30 = -fma(l31, -l10, fma(l32, n20, l30));
  double n = i16 == kq ? 1.0 : 0.0;                                  // (kq < 4)
  if (i16 == 1 && kq == 0) n = -l10;
  if (i16 == 2 && kq == 0) n = n20;
  if (i16 == 2 && kq == 1) n = -l21;
  if (i16 == 3 && kq == 0) n = n30;
  if (i16 == 3 && kq == 1) n = n31;
  if (i16 == 3 && kq == 2) n = -l32;
  const f64x4_t zero = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  const double w = __builtin_amdgcn_mfma_f64_16x16x4f64(n, x[t], zero, 0, 0, 0)[0];
  const double r = kq == 0 ? r0 : kq == 1 ? r1 : kq == 2 ? r2 : r3;
  piv = kq == 0 ? p0 : kq == 1 ? p1 : kq == 2 ? p2 : p3;
  const double below = (i16 > 4 * t + 3 ? -r : 0.0) * w;             // rows above stay: the unit matrix has results there
  if (t < 3) x = __builtin_amdgcn_mfma_f64_16x16x4f64(below, w, x, 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);                                 // the products with the unit matrix are not part of the chain
  const double uw = __builtin_amdgcn_mfma_f64_16x16x4f64(n, u[t], zero, 0, 0, 0)[0];
  u[t] = uw;
  if (t < 3) u = __builtin_amdgcn_mfma_f64_16x16x4f64(below, uw, u, 0, 0, 0);
}

// Wave 0: x <- the inverse of the factor of the tile (its pivots' floors given), piv <- the pivots
__device__ __forceinline__ void eliminate_tile(f64x4_t& x, double (&piv)[4], const double* floors) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  f64x4_t u;
#pragma unroll
  for (int v = 0; v < 4; ++v) u[v] = i16 == 4 * v + kq ? 1.0 : 0.0;
  eliminate_panel<0>(x, u, floors, piv[0]);
  eliminate_panel<1>(x, u, floors, piv[1]);
  eliminate_panel<2>(x, u, floors, piv[2]);
  eliminate_panel<3>(x, u, floors, piv[3]);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    double rs = __builtin_amdgcn_rsq(piv[v]);
    rs = rs * fma(-0.5 * piv[v], rs * rs, 1.5);
    rs = rs * fma(-0.5 * piv[v], rs * rs, 1.5);
    x[v] = i16 <= 4 * v + kq ? u[v] * rs : 0.0;
    piv[v] *= rs;
  }
}

// `a` and `inv` of a lane: [0] is its element of an operand by rows (row i, column q of a tile), [1] of one by columns (row q, column i,
// which is also what a product leaves).
struct LaneTiles {
  double *a[2], *inv[2];
  __device__ __forceinline__ LaneTiles(double* a_, double* inv_) {
    const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
    int by_row = i16 * NBP + kq, by_col = kq * NBP + i16;
    asm volatile("" : "+v"(by_row), "+v"(by_col));       // or a register for each tile's address is kept across the loop, and spills
    a[0] = a_ + by_row; a[1] = a_ + by_col;
    inv[0] = inv_ + by_row; inv[1] = inv_ + by_col;
  }
};
__device__ __forceinline__ int tile_off(int t, int s) { return 16 * (t * NBP + s); }

// L_ts^T = inv(L_ss) A_ts^T, one wave: lane (q, i) gets the elements (i, 4v + q) of L_ts
__device__ __forceinline__ f64x4_t solve_tile(const LaneTiles& p, int t, int s) {
  f64x4_t o = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  const double *d = p.inv[0] + tile_off(s, s), *x = p.a[0] + tile_off(t, s);
#pragma unroll
  for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(d[4 * j], x[4 * j], o, 0, 0, 0);
  return o;
}

// A_rc -= L_rs L_cs^T, one wave
__device__ __forceinline__ void update_tile(const LaneTiles& p, int r, int c, int s) {
  const double *x = p.a[0] + tile_off(r, s), *y = p.a[0] + tile_off(c, s);
  double* z = p.a[1] + tile_off(r, c);
  f64x4_t o;
#pragma unroll
  for (int v = 0; v < 4; ++v) o[v] = z[4 * v * NBP];
#pragma unroll
  for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(-x[4 * j], y[4 * j], o, 0, 0, 0);
#pragma unroll
  for (int v = 0; v < 4; ++v) z[4 * v * NBP] = o[v];
}

// sum over u from s to t - 1 of L_tu inv_us, one wave
__device__ __forceinline__ f64x4_t invert_sum(const LaneTiles& p, int t, int s) {
  f64x4_t sum = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int u = s; u < t; ++u) {
    const double *x = p.a[0] + tile_off(t, u), *y = p.inv[1] + tile_off(u, s);
#pragma unroll
    for (int j = 0; j < 4; ++j) sum = __builtin_amdgcn_mfma_f64_16x16x4f64(x[4 * j], y[4 * j * NBP], sum, 0, 0, 0);
  }
  return sum;
}

// a tile of the inverse from LDS to memory
__device__ __forceinline__ void hand_on(const LaneTiles& p, double* Db, int t, int s) {
  const double* d = p.inv[0] + tile_off(t, s);
  frag_store_through(Db + (4 * t + s) * kFragTile, threadIdx.x & 63, present((f64x4_t){d[0], d[4], d[8], d[12]}));
}

// between: called by all waves with their own stores of before acknowledged, one thread of wave 7 raising a flag for it
template <typename Between>
__device__ __forceinline__ void factor_invert(f64x4_t x, double* a, double* inv, double* Db, double* dl, const double* floors, Between between) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i16 = lane & 15, kq = lane >> 4;
  const int col = 7 - w;                             // waves 7, 6 and 5 have a column of the inverse each
  f64x4_t sum = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    const LaneTiles p(a, inv);
    if (w == 0) {
      double root[4];
      eliminate_tile(x, root, floors + 16 * s);
      if (i16 == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) dl[16 * s + 4 * v + kq] = root[v];
      }
    } else if (s > 0) {
      // what step s - 1 left: the tiles beyond (s, s), and row s - 1 of the inverse
      const int e = w < 3 ? 1 : 2, f = w - e * (e + 1) / 2;
      if (w < 6 && s + e < 4) update_tile(p, s + e, s + f, s - 1);
      if (col < s - 1) {
        const f64x4_t t = invert_sum(p, s - 1, col);
        const double* d = p.inv[0] + tile_off(s - 1, s - 1);
        double* z = p.inv[1] + tile_off(s - 1, col);
        f64x4_t o = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(-d[4 * j], t[j], o, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) z[4 * v * NBP] = o[v];
      }
      if (s == 3) {
        if (w < 4) hand_on(p, Db, w - 1, w - 1);
        else if (w == 4) hand_on(p, Db, 1, 0);
        else {
          if (col < 2) hand_on(p, Db, 2, col);
          sum = invert_sum(p, 3, col);
        }
      }
    }
    if (s == 0) between();                           // `inv` has been read, the tiles of `a` are there
    if (w == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) p.inv[1][tile_off(s, s) + 4 * v * NBP] = x[v];
    }
    __syncthreads();
    if (s < 3) {
      const int t = s + 1 + w;
      if (t < 4) {
        const f64x4_t l = solve_tile(p, t, s);
        if (w == 0) {                              // A_tt - L_ts L_ts^T: l^T is both operands
#pragma unroll
          for (int v = 0; v < 4; ++v) {            // from its lower triangle
            const int k = 4 * v + kq, hi = k > i16 ? k : i16, lo = k > i16 ? i16 : k;
            x[v] = a[tile_off(t, t) + hi * NBP + lo];
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) x = __builtin_amdgcn_mfma_f64_16x16x4f64(-l[v], l[v], x, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) p.a[0][tile_off(t, s) + 4 * v] = l[v];
      }
      __syncthreads();
    }
  }
  const LaneTiles p(a, inv);
  if (w == 0) {
    hand_on(p, Db, 3, 3);
  } else if (w > 4) {                                // -inv_33 sum, transposed: in fragment order
    const double* d = p.inv[0] + tile_off(3, 3);
    f64x4_t o = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 4; ++j) o = __builtin_amdgcn_mfma_f64_16x16x4f64(sum[j], -d[4 * j], o, 0, 0, 0);
    frag_store_through(Db + (12 + col) * kFragTile, lane, present(o));
  }
}

// Progress of the factorisation of one image: written by the workgroup of a block row, polled by those of the rows after it.
// Cleared at the start of a pass.
struct CholFlags {
  unsigned int ticket;          // next block row to hand to a starting workgroup
  int failed;                   // a workgroup gave up waiting
  int cols[kMaxBlocks];         // per block row: 1 when its part of L is in memory
  int done[kMaxBlocks];         // its diagonal and smallest pivot are in memory, and everything else of it
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

// Block row `row` of the Cholesky factorisation S[b] = L L^T (P x P, P % 64 == 0, [P/16][P/16] tiles in fragment order, those on and below
// the diagonal), one 512-thread workgroup per block row of 64 and image.  The workgroup of block row i:
//   for K < i:  T = S[i,K] - sum over K' < K of L[i,K'] L[K,K']^T;   L[i,K] = T inv(L_KK)^T, in place;   D += L[i,K] L[i,K]^T
//   factors and inverts S[i,i] - D (factor_invert); the inverse goes to Dinv[b][i] (its tiles).
// It waits for row K's columns before the sum and for row K's inverse (its elements are there when they are not kAbsent) before the product with it, so
// that the sum runs while row K is being factored; rows are taken in order (a ticket per image), so that a workgroup only waits for rows that have started
// before it, whatever else the device is doing; every wait is bounded.  What the rows hand one another is stored through the L2.
// Every product is formed transposed, so that its result is the fragment of the tile it goes to.
// The inverses of even and odd turns have a buffer each (orth_kernel clears the other one).
// On return the strictly-lower blocks of S hold L; its diagonal blocks are represented by their inverses.
// A pivot is floored relative to its own row's squared length (rows may differ in length by any number of digits: after a block of
// products they do, by the growth of the first row over the last), at the rounding of S: what is left of a row below that is noise, which
// the floor keeps shorter than the other rows, and the next factorisation makes a row of length one of it.  (At 1e-28 such a row came out
// up to 1e7 long, with as much of the other rows in it, and the image ended in the full solve.)
// Bound by the chain of diagonal blocks: factor (8.8 us), flag, product with the inverse, D.  One workgroup per image, which did the
// trailing updates itself beside the factorisation of the next block by one of its waves, took, us: one image of order 192 67,
// eight of 384 172; by block rows with one pivot at a time 53 and 109; four at a time, the flag of a row's columns raised beside its
// first diagonal tile and the inverse handed on as it comes 41 and 87.
// lds: 2 * 64 * 65 doubles.
__device__ __forceinline__ void chol_row(double* lds, int* s_flag, double* S, double* __restrict__ Dinv, double* __restrict__ diag, double* __restrict__ pivots,
                                         int P, int b, int row, const PlanArgs& q, CholFlags* f, long long limit_ticks) {
  double* a = lds;                  // [64][65] diagonal block, see factor_invert
  double* inv = lds + NB * NBP;     // [64][65] the inverse of its factor; before: T, then L[i,K]
  __shared__ double dl[NB], diag0[NB], floors[NB];
  __shared__ int s_gave_up;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), i16 = lane & 15, kq = lane >> 4;
  const int nblk = P / NB, per16 = P / 16;
  const int turn = q.in[ST_TURN * q.B + b] & 1;
  if (tid == 0) s_gave_up = 0;                      // (a barrier before it is set)
  double* Sb = S + (long)b * P * P;
  double* Db = Dinv + ((long)turn * q.B + b) * nblk * NB * NB;
  auto tile = [&](int rt, int ct) -> double* { return Sb + ((long)rt * per16 + ct) * kFragTile; };
  if (tid < NB) {
    diag0[tid] = tile(4 * row + (tid >> 4), 4 * row + (tid >> 4))[frag_at(tid & 15, tid & 15)];
    floors[tid] = fma(kPivotFloor, diag0[tid], 1e-300);
  }
  // t-th tile of a block on or below its diagonal; wave w has the tiles w and, w = 2, 3, w + 6 (wave 0, and wave 4 beside it on its
  // SIMD, one each: the factorisation begins with tile 0)
  auto low = [](int t, int& x, int& y) { x = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3; y = t - x * (x + 1) / 2; };
  auto own = [&](int e) { return e == 0 ? w : w == 2 || w == 3 ? w + 6 : 10; };
  f64x4_t dacc[2], own_tile[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    dacc[e] = own_tile[e] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    if (own(e) < 10) {
      int x, y;
      low(own(e), x, y);
      own_tile[e] = frag_load(tile(4 * row + x, 4 * row + y), lane);
    }
  }
  const __amdgpu_buffer_rsrc_t inverses = __builtin_amdgcn_make_buffer_rsrc((void*)Db, (short)0, nblk * NB * NB * 8, 0x00020000);
  const int rx = w >> 1;                                        // row tile of this wave, column tiles 2 (w & 1) + 0, 1 of the sum
  bool alive = true;
  for (int K = 0; K < row; ++K) {
    f64x4_t t[2];
    const int c0 = 2 * (w & 1);
#pragma unroll
    for (int y = 0; y < 2; ++y) t[y] = frag_load(tile(4 * row + rx, 4 * K + c0 + y), lane);
    if (K > 0) {
      if (!(alive = wait_flag(&f->cols[K], 1, f, s_flag, limit_ticks))) break;
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
    __syncthreads();
    // L[i,K]: this wave's column tiles are 0 and 3, or 1 and 2 (five products each)
    f64x4_t in[4], out[2];
    f64x2_t d[5][2];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) in[c][v] = inv[(16 * rx + i16) * NBP + 16 * c + 4 * v + kq];
    const int odd = w & 1, y0 = odd, y1 = 3 - odd;
    {
      int at[5];
#pragma unroll
      for (int n = 0; n < 5; ++n) {                             // tiles (y0, 0 .. y0), then (y1, 0 .. y1)
        const int t = n <= y0 ? 4 * y0 + n : 4 * y1 + n - y0 - 1;
        at[n] = (K * 16 + t) * (kFragTile * 8) + 16 * lane;
      }
      if (!fetch_present<5>(inverses, at, d, &f->failed, limit_ticks) && lane == 0) s_gave_up = 1;
    }
    out[0] = out[1] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    if (odd) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          out[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[2 + c][v >> 1][v & 1], in[c][v], out[1], 0, 0, 0);
          if (c < 2) out[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[c][v >> 1][v & 1], in[c][v], out[0], 0, 0, 0);
        }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          out[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[1 + c][v >> 1][v & 1], in[c][v], out[1], 0, 0, 0);
          if (c < 1) out[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[c][v >> 1][v & 1], in[c][v], out[0], 0, 0, 0);
        }
    }
    __syncthreads();                                            // T has been read
    if (s_gave_up) { alive = false; break; }
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
      const int tt = own(e);
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
    // the next round writes to LDS behind its first wait
  }
  if (alive) {
    double* Di = Db + (long)row * NB * NB;
    f64x4_t x0 = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int tt = own(e);
      if (tt < 10) {
        int x, y;
        low(tt, x, y);
        const f64x4_t c = own_tile[e] - dacc[e];
        if (tt == 0) {
          x0 = c;
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) a[(16 * x + i16) * NBP + 16 * y + 4 * v + kq] = c[v];
        }
      }
    }
    factor_invert(x0, a, inv, Di, dl, floors, [&]() {
      __builtin_amdgcn_s_waitcnt(0x0070);          // vmcnt(0) lgkmcnt(0): L[row, .] has been stored
      __syncthreads();
      if (tid == 7 * kWave) __hip_atomic_store(&f->cols[row], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
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
  for (int k = 0; alive && k < row; ++k) {
    const long long t0 = wall_clock64();
    while (alive && __hip_atomic_load(&f->done[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) alive = wall_clock64() - t0 <= limit_ticks;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (alive) {
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

// 16 columns of Y <- L^-1 Y (P x nP, pitch nP, in place), one wave, by blocked forward substitution with the factor chol_row leaves in S
// (strictly-lower blocks) and Dinv (inverted diagonal blocks), both tiles in fragment order.  Columns are independent: no wave reads what
// another wrote.  L, D, Y: of the image, lane offsets included.  All waves of the workgroup call it (mine: this one has columns).
//   for block row bi:  T = Y[bi] - sum_{K<bi} L[bi,K] Y[K];   Y[bi] = inv(L_bibi) T
// The workgroups of an image's columns are in the launch of its factorisation and follow it block row by block row: the sum as soon as row
// bi of L is there, the product with the inverted block when that is, so that behind the last flag only that product is left.
// What the MFMA returns (lane = column, register = k) is exactly the layout its B operand wants; solved blocks are read back by the lane
// that wrote them, two groups of 16 k ahead, as are those of L.
// As a launch behind the factorisation, the solved blocks in registers, it took, us: 192 x 320 14.5, 192 x 1664 batch 4 19, 384 x 1152
// batch 8 44, 256 x 640 batch 64 73; the factorisation by itself 40, 43, 87 and 71, both in one launch 45, 49, 95 and 126.
__device__ __forceinline__ bool substitute(const double* L, const double* D, double* Y, long nP, int P, bool mine, CholFlags* f, int* s_flag,
                                           long long limit_ticks) {
  const __amdgpu_buffer_rsrc_t inverses = __builtin_amdgcn_make_buffer_rsrc((void*)D, (short)0, P / NB * NB * NB * 8, 0x00020000);
  bool alive = true;
  const int nblk = P / NB;
  const long row_tiles = (long)(P / 16) * kFragTile;
#pragma unroll 1
  for (int bi = 0; bi < nblk; ++bi) {
    f64x4_t acc[4], rhs[4];
    double* Yb = Y + (long)bi * NB * nP;
    const f64x4_t zero = (f64x4_t){0.0, 0.0, 0.0, 0.0};
    if (mine) {
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) rhs[x][v] = Yb[(long)(16 * x + 4 * v) * nP];
    }
    if (bi > 0 && !wait_flag(&f->cols[bi], 1, f, s_flag, limit_ticks)) return false;
    if (bi > 0 && mine) {
      constexpr int kAhead = 2;
      const double* Lb = L + 4 * bi * row_tiles;
      f64x4_t fa[kAhead][4], fb[kAhead];
      auto fetch = [&](int g, int slot) {
#pragma unroll
        for (int x = 0; x < 4; ++x) fa[slot][x] = frag_load(Lb + x * row_tiles + g * kFragTile, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) fb[slot][v] = Y[(long)(16 * g + 4 * v) * nP];
      };
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] = zero;
#pragma unroll
      for (int g = 0; g < kAhead; ++g) fetch(g, g);
#pragma unroll 1
      for (int g = 0; g < 4 * bi; g += kAhead) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[h][x][v], fb[h][v], acc[x], 0, 0, 0);
          if (g + kAhead < 4 * bi) fetch(g + kAhead + h, h);
          __builtin_amdgcn_sched_barrier(0);            // the loads stay that far ahead of their use
        }
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) rhs[x] = rhs[x] - acc[x];
    }
    if (mine) {
      f64x2_t fd[10][2];                                // the inverted block is lower triangular
      int at[10];
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int q = 0; q <= x; ++q) at[x * (x + 1) / 2 + q] = (bi * 16 + 4 * x + q) * (kFragTile * 8) + 16 * (threadIdx.x & 63);
      alive = fetch_present<10>(inverses, at, fd, &f->failed, limit_ticks) && alive;
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] = zero;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int x = q; x < 4; ++x) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(fd[x * (x + 1) / 2 + q][v >> 1][v & 1], rhs[q][v], acc[x], 0, 0, 0);
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) Yb[(long)(16 * x + 4 * v) * nP] = acc[x][v];
    }
  }
  return alive;
}

// The factorisation of all images and the substitution behind it.  Per image the first P / 64 workgroups to start have a block row
// each, the others 16 columns per wave of their first `waves` (four: a SIMD each, while there are compute units for that).  A workgroup
// only waits for some that have started before it, in whatever order the device starts them.  Dynamic LDS: 2 * 64 * 65 doubles.
__global__ __launch_bounds__(512) void orth_kernel(double* S, double* __restrict__ Dinv, double* __restrict__ diag, double* __restrict__ pivots, int P,
                                                   PlanArgs q, CholFlags* flags, long long limit_ticks, double* Yt, long other, int nP, int waves) {
  extern __shared__ double lds[];
  __shared__ int s_flag;
  const int b = blockIdx.x % q.B, tid = threadIdx.x;
  if (q.in[ST_REST * q.B + b] > (q.slots == 0 ? 1 : 0)) {      // no part in this orthonormalisation
    if (tid == 0 && blockIdx.x < (unsigned)q.B) rest_on(q, b);
    return;
  }
  CholFlags* f = flags + b;
  if (tid == 0) s_flag = (int)atomicAdd(&f->ticket, 1u);
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(s_flag);
  __syncthreads();                                   // s_flag is reused by the waits
  const int nblk = P / NB;
  if (ticket < nblk) {
    chol_row(lds, &s_flag, S, Dinv, diag, pivots, P, b, ticket, q, f, limit_ticks);
    return;
  }
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), col = ((ticket - nblk) * waves + w) * 16;
  const bool mine = w < waves && col < nP;           // nP % 64 == 0
  const int turn = q.in[ST_TURN * q.B + b] & 1;
  // the inverses of the turn before make room for those of the next one, while the first of this one is on its way
  const int parts = gridDim.x / q.B - nblk;
  for (int k = ticket - nblk; k < nblk; k += parts) {
    double* block = Dinv + (((long)(turn ^ 1) * q.B + b) * nblk + k) * (NB * NB);
    for (int e = tid; e < NB * NB; e += 512)
      if (e >> 10 >= (e >> 8 & 3)) store_through(block + e, absent());      // tiles on and below the diagonal
  }
  double* Y = Yt + (q.in[ST_END * q.B + b] ? other : 0) + (long)b * P * nP + (long)(lane >> 4) * nP + (mine ? col : 0) + (lane & 15);
  // gave up: the image's rows are not orthonormal, which the check of the residual refuses
  if (!substitute(S + (long)b * P * P + 2 * lane, Dinv + ((long)turn * q.B + b) * nblk * NB * NB, Y, nP, P, mine, f, &s_flag, limit_ticks) && lane == 0)
    __hip_atomic_store(&f->failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// See launch_lowrank_prepare.  One thread per element of the start block Omega, a fixed pattern of +-1, and of the padding; the words with
// them.  (These were five launches of 2 to 4 us each.  Clearing all of the matrices in front of the products that fill them took 16 us for four of
// 1664 and 13 for four of 1280.)
struct PrepareArgs {
  int *status, *ctl, *flags, *state, *left, *failed;
  IterPlan* plan;
  double *A, *om, *inverses;
  int* cut;
  long words, flag_words, cut_words, pad, omega, blocks;      // numbers of elements; pad: of one matrix
  int B, n, nP;
};
__global__ __launch_bounds__(256) void prepare_kernel(PrepareArgs q) {
  const long at = (long)blockIdx.x * 256 + threadIdx.x, step = (long)gridDim.x * 256;
  for (long i = at; i < q.omega; i += step) {
    const int r = (int)(i / q.nP), c = (int)(i - (long)r * q.nP);
    uint32_t h = (uint32_t)r * 0x9E3779B1u ^ ((uint32_t)c + 0x7F4A7C15u) * 0x85EBCA77u;
    h ^= h >> 15; h *= 0x2C1B3C6Du; h ^= h >> 12; h *= 0x297A2D39u; h ^= h >> 15;
    q.om[i] = (c < q.n) ? ((h & 1u) ? 1.0 : -1.0) : 0.0;
  }
  const long right = (long)q.n * (q.nP - q.n);
  const int w = q.nP - q.n;
  for (long i = at; i < q.pad * q.B; i += step) {
    const long b = i / q.pad, e = i - b * q.pad;
    q.A[b * q.nP * q.nP + (e < right ? (e / w) * q.nP + q.n + e % w : (long)q.n * q.nP + (e - right))] = 0.0;
  }
  for (long i = at; i < q.blocks; i += step) q.inverses[i] = absent();
  for (long i = at; i < q.words; i += step) q.ctl[i] = 0;
  for (long i = at; i < q.flag_words; i += step) q.flags[i] = 0;
  for (long i = at; i < q.cut_words; i += step) q.cut[i] = 0;
  for (long b = at; b < q.B; b += step) {
    if (q.status) q.status[b] = 0;
    if (q.state) {                         // every block is in buffer 0
#pragma unroll
      for (int k = 0; k < ST_FIELDS; ++k) q.state[k * q.B + b] = 0;
      q.plan[b].redo = 0;
      q.left[b] = q.failed[b] = 0;
    }
  }
}

// The workspace of a direct split.
struct DirectBuffers {
  double *X0, *Y, *X1;
  void* scratch;
  DirectBuffers(void* ws, int B, int nP) {
    const size_t sq = (size_t)B * nP * nP;
    X0 = (double*)ws;
    Y = X0 + sq;
    X1 = Y + sq;
    scratch = (void*)(((uintptr_t)(X1 + sq) + 255) & ~(uintptr_t)255);
  }
};

// The workspace of the iteration.
struct IterBuffers {
  double *Yt, *Zt, *Om, *S, *H, *D, *Pi;   // D: [2][B][P][64] inverted diagonal blocks; Pi: [B][P][P] the projector
  void* scratch;                           // of the split
  IterPlan* plan;                          // [B]
  int *states, *left, *failed;             // [kStates][ST_FIELDS][B]; [B] nothing left to do in this pass; [B] failed the check of the first pass
  CholFlags* flags;                        // [kOrths][B]
  double *diag, *pivots;                   // [B][P] diagonal of the factor, [B][P / 64] smallest scaled pivots
  double* X1;                              // an iterate of the split, then U [B][P][nP] = Pi Q^T,
  double *cpart, *rnorm;                   // [B][P / 32][nP] partial energies, [B][P][nP / 32] of the residual's row lengths
  IterBuffers(void* ws_, int B, int nP, int P) {
    const size_t blk = (size_t)B * P * nP;
    Yt = (double*)ws_;
    Zt = Yt + blk;
    Om = Zt + blk;
    S = Om + (size_t)P * nP;
    H = S + (size_t)B * P * P;
    D = H + (size_t)B * P * P;
    Pi = D + 2 * (size_t)B * P * NB;
    scratch = (void*)(((uintptr_t)(Pi + (size_t)B * P * P) + 255) & ~(uintptr_t)255);
    plan = (IterPlan*)((char*)scratch + split_scratch_bytes(B, P));
    states = (int*)(plan + B);
    left = states + (size_t)kStates * ST_FIELDS * B;
    failed = left + B;
    flags = (CholFlags*)(failed + B);
    diag = (double*)(((uintptr_t)(flags + (size_t)kOrths * B) + 255) & ~(uintptr_t)255);
    pivots = diag + (size_t)B * P;
    X1 = (double*)(((uintptr_t)(pivots + (size_t)B * (P / NB)) + 255) & ~(uintptr_t)255);
    cpart = X1 + blk;
    rnorm = cpart + (size_t)B * (P / kSymTile) * nP;
  }
};

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
  return 2 * blk + (size_t)P * nP * 8 + 3 * (size_t)B * P * P * 8 + 2 * (size_t)B * P * NB * 8 + split_scratch_bytes(B, P) + 256 +
         (size_t)B * (sizeof(IterPlan) + (kStates * ST_FIELDS + 2) * sizeof(int) + kOrths * sizeof(CholFlags) + (P + P / NB) * 8) + 512 + tail_doubles(B, P, nP) * 8 + 256;
}

// Launches of the probed shape: start block and the products of the first pass (blocks that take fewer leave the rest out).
int subspace_product_launches() {
  int n = 2;
  for (int k = 0; k < kBlocks; ++k) n += kSlots[k];
  return n;
}

hipError_t launch_lowrank_prepare(int* status, void* ctl, size_t words, double* A, int B, int n, int nP, int P, void* ws, hipStream_t st) {
  if (n > nP || B < 1) return hipErrorInvalidValue;
  PrepareArgs q = {};
  q.status = status;
  q.ctl = (int*)ctl;
  q.words = ctl ? (long)words : 0;
  q.A = A;
  q.pad = (long)nP * nP - (long)n * n;
  q.B = B; q.n = n; q.nP = nP;
  if (P > 0) {
    const IterBuffers w(ws, B, nP, P);
    q.om = w.Om;
    q.omega = (long)P * nP;
    q.inverses = w.D;
    q.blocks = 2 * (long)B * P * NB;
    q.plan = w.plan;
    q.state = w.states;
    q.left = w.left;
    q.failed = w.failed;
    q.flags = (int*)w.flags;
    q.flag_words = (long)kOrths * B * (long)(sizeof(CholFlags) / sizeof(int));
  }
  if (ws && (P > 0 || split_direct(nP))) {
    size_t bytes = 0;
    q.cut = (int*)(P > 0 ? split_cleared(IterBuffers(ws, B, nP, P).scratch, B, P, &bytes) : split_cleared(DirectBuffers(ws, B, nP).scratch, B, nP, &bytes));
    q.cut_words = (long)(bytes / sizeof(int));
  }
  long most = q.pad * B;
  for (long k : {q.omega, q.blocks, q.words, q.flag_words, q.cut_words, (long)B}) most = k > most ? k : most;
  const long blocks = (most + 255) / 256;
  hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st, q);
  return hipGetLastError();
}

hipError_t launch_subspace_eigen(const double* G, int B, int n, int nP, int r, int P, void* ws_, int* ok,
                                 float* c, hipEvent_t probe_begin, hipEvent_t probe_end, hipStream_t st) {
  if (P == 0) {
    // the whole matrix is the window
    if (!split_direct(nP)) return hipErrorInvalidValue;
    const DirectBuffers w(ws_, B, nP);
    double *X0 = w.X0, *Y = w.Y, *X1 = w.X1;
    void* scratch = w.scratch;
    const hipError_t ed = launch_spectral_split(G, B, nP, r, false, X0, Y, X1, scratch, nullptr, nullptr, 0, st);
    return ed != hipSuccess ? ed : launch_direct_energy(G, Y, B, n, nP, r, scratch, ok, c, st);
  }
  hipError_t e0;
  if (P <= 0 || P % NB != 0 || P > n || P > 4096 || nP % NB != 0) return hipErrorInvalidValue;
  {
    static PerDeviceInt raised;
    if ((e0 = ensure_dynamic_lds(raised, (const void*)orth_kernel, kCholLds)) != hipSuccess) return e0;
  }
  const IterBuffers w(ws_, B, nP, P);
  double *Yt = w.Yt, *Zt = w.Zt, *S = w.S, *H = w.H, *D = w.D, *Pi = w.Pi, *U = w.X1, *diag = w.diag, *pivots = w.pivots;
  IterPlan* plan = w.plan;
  int *states = w.states, *left = w.left;
  CholFlags* flags = w.flags;
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
    const int nblk = P / NB, n64 = nP / NB;
    const int waves = B * (nblk + n64) <= 256 ? 4 : 8, parts = waves == 4 ? n64 : (n64 + 1) / 2;
    hipLaunchKernelGGL(orth_kernel, dim3((unsigned)(B * (nblk + parts))), dim3(512), kCholLds, st, S, D, diag, pivots, P, q, flags + (size_t)orth * B,
                       barrier_limit_ticks(), Yt, other, nP, waves);
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
    if ((e = launch_spectral_split(H, B, P, r, true, S, Pi, w.X1, w.scratch, left, pass_no == 1 ? nullptr : w.failed, pass_no - 1, st)) != hipSuccess) return e;
    // U = Pi Q^T, and the energies (U Q^T G)_ii
    {
      GemmArgs g;
      g.A = Pi; g.B = Yt; g.C = U; g.D = Zt; g.dots = w.cpart; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * nP;
      g.sel = sel; g.selB = other; g.selD = -other;
      g.skip = left; g.skip_if = 0;
      if ((e = launch_gemm64_store_dot(g, st)) != hipSuccess) return e;
    }
    // row lengths of the residual Pi Q^T G - H U
    {
      GemmArgs g;
      g.A = Pi; g.B = Zt; g.A2 = H; g.B2 = U; g.C = w.rnorm; g.M = P; g.N = nP; g.K = P; g.lda = P; g.ldb = nP; g.ldc = nP / kSymTile;
      g.batch = B; g.strideA = (long)P * P; g.strideB = (long)P * nP; g.strideC = (long)P * (nP / kSymTile);
      g.sel = sel; g.selB = -other;
      g.skip = left; g.skip_if = 0;
      if ((e = launch_gemm64_rownorm_dual(g, st)) != hipSuccess) return e;
    }
    NextPass next = {};
    if (pass_no == 1)
      next = {state(kStates1), left, w.failed, &plan->redo, (int*)flags, state(kStates1 - 1), (int)(sizeof(IterPlan) / sizeof(int)), kBlocks2 + 1,
              kOrths, (int)(sizeof(CholFlags) / sizeof(int)), (int)(offsetof(CholFlags, failed) / sizeof(int))};
    return launch_split_finish(H, Pi, w.rnorm, nP / kSymTile, w.cpart, P / kSymTile, B, P, n, nP, r, kRitzTol, w.scratch, left, ok, pass_no, c, next, st);
  };
  // start block: Omega G
  if (probe_begin && (e = hipEventRecord(probe_begin, st)) != hipSuccess) return e;
  {
    GemmArgs g;
    g.A = w.Om; g.B = G; g.C = Yt; g.M = P; g.N = nP; g.K = nP; g.lda = nP; g.ldb = nP; g.ldc = nP;
    g.batch = B; g.strideA = 0; g.strideB = (long)nP * nP; g.strideC = (long)P * nP;
    g.epilogue = EPI_STORE_F64;
    if ((e = launch_gemm64_nt(g, true, true, st)) != hipSuccess) return e;
  }
  if (probe_end && (e = hipEventRecord(probe_end, st)) != hipSuccess) return e;
  for (int k = 0; k < kBlocks; ++k) {
    if ((e = cholqr(k, kSlots[k], k == 0, 1, k == kBlocks - 1)) != hipSuccess) return e;
    if ((e = block(k + 1, kSlots[k])) != hipSuccess) return e;
  }
  if ((e = finish(kBlocks, 1)) != hipSuccess) return e;
  // images whose subspace is not there yet (slower decay of the spectrum than the blocks of the first pass allow for) take
  // one or two more; for the others every kernel of this pass returns at once
  for (int k = 0; k < kBlocks2; ++k) {
    if ((e = cholqr(kStates1 + k, kSlots2[k], false, 2, k == kBlocks2 - 1)) != hipSuccess) return e;
    if ((e = block(kStates1 + k + 1, kSlots2[k])) != hipSuccess) return e;
  }
  return finish(kStates1 + kBlocks2, 2);
}

}  // namespace covspec
