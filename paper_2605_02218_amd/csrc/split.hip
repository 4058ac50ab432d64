// Spectral split of a symmetric matrix H at its r-th eigenvalue: the orthogonal projector Pi onto the span of the
// r dominant eigenvectors (paper Sec. III-A.3: the energies c_i need the rank-r subspace, not its eigenvectors:
// c_i = (Pi G)_ii).
//
// Pi = (I + sign(H - mu I)) / 2 with mu between the r-th and the (r+1)-th eigenvalue.  Two steps:
//   split_kernel, or cut_kernel for a few images, finds mu.  The rows of H are ordered like its eigenvalues (block iteration, subspace.hip), so the
//     two eigenvalues at the cut are those of a 64 x 64 window of rows around r: what the rows outside couple to it
//     enters an eigenvalue squared (rows p and q couple by (lambda_q / lambda_p)^s after s products; 32 rows apart that shifts
//     the eigenvalue by less than a tenth of the half gap for every decay the iteration converges on; an image that failed
//     the check gets 128 rows).  In split_kernel the window is brought to tridiagonal form by Householder reflections with the
//     matrix in the registers of one workgroup, and the two eigenvalues are cut out of it by Sturm counts, 128 trial
//     points per pass and eigenvalue; cut_kernel counts without it.  A matrix of order <= 128 is its own window, whatever the order of its rows.
//   sign_kernel first lifts the cut: H is positive semidefinite and mu far below its norm, so X <- alpha X - beta X^2 with the
//     largest alpha that keeps X in [0, 1] and its top above the image of mu multiplies mu, and the gap around it, by almost 4
//     per product; it ends with mu in [0.1, 0.4] of the norm.  Then X <- 1.5 s X - 0.5 s^3 X^3 from the shifted X (Newton-Schulz;
//     s is the factor for which the image of [l, 1] has the largest lower end, l the known lower bound on |eigenvalues of X|: a step
//     then multiplies a small l by 2.6, against 1.5 without), two symmetric products per step on the fp64 MFMA, until
//     X no longer changes.
// Before: the P x P problem was diagonalised by block Jacobi (six sweeps of P/32 - 1 rounds of 32 dependent rotation
// steps each).  An eigen-decomposition orders every pair of rows; the energies only ask which side of the cut a
// direction is on, and the products that answer that are matrix-core work without a serial chain of rotations.
// Without the lift (Newton-Schulz from the unlifted cut, mu / norm = 2e-5 to 3e-2) the iteration took 15 to 20 steps, so 10 to 11 and
// 2 to 7 single products: one matrix of order 192 193 -> 160 us, one of 128 127 -> 104.
// Jacobi against split + sign before that, us: one matrix of order 128 2727 -> 124 + 131, one of 192 1482 -> 124 + 197, four of 192
// 1769 -> 124 + 200, eight of 384 3551 -> 124 + 259, sixty-four of 256 3894 -> 124 + 1061.
//
// Leading rows [0, a) of an ordered H that do not couple to the rows around and beyond the cut (kLeadFar) and whose
// eigenvalues are above mu by their diagonal (row sums of the scaled couplings below 1/2: no eigenvalue of the block is
// below half its smallest diagonal entry) are wanted as they are: the iteration then runs on the trailing block only,
// which is smaller and, without the largest eigenvalues, needs fewer steps.  What it leaves out shows in the residual
// check of the caller.
#include "common.h"
#include "host_cache.h"
#include "kernels.h"
#include "pivots.h"

namespace covspec {

namespace {

constexpr int SN = 128;              // order of the largest window
constexpr int kMaxSignSteps = 40;    // 25 take the smallest admitted l to 1 / 2.6, a handful more to 1
constexpr double kMinGap = 1e-10;    // smallest half gap at the cut, relative to the norm, that is iterated on
constexpr double kLiftTo = 0.1;      // the cut is lifted until it is at least this part of the norm
// Couplings |H_pq| / H_rr below which a leading row p is left out of the iteration: to rows beyond the cut (they go into
// the residual as they are, in quadrature over the rows left out) and to the 32 rows before it (they meet the unwanted
// directions only through these directions' tails).
constexpr double kLeadFar = 2e-11, kLeadNear = 1e-6;

struct SplitCtl {
  unsigned long long dev[kMaxSignSteps + 2];   // per step: bits of the largest change of an entry of X
  ImageBarrier bar;
  unsigned int ticket;                         // ctl[0] only: next (image, slot) to hand to a starting workgroup
  int state;                                   // 0: to be iterated, 1: left alone (no usable gap, or not asked for), 2: projector valid, 3: gave up
  double mu, half, theta;                      // cut, half gap at the cut, r-th eigenvalue
};

// Sums over the 16 lanes of a DPP row, the same in all of them; of X0..7 at once, so that the steps of one fill the waits of
// the others.
template <int CTRL>
__device__ __forceinline__ double row_rotated(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
template <int X, int FIRST>
__device__ __forceinline__ void row16_sums(double (&v)[X]) {
#pragma unroll
  for (int x = FIRST; x < X; ++x) v[x] += row_rotated<0x128>(v[x]);
#pragma unroll
  for (int x = FIRST; x < X; ++x) v[x] += row_rotated<0x124>(v[x]);
#pragma unroll
  for (int x = FIRST; x < X; ++x) v[x] += row_rotated<0x122>(v[x]);
#pragma unroll
  for (int x = FIRST; x < X; ++x) v[x] += row_rotated<0x121>(v[x]);
}
__device__ __forceinline__ double row16_sum(double v) {
  v += row_rotated<0x128>(v);
  v += row_rotated<0x124>(v);
  v += row_rotated<0x122>(v);
  return v + row_rotated<0x121>(v);
}

// Per row p of H: off[p] = sum over q != p of |H_pq|, and link[p] = the largest coupling to the rows from r - 32 on as a
// multiple of what kLeadFar / kLeadNear admit; 1 where the |H_pq| / sqrt(H_pp H_qq) of the row sum to more than 1/2 (no
// candidate for being left out of the iteration).  One wave per row, 16 rows p0 .. per workgroup (the diagonal is read once for them).
__device__ __forceinline__ void row_profile(const double* __restrict__ Hb, int P, int r, int p0, double* __restrict__ off, double* __restrict__ link,
                                            double* rd) {   // rd: reciprocal square roots of the diagonal, 0 for rows of length zero
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const double hrr = Hb[(long)(r - 1) * P + r - 1];
  for (int q = threadIdx.x; q < P; q += 256) {
    const double d = Hb[(long)q * P + q];
    rd[q] = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
  }
  __syncthreads();
#pragma unroll 1
  for (int x = 0; x < 4; ++x) {
    const int p = p0 + 4 * x + wv;                   // P % 16 == 0
    const double rp = rd[p];
    double s = 0.0, t = 0.0, m = 0.0;
    const double far = 1.0 / (kLeadFar * hrr), near = 1.0 / (kLeadNear * hrr);
#pragma unroll 4
    for (int q = lane; q < P; q += 64) {
      const double h = q == p ? 0.0 : fabs(Hb[(long)p * P + q]);
      const double w = h * rp * rd[q];
      s += h;
      t += w;
      if (q >= r - 32 && q > p) m = fmax(m, h * (q >= r ? far : near));
    }
    s = wave_sum(s);
    t = wave_sum(t);
    m = wave_max(m);
    if (lane == 0) {
      off[p] = s;
      link[p] = t < 0.5 && rp > 0.0 && m < 1.0 ? m : 1.0;      // NaN: 1
    }
  }
}

// Reflections 16 a0 .. 16 a0 + 15 (to 16 X - 3) of the Householder reduction of split_kernel's window of 16 X rows.  Reflection k takes row k
// beyond the diagonal to one entry; rows and columns up to k are done.  a0 is a compile-time constant, so that finished
// blocks of 16 cost nothing and the elements stay in registers.
template <int X, int a0>
__device__ __forceinline__ void reflect_block(double (&A)[X][X], double* xs, double* ps, double* dv, double* es) {
  const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
  const int kend = a0 == X - 1 ? 14 : 16;       // k <= 16 X - 3
#pragma unroll 1
  for (int kk = 0; kk < kend; ++kk) {
    const int k = 16 * a0 + kk;
    if (ti == kk) {                             // the owners of row k
#pragma unroll
      for (int y = a0; y < X; ++y) {
        const int j = tj + 16 * y;
        if (j == k) dv[k] = A[a0][y];
        xs[j] = j <= k ? 0.0 : A[a0][y];
      }
    }
    __syncthreads();
    double v[X], vi[X], p[X], ss = 0.0;
#pragma unroll
    for (int y = a0; y < X; ++y) { v[y] = xs[tj + 16 * y]; vi[y] = xs[ti + 16 * y]; }
    const double alpha = xs[k + 1];
#pragma unroll
    for (int y = a0; y < X; ++y) ss = fma(v[y], v[y], ss);
    ss = row16_sum(ss);
    // |row|, and 1 / (|row|^2 + |alpha| |row|): estimates refined by Newton steps.  A row that is zero needs no reflection.
    const bool zero = !(ss > 1e-280);
    const double rs = __builtin_amdgcn_rsq(zero ? 1.0 : ss);
    double nrm = zero ? 0.0 : ss * rs;
    nrm = fma(0.5 * rs, fma(-nrm, nrm, ss), nrm);
    nrm = fma(0.5 * rs, fma(-nrm, nrm, ss), nrm);
    const double den = zero ? 1.0 : fma(fabs(alpha), nrm, ss);
    double hinv = __builtin_amdgcn_rcp(den);
    hinv = fma(hinv, fma(-den, hinv, 1.0), hinv);
    hinv = zero ? 0.0 : fma(hinv, fma(-den, hinv, 1.0), hinv);
    const double v1 = alpha + copysign(nrm, alpha);
    if (tid == 0) es[k] = ss;
#pragma unroll
    for (int y = a0; y < (a0 + 2 < X ? a0 + 2 : X); ++y) {
      if (tj + 16 * y == k + 1) v[y] = v1;
      if (ti + 16 * y == k + 1) vi[y] = v1;
    }
#pragma unroll
    for (int x = a0; x < X; ++x) {
      p[x] = 0.0;
#pragma unroll
      for (int y = a0; y < X; ++y) p[x] = fma(A[x][y], v[y], p[x]);
    }
    row16_sums<X, a0>(p);
#pragma unroll
    for (int x = a0; x < X; ++x) p[x] = ti + 16 * x > k ? p[x] * hinv : 0.0;
    if (tj == 0) {
#pragma unroll
      for (int x = a0; x < X; ++x) ps[ti + 16 * x] = p[x];
    }
    __syncthreads();
    double q[X], dot = 0.0;
#pragma unroll
    for (int y = a0; y < X; ++y) { q[y] = ps[tj + 16 * y]; dot = fma(q[y], v[y], dot); }
    dot = 0.5 * hinv * row16_sum(dot);
#pragma unroll
    for (int y = a0; y < X; ++y) { q[y] = fma(-dot, v[y], q[y]); p[y] = fma(-dot, vi[y], p[y]); }
#pragma unroll
    for (int x = a0; x < X; ++x)
#pragma unroll
      for (int y = a0; y < X; ++y) A[x][y] = fma(-p[x], v[y], fma(-vi[x], q[y], A[x][y]));
  }
}

template <int X, int a0 = 0>
__device__ __forceinline__ void reflect_all(double (&A)[X][X], double* xs, double* ps, double* dv, double* es) {
  if constexpr (a0 < X) {
    reflect_block<X, a0>(A, xs, ps, dv, es);
    reflect_all<X, a0 + 1>(A, xs, ps, dv, es);
  }
}

// See the head of the file.  Workgroups 0 .. B - 1, of 256 threads, take an image each: thread (ti, tj) = (tid / 16, tid % 16) holds the
// elements (ti + 16 x, tj + 16 y) of the window of N rows, x, y < N / 16, in registers; a sum over a row is then 16 lanes of one DPP
// row.  The others profile 16 rows each (a launch of 9 us by itself).  Two barriers per reflection.  Bound by instruction issue (one wave per SIMD, some 400 instructions a reflection; one
// barrier instead of two measured the same): 126 reflections 100 us, a Sturm pass of 128 trial points 6.6.  144 us in all with
// library square roots and divisions and the row sums one after the other, 124 so; a window of 64 rows 45.
template <int N>
__device__ __forceinline__ void split_window(const double* __restrict__ H, int P, long stride, int r, int b, SplitCtl* cb, double* rd) {
  constexpr int X = N / 16;
  double *xs = rd, *ps = rd + N, *dv = rd + 2 * N, *es = rd + 3 * N;   // es: squared off-diagonals
  __shared__ double red[4];
  __shared__ int cnt[2][4];
  const int tid = threadIdx.x, ti = tid >> 4, tj = tid & 15, lane = tid & 63, wv = tid >> 6;
  const double* Hb = H + b * stride;
  const int w0 = P <= N ? 0 : (r - N / 2 < 0 ? 0 : (r - N / 2 > P - N ? P - N : r - N / 2));
  const int nw = P - w0 < N ? P - w0 : N;

  double A[X][X];
  double big = 0.0;
#pragma unroll
  for (int x = 0; x < X; ++x)
#pragma unroll
    for (int y = 0; y < X; ++y) {
      const int i = ti + 16 * x, j = tj + 16 * y;
      A[x][y] = (i < nw && j < nw) ? Hb[(long)(w0 + i) * P + w0 + j] : 0.0;
    }
#pragma unroll
  for (int x = 0; x < X; ++x)
    if (ti == tj) big = fmax(big, A[x][x]);       // H is positive semidefinite: no entry exceeds the largest diagonal entry
  big = wave_max(big);
  if (lane == 0) red[wv] = big;
  __syncthreads();
  big = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  if (!(big > 0.0) || !(big < 1e300)) return;     // zero matrix, infinities, NaN: left to the caller's fallback
  const double scale = 1.0 / big;
#pragma unroll
  for (int x = 0; x < X; ++x)
#pragma unroll
    for (int y = 0; y < X; ++y) A[x][y] *= scale;

  // ---- Householder reduction
  reflect_all<X>(A, xs, ps, dv, es);
  if (ti >= 14 && tj >= 14) {
    if (ti == tj) dv[N - 16 + ti] = A[X - 1][X - 1];
    else if (ti == 14) es[N - 2] = A[X - 1][X - 1] * A[X - 1][X - 1];
  }
  if (tid == 0) es[N - 1] = 0.0;
  __syncthreads();

  // ---- the m-th and (m+1)-th largest eigenvalue of the window, m = r - w0, by Sturm counts.  Threads 0..127 narrow
  //      the interval of the first, the others that of the second, until both are known to 2 % of what separates them.
  double top = 0.0;
  if (tid < N) top = dv[tid] + sqrt(es[tid]) + (tid > 0 ? sqrt(es[tid - 1]) : 0.0);
  top = wave_max(top);
  if (lane == 0) red[wv] = top;
  __syncthreads();
  top = fmax(fmax(red[0], red[1]), fmax(red[2], red[3])) * 1.0001 + 1e-12;
  double lo[2] = {-1e-3 * top, -1e-3 * top}, hi[2] = {top, top};
  const int g = tid >> 7, m = r - w0 + g;
#pragma unroll 1
  for (int pass = 0; pass < 8; ++pass) {
    const double l_ = g ? lo[1] : lo[0], h_ = g ? hi[1] : hi[0];
    const double x = l_ + (h_ - l_) * ((double)((tid & 127) + 1) * (1.0 / 129.0));
    double q = dv[0] - x;
    int neg = q < 0.0 ? 1 : 0;
#pragma unroll 8
    for (int i = 1; i < N; ++i) {
      if (!(fabs(q) > 1e-200)) q = -1e-200;
      double rq = __builtin_amdgcn_rcp(q);
      rq = fma(rq, fma(-q, rq, 1.0), rq);
      q = fma(-es[i - 1], rq, dv[i] - x);
      neg += q < 0.0 ? 1 : 0;
    }
    // N - neg eigenvalues lie at x or above: the m-th largest does where that is at least m
    const unsigned long long yes = __ballot(N - neg >= m);
    if (lane == 0) cnt[pass & 1][wv] = __popcll(yes);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int t = cnt[pass & 1][2 * e] + cnt[pass & 1][2 * e + 1];
      const double w = hi[e] - lo[e], l0 = lo[e], h0 = hi[e];
      if (t > 0) lo[e] = l0 + w * ((double)t * (1.0 / 129.0));
      if (t < 128) hi[e] = fmin(h0, l0 + w * ((double)(t + 1) * (1.0 / 129.0)));
    }
    const double gap = lo[0] - hi[1];
    if (fmax(hi[0] - lo[0], hi[1] - lo[1]) <= 0.02 * gap) break;      // the same in every thread
  }
  const double gap = (lo[0] - hi[1]) * big;
  const double mu = 0.25 * (lo[0] + hi[0] + lo[1] + hi[1]) * big;

  if (tid == 0) {
    cb->mu = mu;
    cb->half = 0.45 * gap;                           // a tenth off the half gap for what the window leaves out
    cb->theta = lo[0] * big;
    cb->state = gap > 0.0 && mu > 0.0 ? 0 : 1;
  }
}

// State of an image's split before its cut is known.
__device__ __forceinline__ void start_ctl(SplitCtl* cb) {
  for (int k = threadIdx.x; k < kMaxSignSteps + 2; k += 256) cb->dev[k] = 0ull;
  if (threadIdx.x == 0) {
    cb->bar.arrived = 0u;
    cb->bar.failed = 0;
    cb->state = 1;
  }
}

// Workgroup `at` of those that profile 16 rows each, P / 16 per image.  X0, X1, Y (optional): the buffers of sign_small_kernel, which finds its
// words at zero.
__device__ __forceinline__ void profile_rows(const double* __restrict__ H, int P, long stride, int r, int at, double* __restrict__ off, double* __restrict__ link,
                                             const int* __restrict__ skip, double* X0, double* X1, double* Y, double* rd) {
  const int per = P / 16, img = at / per;
  if (skip && skip[img]) return;
  if (X0) {
    const long from = img * stride + 16l * (at - img * per) * P;
    const f64x2_t zero = (f64x2_t){0.0, 0.0};
    for (int k = threadIdx.x; k < 8 * P; k += 256) {
      *(f64x2_t*)(X0 + from + 2 * k) = zero;
      *(f64x2_t*)(X1 + from + 2 * k) = zero;
      *(f64x2_t*)(Y + from + 2 * k) = zero;
    }
  }
  row_profile(H + img * stride, P, r, 16 * (at - img * per), off + (long)img * P, link + (long)img * P, rd);
}

// wide: every image has a window of SN rows; else those with again[b] != 0 (optional), the others 64.  rest: only those are left, what
// all have in common is done.
__global__ __launch_bounds__(256) void split_kernel(const double* __restrict__ H, int P, long stride, int B, int r, bool wide, double* __restrict__ off,
                                                    double* __restrict__ link, SplitCtl* ctl, const int* __restrict__ skip,
                                                    const int* __restrict__ again, bool rest, double* X0, double* X1, double* Y) {
  __shared__ double rd[4096];
  if (blockIdx.x >= (unsigned)B) {
    profile_rows(H, P, stride, r, blockIdx.x - B, off, link, skip, X0, X1, Y, rd);
    return;
  }
  const int b = blockIdx.x, tid = threadIdx.x;
  SplitCtl* cb = ctl + b;
  if (rest && !again[b]) return;
  if (!rest) {
    if (b == 0 && tid == 0) ctl[0].ticket = 0u;
    start_ctl(cb);
  }
  if (skip && skip[b]) return;
  if (wide || (again && again[b])) split_window<SN>(H, P, stride, r, b, cb, rd);
  else split_window<64>(H, P, stride, r, b, cb, rd);
}

// ---- The cut of a few images by counting: a matrix less x, A - x I = L D L^T without exchanges, has as many eigenvalues below x as D has
// negative entries, and that is worked out for hundreds of x at once, a wave each.
// Per image kTrials waves (half as many for windows of 128) try points of an interval, tell one another the counts (each with the
// number of the pass), and agree on the next interval until eight points lie between the two eigenvalues.  The first interval of an ordered
// window are the diagonal entries four rows to either side of the cut, otherwise everything.  A wave holds the upper triangle of
// 16 x 16 tiles in its registers and eliminates four pivots at a time: the 4 x 4 block at the pivots in scalars, as eliminate_panel
// (subspace.hip) does without its floors, the rest as products of rank 4.  (A pivot of relative size p perturbs the matrix by 1e-16 / p; that
// this moves an eigenvalue over a trial point, 1e-6 of the norm away and more, takes a pivot below 1e-10.  An exact zero counts for a matrix
// 1e-8 away, see pivots.h.  A count that is wrong shows in the trace of the projector.)
// Bound by the chain of pivots and the MFMAs of a wave.  us, split_kernel and here: one window of 64 44 and 19 (two 44 and 22), of 128 121 and 83.
// A window of 128 is 36 tiles, 288 of a wave's 512 registers: half of them are accumulator registers, 2000 moves between the two kinds a pass of
// 27 us, and 70 others are spilled (84 accesses to scratch memory a pass, 14 of them in the elimination, the rest around the exchange of the
// counts).  A window of 64 has neither.
// Where split_kernel takes over, us of covspec_select by counting / by split_kernel: windows of 128 eight images 184 / 214; windows of 64 in blocks of
// 128 four 306 / 328, five 316 / 330, eight 347 / 352; of 192 three 406 / 425, four 432 / 447, five 477 / 487, eight 560 / 559; of 448 three 1721 / 1736,
// four 1824 / 1819, five 2080 / 2054, eight 2291 / 2265.  (Order 64 as its own window: four 106 / 185, eight 129 / 185.)
constexpr int kCutImages = 8;        // of windows of 128, half as many of 64: a SIMD gets a wave at most
constexpr int kTrials = 256;
constexpr int kCutPasses = 8, kCutPoints = 8;
struct CutArea {
  unsigned int ticket[2], pad[62];             // one per split of the call
  int count[kCutImages][2][kTrials];           // pass << 16 | eigenvalues at the point or above, by turns (who writes the next but one has
                                               // everybody's next one, so everybody has read this one); cleared before the first split
};

template <int NT> __device__ constexpr int tri(int s, int t) { return s * NT - s * (s - 1) / 2 + t - s; }

// Pivots 4 PN .. + 3 of diagonal tile S.
template <int NT, int S, int PN>
__device__ __forceinline__ void count_panel(f64x4_t (&T)[NT * (NT + 1) / 2], int& neg) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  const f64x4_t zero = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  f64x4_t& x = T[tri<NT>(S, S)];
  auto at = [&](int i, int j) { return lane_value(x[PN], 16 * i + 4 * PN + j); };
  const CountedBlock f = count_block(at(0, 0), at(1, 0), at(1, 1), at(2, 0), at(2, 1), at(2, 2), at(3, 0), at(3, 1), at(3, 2), at(3, 3), reciprocal, neg);
  if constexpr (S == NT - 1 && PN == 3) return;
  double n = i16 == kq ? 1.0 : 0.0;
  if (i16 == 1 && kq == 0) n = f.n10;
  if (i16 == 2 && kq == 0) n = f.n20;
  if (i16 == 2 && kq == 1) n = f.n21;
  if (i16 == 3 && kq == 0) n = f.n30;
  if (i16 == 3 && kq == 1) n = f.n31;
  if (i16 == 3 && kq == 2) n = f.n32;
  const double r = kq == 0 ? f.r0 : kq == 1 ? f.r1 : kq == 2 ? f.r2 : f.r3;
  double below = 0.0, u[NT], ru[NT];
  if constexpr (PN < 3) {
    const double w = __builtin_amdgcn_mfma_f64_16x16x4f64(n, x[PN], zero, 0, 0, 0)[0];
    below = (i16 > 4 * PN + 3 ? -r : 0.0) * w;
    x = __builtin_amdgcn_mfma_f64_16x16x4f64(below, w, x, 0, 0, 0);
  }
#pragma unroll
  for (int t = S + 1; t < NT; ++t) {
    u[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(n, T[tri<NT>(S, t)][PN], zero, 0, 0, 0)[0];
    ru[t] = -r * u[t];
    if (PN < 3) T[tri<NT>(S, t)] = __builtin_amdgcn_mfma_f64_16x16x4f64(below, u[t], T[tri<NT>(S, t)], 0, 0, 0);
  }
#pragma unroll
  for (int t = S + 1; t < NT; ++t)
#pragma unroll
    for (int v = t; v < NT; ++v) T[tri<NT>(t, v)] = __builtin_amdgcn_mfma_f64_16x16x4f64(ru[t], u[v], T[tri<NT>(t, v)], 0, 0, 0);
}
template <int NT, int S>
__device__ __forceinline__ void count_from(f64x4_t (&T)[NT * (NT + 1) / 2], int& neg) {
  if constexpr (S < NT) {
    count_panel<NT, S, 0>(T, neg);
    count_panel<NT, S, 1>(T, neg);
    count_panel<NT, S, 2>(T, neg);
    count_panel<NT, S, 3>(T, neg);
    count_from<NT, S + 1>(T, neg);
  }
}

// Workgroups 0 .. B trials / 4 - 1 try four points of an image each, which image and which points by ticket (so that whoever waits for the
// counts of others waits for some that have started or start next), the others profile 16 rows each (see split_kernel).  again:
// images that split_kernel takes instead.  epoch: 0 for the first split of a call, 1 for the second.
template <int N>
__global__ __launch_bounds__(256, N == 64 ? 2 : 1) void cut_kernel(const double* __restrict__ H, int P, long stride, int B, int r, bool ordered, int trials,
                                                                  double* __restrict__ off, double* __restrict__ link, SplitCtl* ctl, CutArea* area, int epoch,
                                                                  const int* __restrict__ skip, const int* __restrict__ again, double* X0, double* X1, double* Y,
                                                                  long long limit_ticks) {
  constexpr int NT = N / 16, PITCH = N + 1;
  extern __shared__ double lds[];               // [N][N + 1], or the profile's reciprocal square roots
  __shared__ double red[8];
  __shared__ int s_ticket;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  const int per = trials / 4;
  if (blockIdx.x >= (unsigned)(B * per)) {
    profile_rows(H, P, stride, r, blockIdx.x - B * per, off, link, skip, X0, X1, Y, lds);
    return;
  }
  if (tid == 0) s_ticket = (int)atomicAdd(&area->ticket[epoch], 1u);
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(s_ticket), b = ticket / per, slot = ticket - b * per;
  SplitCtl* cb = ctl + b;
  if (slot == 0) {
    if (b == 0 && tid == 0) ctl[0].ticket = 0u;
    start_ctl(cb);
  }
  if ((skip && skip[b]) || (again && again[b])) return;
  const double* Hb = H + b * stride;
  const int w0 = P <= N ? 0 : (r - N / 2 < 0 ? 0 : (r - N / 2 > P - N ? P - N : r - N / 2));
  const int nw = P - w0 < N ? P - w0 : N;
  {
    typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int PAIRS = N * N / 512;          // per thread
    pair_t v[PAIRS];
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) {
      const int e = 2 * (tid + 256 * k), i = e / N, j = e % N;        // nw is even
      v[k] = i < nw && j < nw ? *(const pair_t*)(Hb + (long)(w0 + i) * P + w0 + j) : (pair_t){0.0, 0.0};
    }
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) {
      const int e = 2 * (tid + 256 * k), i = e / N, j = e % N;
      lds[i * PITCH + j] = v[k][0];
      lds[i * PITCH + j + 1] = v[k][1];
    }
  }
  __syncthreads();
  double big, top = 0.0;                        // largest diagonal entry (no entry exceeds it), and a bound on the eigenvalues
  {
    constexpr int SHARE = 256 / N;              // threads of a row
    const int i = tid / SHARE, j0 = tid % SHARE * (N / SHARE);
    big = lds[i * PITCH + i];
#pragma unroll 16
    for (int j = 0; j < N / SHARE; ++j) top += fabs(lds[i * PITCH + j0 + j]);
#pragma unroll
    for (int o = 1; o < SHARE; o <<= 1) top += __shfl_xor(top, o, 64);
  }
  big = wave_max(big);
  top = wave_max(top);
  if (lane == 0) { red[wv] = big; red[4 + wv] = top; }
  __syncthreads();
  big = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  top = fmax(fmax(red[4], red[5]), fmax(red[6], red[7]));
  if (!(big > 0.0) || !(top < 1e300)) return;   // zero matrix, infinities, NaN: left to the caller's fallback
  const double scale = 1.0 / big;
  top = top * scale * 1.0001 + 1e-12;
  const int m = r - w0;                         // the m-th largest eigenvalue of the window and the one below it
  double lo = -1e-3 * top, hi = top;
  bool ratios = true;                           // points at equal ratios from 1e-6 of the bound to it, for the first pass over everything
  if (ordered && m >= 5 && m + 4 < nw) {
    const double d0 = lds[(m + 4) * PITCH + m + 4] * scale, d1 = lds[(m - 5) * PITCH + m - 5] * scale;
    if (d0 < d1) { lo = d0; hi = d1; ratios = false; }
  }
  const int mine = 4 * slot + wv;
  bool found = false, alive = true;
  double at0 = 0.0, at1 = 0.0;                  // points between the two eigenvalues, the first and the last
#pragma unroll 1
  for (int pass = 1; pass <= kCutPasses && alive && !found; ++pass) {
    const double dx = (hi - lo) / (double)(trials + 1), l0 = lo;
    auto point = [&](int j) { return ratios ? top * exp2(20.0 * ((double)(j + 1) / (double)(trials + 1) - 1.0)) : l0 + dx * (double)(j + 1); };
    const double x = point(mine);
    f64x4_t T[NT * (NT + 1) / 2];
#pragma unroll
    for (int s = 0; s < NT; ++s)
#pragma unroll
      for (int t = s; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) T[tri<NT>(s, t)][v] = fma(lds[(16 * s + 4 * v + kq) * PITCH + 16 * t + i16], scale, s == t && 4 * v + kq == i16 ? -x : 0.0);
    int neg = 0;
    count_from<NT, 0>(T, neg);
    const int mark = (epoch * kCutPasses + pass) << 16;
    int* counts = area->count[b][pass & 1];
    if (lane == 0) __hip_atomic_store(&counts[mine], mark | (N - neg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // everybody's: lane l looks at l, l + 64, ..
    int c[kTrials / 64];
    long long t0 = 0;
    for (int tries = 0;; ++tries) {
      bool there = true;
#pragma unroll
      for (int q = 0; q < kTrials / 64; ++q) {
        c[q] = 64 * q < trials ? __hip_atomic_load(&counts[64 * q + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : mark;
        there = there && (c[q] & ~0xFFFF) == mark;
      }
      if (!__any(!there)) break;
      __builtin_amdgcn_s_sleep(4);
      if ((tries & 63) == 63) {
        if (tries == 63) t0 = wall_clock64();
        if (wall_clock64() - t0 > limit_ticks) { alive = false; break; }
      }
    }
    if (!alive) break;
    int first = trials, last = -1;              // first point with at most m at it or above, last one with at least m
#pragma unroll
    for (int q = 0; q < kTrials / 64; ++q)
      if (64 * q < trials) {
        const unsigned long long few = __ballot((c[q] & 0xFFFF) <= m), many = __ballot((c[q] & 0xFFFF) >= m);
        if (few && first == trials) first = 64 * q + __ffsll((long long)few) - 1;
        if (many) last = 64 * q + 63 - __clzll((long long)many);
      }
    at0 = point(first);
    at1 = point(last);
    found = last - first >= kCutPoints || (pass == kCutPasses && last > first);
    if (last >= first) {                        // some between the two: closer in on them
      const double l1 = first == 0 ? (pass == 1 ? -1e-3 * top : lo) : point(first - 1);
      hi = last == trials - 1 ? (pass == 1 ? top : hi) : point(last + 1);
      lo = l1;
    } else {                                    // both between two points, or beyond the interval
      const double l1 = last < 0 ? -1e-3 * top : point(last);
      hi = first == trials ? top : point(first);
      lo = l1;
    }
    ratios = false;
  }
  if (slot == 0 && tid == 0) {
    const double gap = (at1 - at0) * big;
    cb->mu = 0.5 * (at0 + at1) * big;
    cb->half = 0.45 * gap;                           // a tenth off the half gap for what the window leaves out
    cb->theta = at1 * big;
    cb->state = found && gap > 0.0 && cb->mu > 0.0 ? 0 : 1;
  }
}

constexpr int ST = 32;            // tile of a wave in the sign iteration
constexpr int STP = ST + 1;

// The iterates are kept as [P/16][P/16] tiles in fragment order (common.h), both triangles.
__device__ __forceinline__ long tile16(int rt, int ct, int P) { return ((long)rt * (P >> 4) + ct) * kFragTile; }

// Tile (r0, c0), 32 x 32, of X Z for symmetric X, Z of order P, k over [k0, k0 + kn), kn % 16 == 0: one wave, operands
// straight from global memory, DEPTH groups of 16 k in flight; the result goes to `out` (LDS).
template <int DEPTH>
__device__ __forceinline__ void tile_product(const double* X, const double* Z, int P, int k0, int kn, int r0, int c0, double* out) {
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = lane >> 4;
  const double* xr = X + tile16(r0 >> 4, k0 >> 4, P);
  const double* zr = Z + tile16(c0 >> 4, k0 >> 4, P);
  const long step = tile16(1, 0, P);
  f64x4_t acc[2][2], fx[DEPTH][2], fz[DEPTH][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  const int nc = kn >> 4;
  auto load = [&](int s, int c) {
    if (c < nc) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        fx[s][x] = frag_load(xr + x * step + c * kFragTile, lane);
        fz[s][x] = frag_load(zr + x * step + c * kFragTile, lane);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) load(s, s);
#pragma unroll 1
  for (int c = 0; c < nc; c += DEPTH) {
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      if (c + s < nc) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(fx[s][x][k], fz[s][y][k], acc[x][y], 0, 0, 0);
        load(s, c + s + DEPTH);
      }
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(16 * x + 4 * v + kq) * STP + 16 * y + i16] = acc[x][y][v];
}

__device__ __forceinline__ void tile_of(int t, int& i, int& j) {      // t-th tile on or below the diagonal, row by row
  int q = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((q + 1) * (q + 2) / 2 <= t) ++q;
  while (q * (q + 1) / 2 > t) --q;
  i = q;
  j = t - q * (q + 1) / 2;
}

// Rows that are wanted as they are (those before the returned one, a multiple of 64), and the norm of the rest: the same in every
// workgroup of the image.  red: WAVES doubles of LDS.
template <int WAVES>
__device__ __forceinline__ int leading_rows(const double* __restrict__ Hb, const double* __restrict__ off, const double* __restrict__ link, int P, int r,
                                            bool ordered, double mu, double* red, double& norm) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int a = 0;
  if (ordered) {
    int bad = r - 32;                                // first row that couples across the cut
    for (int p = tid; p < r - 32; p += 64 * WAVES)
      if (!(link[p] < 1.0 && 0.5 * Hb[(long)p * P + p] > mu)) bad = p < bad ? p : bad;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { const int t = __shfl_xor(bad, o, 64); bad = t < bad ? t : bad; }
    if (lane == 0) red[wv] = (double)bad;
    __syncthreads();
    double m = red[0];
    for (int w = 1; w < WAVES; ++w) m = fmin(m, red[w]);
    a = m < 64.0 ? 0 : (int)m / 64 * 64;
    __syncthreads();
  }
  norm = 0.0;
  for (int p = a + tid; p < P; p += 64 * WAVES) norm = fmax(norm, fabs(Hb[(long)p * P + p]) + off[p]);
  norm = wave_max(norm);
  if (lane == 0) red[wv] = norm;
  __syncthreads();
  for (int w = 0; w < WAVES; ++w) norm = fmax(norm, red[w]);
  __syncthreads();
  return a;
}

// The whole iteration of all images: workgroup (image, slot) owns the tiles slot, slot + W, ... on and below the
// diagonal and stores each also transposed; the workgroups of an image meet after every product.  (Image, slot)
// pairs are handed out by a ticket counter, so that resident workgroups always form whole images plus at most one
// partial image whose missing workgroups start next; every wait is bounded.
// X0, X1, Y: P x P per image; the projector is left in Y.
// What the workgroups hand one another is stored through the L2 (store_through), which spares the write-back of a whole L2
// at every meeting: eight images of order 192 to 320 took 553 us with write-backs and 366 us without (a single image of
// order 192: 259 and 292 us, sixty-four of order 256: 1.70 and 1.53 ms).  The iterates in fragment order instead of row-major
// (64 cache lines per load): 366 -> 259, 292 -> 197 us, 1.53 -> 1.06 ms.
// WIDE = false: a workgroup's tile is 32 x 32, its waves take a quarter of k each; WIDE = true: the tile is 64 x 64, a
// wave takes a quadrant of it and all of k, or half of it with KS = 2 (a quarter of the workgroups: sixty-four images of order
// 256 took 3.7 ms on small tiles, whose workgroups the device holds only a quarter of at a time, and 1.7 ms on wide ones).
// Everything is kept symmetric to the bit (the elements above the diagonal are those below it): rounding that differs
// between the two would be a skew perturbation, which the iteration magnifies by 1 / l0.
template <bool WIDE, int KS>
__global__ __launch_bounds__(256 * KS, WIDE && KS == 1 ? 3 : 2) void sign_kernel(const double* __restrict__ H, double* X0, double* Y, double* X1, int P,
                                                                 int r, const double* __restrict__ off, const double* __restrict__ link, bool ordered,
                                                                 int W, SplitCtl* ctl, long long limit_ticks) {
  static_assert(WIDE || KS == 1, "");
  constexpr int TT = WIDE ? 2 * ST : ST;             // tile of the workgroup
  extern __shared__ double part[];                   // [4 KS][ST][STP], one tile of 32 x 32 per wave
  __shared__ int s_flag;
  __shared__ double s_dev[4 * KS];
  const int tid = threadIdx.x, wv = tid >> 6, grp = wv >> 2, lane = tid & 63, i16 = lane & 15, kq = lane >> 4;
  if (tid == 0) s_flag = (int)atomicAdd(&ctl[0].ticket, 1u);
  __syncthreads();
  const int ticket = s_flag;
  __syncthreads();                                   // s_flag is reused by the barriers
  const int b = ticket / W, slot = ticket - b * W;
  SplitCtl* cb = ctl + b;
  if (cb->state != 0) return;                        // set before the launch; nobody of this image writes it before all have read it
  double norm;
  const int a = leading_rows<4 * KS>(H + b * (long)P * P, off + (long)b * P, link + (long)b * P, P, r, ordered, cb->mu, s_dev, norm);
  if (!(cb->half > kMinGap * norm && norm < 1e300)) return;      // no usable gap: the image gets no projector
  const int ns = (P - a) / TT, ntiles = ns * (ns + 1) / 2;
  const int nact = ntiles < W ? ntiles : W;
  if (slot >= nact) return;
  // cut and half gap as parts of the norm, and the number of lifting steps that follows from them
  double m = cb->mu / norm, l = cb->half / norm;
  const bool lift = m < kLiftTo;
  const double mu = lift ? 0.0 : cb->mu, inv = 1.0 / (lift ? norm : fmax(norm - mu, mu));
  if (!lift) l = cb->half * inv;
  const long pp = (long)P * P;
  const double* Hb = H + b * pp;
  double *X = X0 + b * pp, *Xn = X1 + b * pp, *Yb = Y + b * pp;
  unsigned int target = 0;
  bool alive = true, done = false;
  auto meet = [&]() {
    target += nact;
    alive = image_barrier_wait<false>(&cb->bar, target, &s_flag, limit_ticks);
  };
  // fn(r0, c0, above) on the 32 x 32 tiles on and below the diagonal that this wave helps to store; above: this one is above
  // the diagonal (and left out)
  auto for_tiles = [&](auto fn) {
    for (int t = slot; t < ntiles; t += W) {
      int ti, tj;
      tile_of(t, ti, tj);
      if (WIDE) {
        const int qi = (wv >> 1) & 1, qj = wv & 1;
        fn(a + TT * ti + ST * qi, a + TT * tj + ST * qj, ti == tj && qj > qi);
      } else {
        fn(a + TT * ti, a + TT * tj, false);
      }
    }
  };
  // fn(tile row, tile column), in units of 16, on the 16 x 16 tiles of a 32 x 32 tile, dealt to the waves that share it
  auto for_frags = [&](int r0, int c0, auto fn) {
    for (int q = WIDE ? grp : wv; q < 4; q += WIDE ? KS : 4) fn((r0 >> 4) + (q >> 1), (c0 >> 4) + (q & 1));
  };
  // the 32 x 32 tiles of the product X Z in LDS, then fn(r0, c0, sum) with sum(i, j) an element of it
  auto product = [&](const double* Z, auto fn) {
    for_tiles([&](int r0, int c0, bool above) {
      double* mine = part + wv * (ST * STP);
      const int kn = WIDE ? (P - a) / KS : (P - a) >> 2;     // P - a is a multiple of 64
      if (!above) tile_product<WIDE ? 2 : 3>(X, Z, P, a + (WIDE ? grp : wv) * kn, kn, r0, c0, mine);
      __syncthreads();
      auto sum = [&](int i, int j) {
        const double* q = part + (WIDE ? (wv & 3) * (ST * STP) : 0) + i * STP + j;
        return WIDE ? (KS == 2 ? q[0] + q[4 * ST * STP] : q[0]) : (q[0] + q[ST * STP]) + (q[2 * ST * STP] + q[3 * ST * STP]);
      };
      if (!above) fn(r0, c0, sum);
      __syncthreads();
    });
  };
  // a lane's element v of tile (rt, ct) is (16 rt + i16, 16 ct + 4 v + kq)
  auto put = [&](double* M, int rt, int ct, const f64x4_t& x) {
    double* t = M + tile16(rt, ct, P) + 2 * lane;
    store_through(t, x[0]);
    store_through(t + 1, x[1]);
    store_through(t + 128, x[2]);
    store_through(t + 129, x[3]);
  };
  for_tiles([&](int r0, int c0, bool above) {
    if (above) return;
    for_frags(r0, c0, [&](int rt, int ct) {
      f64x4_t x, y;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        // the element above the diagonal serves for both
        const int i = 16 * rt + i16, j = 16 * ct + 4 * v + kq, i2 = 16 * ct + i16, j2 = 16 * rt + 4 * v + kq;
        x[v] = ((i < j ? Hb[(long)i * P + j] : Hb[(long)j * P + i]) - (i == j ? mu : 0.0)) * inv;
        y[v] = Hb[(long)(i2 < j2 ? i2 : j2) * P + (i2 < j2 ? j2 : i2)] * inv;
      }
      put(X, rt, ct, x);
      if (r0 != c0) put(X, ct, rt, y);
    });
  });
  meet();
#pragma unroll 1
  while (alive && m < kLiftTo) {
    // y = alpha x - beta x^2 is at most 1, and y(1) = y(3 m): what is wanted stays above the image of the cut
    const double top = 3.0 * m, al = 4.0 / (1.0 + top), be = al / (1.0 + top);
    const double cut = m * (al - be * m), gap = l * (al - be * (2.0 * m + l));
    const bool last = cut >= kLiftTo;                // then also shifted and scaled to [-1, 1]
    const double shift = last ? cut : 0.0, sc = last ? 1.0 / (1.0 - cut) : 1.0;
    product(X, [&](int r0, int c0, auto sum) {
      for_frags(r0, c0, [&](int rt, int ct) {
        const int i = 16 * rt - r0 + i16, j = 16 * ct - c0 + kq, i2 = 16 * ct - c0 + i16, j2 = 16 * rt - r0 + kq;
        f64x4_t x = frag_load(X + tile16(rt, ct, P), lane);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          x[v] = (fma(al, x[v], -be * sum(i, j + 4 * v)) - (16 * rt + i16 == 16 * ct + 4 * v + kq ? shift : 0.0)) * sc;
        put(Xn, rt, ct, x);
        if (r0 != c0) {
          f64x4_t y = frag_load(X + tile16(ct, rt, P), lane);
#pragma unroll
          for (int v = 0; v < 4; ++v) y[v] = fma(al, y[v], -be * sum(j2 + 4 * v, i2)) * sc;
          put(Xn, ct, rt, y);
        }
      });
    });
    meet();
    m = cut;
    l = gap * sc;
    double* tmp = X; X = Xn; Xn = tmp;
  }
  int step = 0;
#pragma unroll 1
  for (; alive && !done && step < kMaxSignSteps; ++step) {
    const double s = sqrt(3.0 / (1.0 + l + l * l)), c1 = 1.5 * s, c3 = -0.5 * s * s * s;
    product(X, [&](int r0, int c0, auto sum) {       // Y = X X (a diagonal tile is symmetric: the same products in the same order)
      for_frags(r0, c0, [&](int rt, int ct) {
        const int i = 16 * rt - r0 + i16, j = 16 * ct - c0 + kq, i2 = 16 * ct - c0 + i16, j2 = 16 * rt - r0 + kq;
        put(Yb, rt, ct, (f64x4_t){sum(i, j), sum(i, j + 4), sum(i, j + 8), sum(i, j + 12)});
        if (r0 != c0) put(Yb, ct, rt, (f64x4_t){sum(j2, i2), sum(j2 + 4, i2), sum(j2 + 8, i2), sum(j2 + 12, i2)});
      });
    });
    meet();
    if (!alive) break;
    double dev = 0.0;
    product(Yb, [&](int r0, int c0, auto sum) {      // Xn = c1 X + c3 X Y
      for_frags(r0, c0, [&](int rt, int ct) {
        const int i = 16 * rt - r0 + i16, j = 16 * ct - c0 + kq, i2 = 16 * ct - c0 + i16, j2 = 16 * rt - r0 + kq;
        const f64x4_t x = frag_load(X + tile16(rt, ct, P), lane);
        f64x4_t xn;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          xn[v] = fma(c3, r0 == c0 && j + 4 * v > i ? sum(j + 4 * v, i) : sum(i, j + 4 * v), c1 * x[v]);
          const double d = fabs(xn[v] - x[v]);
          dev = d > dev || !(d == d) ? (d == d ? d : INFINITY) : dev;
        }
        put(Xn, rt, ct, xn);
        if (r0 != c0) {
          const f64x4_t y = frag_load(X + tile16(ct, rt, P), lane);
#pragma unroll
          for (int v = 0; v < 4; ++v) xn[v] = fma(c3, sum(j2 + 4 * v, i2), c1 * y[v]);
          put(Xn, ct, rt, xn);
        }
      });
    });
    dev = wave_max(dev);
    if ((tid & 63) == 0) s_dev[wv] = dev;
    __syncthreads();
    if (tid == 0) {
      double m = s_dev[0];
#pragma unroll
      for (int w = 1; w < 4 * KS; ++w) m = fmax(m, s_dev[w]);
      atomicMax(&cb->dev[step], (unsigned long long)__double_as_longlong(m));
    }
    meet();
    if (!alive) break;
    l = fmin(1.0, c1 * l + c3 * l * l * l);
    const double change =
        __longlong_as_double((long long)__hip_atomic_load(&cb->dev[step], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    // near its limit the iteration squares the error: an entry that moved by 1e-7 is 1e-14 away afterwards
    done = l > 1.0 - 1e-6 && change < 1e-7;
    double* tmp = X; X = Xn; Xn = tmp;
  }
  if (done) {
    // the projector, row-major: the fragment of tile (row, column) is stored as tile (column, row)
    for_tiles([&](int r0, int c0, bool above) {
      if (above) return;
      for_frags(r0, c0, [&](int rt, int ct) {
        const f64x4_t x = frag_load(X + tile16(rt, ct, P), lane), y = frag_load(X + tile16(ct, rt, P), lane);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = 16 * rt + i16, j = 16 * ct + 4 * v + kq, i2 = 16 * ct + i16, j2 = 16 * rt + 4 * v + kq;
          Yb[(long)j * P + i] = 0.5 * (x[v] + (i == j ? 1.0 : 0.0));
          if (r0 != c0) Yb[(long)j2 * P + i2] = 0.5 * y[v];
        }
      });
    });
    for (int p = slot; p < P; p += nact)             // the rows and columns before a: identity
      for (int q = tid; q < (p < a ? P : a); q += 256 * KS) Yb[(long)p * P + q] = p == q ? 1.0 : 0.0;
  }
  if (slot == 0 && tid == 0) cb->state = done ? 2 : 3;   // every workgroup of the image has read it (behind a barrier, or gave up)
}

// The iteration of small matrices (P <= 64 kSmallBlocks): a workgroup per 16 x 16 tile on and below the diagonal, its waves a quarter of k
// each, and no meetings: what a workgroup hands on carries the number of its version in a bit of every element, and the others read an
// element until it is the one they want.
//   The bit is the upper one of the exponent, which only numbers from 2 on have: the iterates are symmetric with eigenvalues in [-1, 1], or
//   their squares, and so are their elements.  (An element that is none of these, NaN included, ends the image's iteration: no projector.)
//   Version v goes to buffer v % 3, the bits are 1, 0, 1, .. with each use of the buffer (cleared before the launch).  A
//   workgroup reads version v - 1 of the tiles in its rows (and columns) to form its part of version v; the left operand of the second
//   product of a step, X, is still in its registers.  So whoever reads a tile's version v - 3 is through with it before version v of
//   the tile is formed; and a workgroup stores version v when the stores of v - 1 have been acknowledged, so that nobody who has
//   anything of version v can still find the words of v - 3 elsewhere.  The operands are loaded past the L2s, which are not coherent.
// Only the steps that may be the last, by the lower bound l, meet at the barrier: they are when no element moved by more than 1e-7.
// Bound by latency: store, load, 3 MFMAs a group of 16 k and wave, four partial sums.  (Five workgroups a compute unit at order 256 leave 96
// registers a wave: 19 are spilled, 12 accesses to scratch memory a step.)  us per product with 32 x 32 tiles and a barrier in
// global memory after each (store, acknowledge, count, see the count, load) and here: one image of order 192 7.0 and 3.4 (155 and 76 in all),
// four 7.1 and 5.3, one of 128 5 and 2.8 (115 and 63).
constexpr int kSmallBlocks = 4;
constexpr int kVersionBit = 0x40000000;              // in the upper word
__device__ __forceinline__ double with_version(double v, int bit) { return __hiloint2double((__double2hiint(v) & ~kVersionBit) | bit, __double2loint(v)); }
__device__ __forceinline__ double without_version(double v) { return __hiloint2double(__double2hiint(v) & ~kVersionBit, __double2loint(v)); }

// BLOCKS = P / 64.
template <int BLOCKS>
__global__ __launch_bounds__(256, BLOCKS == 4 ? 5 : 4) void sign_small_kernel(const double* __restrict__ H, double* X0, double* Y, double* X1, int P, int r,
                                                            const double* __restrict__ off, const double* __restrict__ link, bool ordered, int W,
                                                            SplitCtl* ctl, long long limit_ticks) {
  __shared__ double part[2][4][16][17];
  __shared__ double s_dev[4];
  __shared__ int s_flag, s_fail[2];                  // s_fail: of this product and the next, by turns, as part
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, i16 = lane & 15, kq = lane >> 4;
  if (tid == 0) { s_flag = (int)atomicAdd(&ctl[0].ticket, 1u); s_fail[0] = s_fail[1] = 0; }
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane(s_flag);
  __syncthreads();                                   // s_flag is reused by the barriers
  const int b = ticket / W, slot = ticket - b * W;
  SplitCtl* cb = ctl + b;
  if (cb->state != 0) return;                        // set before the launch; nobody of this image writes it before all have read it
  const long pp = (long)P * P;
  const double* Hb = H + b * pp;
  double norm;
  const int a = leading_rows<4>(Hb, off + (long)b * P, link + (long)b * P, P, r, ordered, cb->mu, s_dev, norm);
  if (!(cb->half > kMinGap * norm && norm < 1e300)) return;      // no usable gap: the image gets no projector
  const int ns = (P - a) >> 4, nact = ns * (ns + 1) / 2;
  if (slot >= nact) return;
  int ti, tj;
  tile_of(slot, ti, tj);
  const int rt = (a >> 4) + ti, ct = (a >> 4) + tj;
  norm = lane_value(norm, 0);                        // the same in all lanes: the loops below are those of a wave, the buffers scalars
  // the lift and the steps, as in sign_kernel
  double m = cb->mu / norm, l = cb->half / norm;
  const bool lift = m < kLiftTo;
  const double mu = lift ? 0.0 : cb->mu, inv = 1.0 / (lift ? norm : fmax(norm - mu, mu));
  if (!lift) l = cb->half * inv;
  double* buf[3] = {X0 + b * pp, X1 + b * pp, Y + b * pp};       // version v is in buf[v % 3]
  __amdgpu_buffer_rsrc_t rs[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) rs[k] = __builtin_amdgcn_make_buffer_rsrc((void*)buf[k], (short)0, (int)(pp * 8), 0x00020000);

  // this thread's element of the tile in fragment order, and the one it has of the tile across the diagonal
  const int ei = (tid >> 1) & 15, ek = ((tid >> 7) << 3) | ((tid & 1) << 2) | ((tid >> 5) & 3);
  const bool diagonal = rt == ct;
  const int ui = diagonal && ek > ei ? ek : ei, uk = diagonal && ek > ei ? ei : ek;      // what is above the diagonal is what is below
  unsigned version = 0;
  bool alive = true;
  int parity = 0;                                    // of the last product
  auto publish = [&](double x, double y) {           // the next version
    const int bit = version / 3 % 2 == 0 ? kVersionBit : 0;
    if (!(fabs(x) < 2.0 && (diagonal || fabs(y) < 2.0))) s_fail[parity ^ 1] = 1;     // (on the diagonal y is not used)
    double* M = version % 3 == 0 ? buf[0] : version % 3 == 1 ? buf[1] : buf[2];
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): the version before
    store_through(M + tile16(rt, ct, P) + tid, with_version(x, bit));
    if (!diagonal) store_through(M + tile16(ct, rt, P) + tid, with_version(y, bit));
    ++version;
  };
  const int nc = ns >> 2;                            // groups of 16 k of a wave
  // The wave's groups of row tiles rt (both: f[0]) and ct (f[1]) of the last version.
  f64x2_t f[2][BLOCKS][2];
  auto fetch = [&](bool both) {
    const unsigned v = version - 1;
    const bool one = v / 3 % 2 == 0;
    const __amdgpu_buffer_rsrc_t M = v % 3 == 0 ? rs[0] : v % 3 == 1 ? rs[1] : rs[2];
    const int base[2] = {(int)(tile16(rt, (a >> 4) + wv * nc, P) * 8) + 16 * lane, (int)(tile16(ct, (a >> 4) + wv * nc, P) * 8) + 16 * lane};
    long long t0 = 0;
    const unsigned groups = (1u << nc) - 1;
    unsigned todo = groups << BLOCKS | (both ? groups : 0);
    // What is on its way takes longer than this, and tries that come too early stand in its way.  us of covspec_select without it, and with 8 / 16 / 28 times
    // 64 clocks: two of order 64 103 and 103 / 106 / 113, eight of 128 192 and 186 / 184 / 187, twenty-three 291 and 280 / 269 / 257, one of 192 373
    // and 370 / 370 / 375, seven 536 and 526 / 520 / 516, one of 256 597 and 597 / 598 / 606.
    __builtin_amdgcn_s_sleep(BLOCKS == 1 ? 8 : 16);
    for (int tries = 0; todo != 0; ++tries) {
      asm volatile("" ::: "memory");                 // loads anew
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < BLOCKS; ++c)
          if (todo >> (BLOCKS * q + c) & 1) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
              f[q][c][h] = __builtin_bit_cast(f64x2_t, __builtin_amdgcn_raw_buffer_load_b128(M, base[q], c * (kFragTile * 8) + 1024 * h, kLoadAgent));
          }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < BLOCKS; ++c)
          if (todo >> (BLOCKS * q + c) & 1) {
            const f64x2_t u = f[q][c][0], w = f[q][c][1];
            const int all = __double2hiint(u[0]) & __double2hiint(u[1]) & __double2hiint(w[0]) & __double2hiint(w[1]);
            const int some = __double2hiint(u[0]) | __double2hiint(u[1]) | __double2hiint(w[0]) | __double2hiint(w[1]);
            if (!__any(((one ? ~all : some) & kVersionBit) != 0)) {
              todo &= ~(1u << (BLOCKS * q + c));
              f[q][c][0] = (f64x2_t){without_version(u[0]), without_version(u[1])};
              f[q][c][1] = (f64x2_t){without_version(w[0]), without_version(w[1])};
            }
          }
      if (todo != 0 && (tries & 63) == 63) {         // 64 tries: some 60 us
        if (tries == 63) t0 = wall_clock64();
        if (__hip_atomic_load(&cb->bar.failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || wall_clock64() - t0 > limit_ticks) {
          if (lane == 0) s_fail[parity ^ 1] = 1;
          break;
        }
      }
    }
  };
  // partial sums of the product of the groups; false: gave up
  auto product = [&]() {
    f64x4_t acc = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < BLOCKS; ++c)
      if (c < nc) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[0][c][k >> 1][k & 1], f[1][c][k >> 1][k & 1], acc, 0, 0, 0);
      }
    parity ^= 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) part[parity][wv][4 * v + kq][i16] = acc[v];
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(s_fail[parity]) == 0;
  };
  auto sum = [&](int i, int k) { return (part[parity][0][i][k] + part[parity][1][i][k]) + (part[parity][2][i][k] + part[parity][3][i][k]); };

  double x, y;                                       // this thread's elements of X
  {
    auto start = [&](int i, int j) { return ((i < j ? Hb[(long)i * P + j] : Hb[(long)j * P + i]) - (i == j ? mu : 0.0)) * inv; };
    x = start(16 * rt + ei, 16 * ct + ek);           // the element above the diagonal serves for both
    y = start(16 * ct + ei, 16 * rt + ek);
  }
  publish(x, y);
#pragma unroll 1
  while (alive && m < kLiftTo) {
    const double top = 3.0 * m, al = 4.0 / (1.0 + top), be = al / (1.0 + top);
    const double cut = m * (al - be * m), gap = l * (al - be * (2.0 * m + l));
    const bool last = cut >= kLiftTo;                // then also shifted and scaled to [-1, 1]
    const double shift = last ? cut : 0.0, sc = last ? 1.0 / (1.0 - cut) : 1.0;
    fetch(true);
    if (!(alive = product())) break;
    x = (fma(al, x, -be * sum(ui, uk)) - (diagonal && ei == ek ? shift : 0.0)) * sc;
    y = fma(al, y, -be * sum(ek, ei)) * sc;
    publish(x, y);
    m = cut;
    l = gap * sc;
  }
  bool done = false;
  unsigned int target = 0;
#pragma unroll 1
  for (int step = 0; alive && !done && step < kMaxSignSteps; ++step) {
    const double s = sqrt(3.0 / (1.0 + l + l * l)), c1 = 1.5 * s, c3 = -0.5 * s * s * s;
    fetch(true);
    if (!(alive = product())) break;
    publish(sum(ui, uk), sum(ek, ei));               // Y = X X
    fetch(false);
    if (!(alive = product())) break;
    const double nx = fma(c3, sum(ui, uk), c1 * x), ny = fma(c3, sum(ek, ei), c1 * y);     // c1 X + c3 X Y
    const double moved = fabs(nx - x);
    x = nx;
    y = ny;
    publish(x, y);
    l = fmin(1.0, c1 * l + c3 * l * l * l);
    if (l > 1.0 - 1e-6) {
      double dev = !(moved == moved) ? INFINITY : moved;
      dev = wave_max(dev);
      if (lane == 0) s_dev[wv] = dev;
      __syncthreads();
      if (tid == 0)
        atomicMax(&cb->dev[step], (unsigned long long)__double_as_longlong(fmax(fmax(s_dev[0], s_dev[1]), fmax(s_dev[2], s_dev[3]))));
      target += nact;
      if (!(alive = __builtin_amdgcn_readfirstlane(image_barrier_wait<false>(&cb->bar, target, &s_flag, limit_ticks)))) break;
      // near its limit the iteration squares the error: an entry that moved by 1e-7 is 1e-14 away afterwards
      done = __longlong_as_double((long long)__hip_atomic_load(&cb->dev[step], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < 1e-7;
    }
  }
  if (done) {
    // the projector, row-major; nobody reads the buffers any more
    double* Yb = Y + b * pp;
    const int i = 16 * rt + ei, j = 16 * ct + ek;
    Yb[(long)i * P + j] = 0.5 * (x + (i == j ? 1.0 : 0.0));
    if (!diagonal) Yb[(long)(16 * ct + ei) * P + 16 * rt + ek] = 0.5 * y;
    for (int p = slot; p < P; p += nact)             // the rows and columns before a: identity
      for (int q = tid; q < (p < a ? P : a); q += 256) Yb[(long)p * P + q] = p == q ? 1.0 : 0.0;
  } else if (!alive && tid == 0) {
    __hip_atomic_store(&cb->bar.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (slot == 0 && tid == 0) cb->state = done ? 2 : 3;   // every workgroup of the image has read it (behind a barrier, or gave up)
}

// A workgroup that gave up has not stored its part, whatever slot 0 went on to report.
__device__ __forceinline__ bool projector_valid(const SplitCtl* cb) { return cb->state == 2 && cb->bar.failed == 0; }

// |trace(Pi) - r| tells whether the cut really has r eigenvalues above it.
__device__ __forceinline__ double trace_minus(const double* Pi, int P, int r, double* red, int threads) {
  double t = 0.0;
  for (int p = threadIdx.x; p < P; p += threads) t += Pi[(long)p * P + p];
  t = wave_sum(t);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  t = 0.0;
  for (int w = 0; w < threads / 64; ++w) t += red[w];
  return fabs(t - (double)r);
}

// Residual check of the dominant subspace and, where it holds, the energies.  With Q the orthonormal rows of the block,
// U = Pi Q and R = Pi Q G - H U (zero where the rows of U span an invariant subspace of G), rnorm holds the squared
// lengths of R's rows, one partial sum per column tile.  Row p of the block carries eigenvalues of about H_pp, so
// |R_p| <= tol max(H_pp, theta_r) is the relative residual of the eigenpairs in it.  ok[b] = pass_no, else 0.
// c[b][i] = sum over the row tiles of cpart: the products of column i of U with column i of Q G.
__global__ __launch_bounds__(1024) void split_finish_kernel(const double* __restrict__ H, const double* __restrict__ Pi,
                                                            const double* __restrict__ rnorm, int rparts, const double* __restrict__ cpart,
                                                            int cparts, int P, int n, int nP, int r, double tol,
                                                            const SplitCtl* __restrict__ ctl, const int* slow, int* ok, int pass_no,
                                                            float* __restrict__ c, NextPass next) {
  __shared__ double red[16];
  __shared__ int bad;
  const int b = blockIdx.x, B = gridDim.x;
  if (pass_no > 1 && ok[b]) return;                  // passed an earlier check; its energies are in place
  const bool split = !slow[b];                       // in this pass
  __shared__ int gave_up;
  if (threadIdx.x == 0) {
    bad = gave_up = 0;
    if (next.state)
      for (int k = 0; k < next.sets_before; ++k) gave_up |= next.flags[((long)k * B + b) * next.flag_words + next.failed_word];
  }
  __syncthreads();
  if (next.state)
    for (int k = threadIdx.x; k < next.flag_sets * next.flag_words; k += 1024) {
      const int set = k / next.flag_words;
      next.flags[((long)set * B + b) * next.flag_words + k - set * next.flag_words] = 0;
    }
  __syncthreads();
  const bool valid = split && projector_valid(ctl + b);
  const double theta = ctl[b].theta;
  if (valid) {
    const double off = trace_minus(Pi + (long)b * P * P, P, r, red, 1024);
    if (threadIdx.x == 0 && !(off < 1e-3)) bad = 1;
    for (int p = threadIdx.x; p < P; p += 1024) {
      const double* rp = rnorm + ((long)b * P + p) * rparts;
      double s = 0.0;
      for (int t = 0; t < rparts; ++t) s += rp[t];
      const double ref = fmax(H[((long)b * P + p) * P + p], theta);
      if (!(sqrt(s) <= tol * ref)) bad = 1;          // also catches NaN
    }
  }
  __syncthreads();
  const bool good = valid && bad == 0;
  if (threadIdx.x == 0) {
    ok[b] = good ? pass_no : 0;
    if (next.state) {
      const int at = next.prev[3 * B + b];
      next.state[b] = good || gave_up ? 2 : 0;
      next.state[B + b] = 0;
      next.state[2 * B + b] = at;
      next.state[3 * B + b] = at;
      next.state[4 * B + b] = next.prev[4 * B + b];
      next.redo[(long)b * next.redo_step] = !good && split;
      next.failed[b] = !good && split;
      next.left[b] = good || gave_up;
    }
  }
  if (!good) return;
  for (int i = threadIdx.x; i < n; i += 1024) {
    double s = 0.0;
    for (int t = 0; t < cparts; ++t) s += cpart[((long)b * cparts + t) * nP + i];
    c[(long)b * n + i] = (float)s;
  }
}

// c[b][i] = (Pi G)_ii for a projector of the Gram matrix itself; done[b] = 3 where the projector is valid, else 0.  One wave per row.
__global__ __launch_bounds__(256) void direct_energy_kernel(const double* __restrict__ G, const double* __restrict__ Pi, int n, int nP, int r,
                                                            const SplitCtl* __restrict__ ctl, int* __restrict__ done, float* __restrict__ c) {
  __shared__ double red[4];
  const int b = blockIdx.y, lane = threadIdx.x & 63;
  const long base = (long)b * nP * nP;
  bool good = projector_valid(ctl + b);              // uniform
  if (good) good = trace_minus(Pi + base, nP, r, red, 256) < 1e-3;
  if (blockIdx.x == 0 && threadIdx.x == 0) done[b] = good ? 3 : 0;
  if (!good) return;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;
  double s = 0.0;
  for (int j = lane; j < nP; j += 64) s = fma(G[base + (long)i * nP + j], Pi[base + (long)i * nP + j], s);
  s = wave_sum(s);
  if (lane == 0) c[(long)b * n + i] = (float)s;
}

}  // namespace

namespace {
inline size_t split_base_bytes(int B, int P) { return (sizeof(SplitCtl) * (size_t)B + 255) / 256 * 256 + 2 * (size_t)B * P * 8; }
}
size_t split_scratch_bytes(int B, int P) { return split_base_bytes(B, P) + (B <= kCutImages ? sizeof(CutArea) : 0); }
void* split_cleared(void* scratch, int B, int P, size_t* bytes) {
  *bytes = B <= kCutImages ? sizeof(CutArea) : 0;
  return (char*)scratch + split_base_bytes(B, P);
}

hipError_t launch_spectral_split(const double* H, int B, int P, int r, bool ordered, double* X0, double* Y, double* X1, void* scratch,
                                 const int* skip, const int* again, int epoch, hipStream_t st) {
  if (P < 64 || P % 64 != 0 || P > 4096 || r < 1 || r >= P || (!ordered && P > SN)) return hipErrorInvalidValue;
  SplitCtl* ctl = (SplitCtl*)scratch;
  double* off = (double*)((char*)scratch + (sizeof(SplitCtl) * (size_t)B + 255) / 256 * 256);
  double* link = off + (size_t)B * P;
  const long n32 = P / 32, n64 = P / 64;
  const long t32 = n32 * (n32 + 1) / 2, t64 = n64 * (n64 + 1) / 2;
  // Small tiles while a compute unit gets one at most; then 64 x 64 tiles, k in two halves while a compute unit gets one of those.
  // us per product: eight images of order 384 30 on small tiles (2.4 a unit), 13 on wide ones with k in halves.
  constexpr long kUnits = 256;
  const int form = B * t32 <= kUnits && t32 <= kUnits / 4 ? 0 : B * t64 <= kUnits ? 1 : 2;     // t32: see the eighth below
  const size_t lds = (form == 1 ? 8 : 4) * ST * STP * sizeof(double);
  static PerDeviceInt raised, cache[3];
  auto kern = form == 0 ? sign_kernel<false, 1> : form == 1 ? sign_kernel<true, 2> : sign_kernel<true, 1>;
  hipError_t e;
  if (form == 1 && (e = ensure_dynamic_lds(raised, (const void*)kern, lds)) != hipSuccess) return e;
  int capacity = 0;
  if ((e = resident_workgroups(cache[form], kern, form == 1 ? 512 : 256, lds, &capacity)) != hipSuccess) return e;
  // An image of more tiles than its workgroups deals them out.  Its workgroups are an eighth of those the device holds at
  // most, so that the partial images of eight concurrent calls never hold all of it while they wait for the rest of theirs.
  const long most = capacity / 8, tiles = form ? t64 : t32;
  const long W = tiles < most ? tiles : most;
  if (W < 1) return hipErrorInvalidValue;
  const long stride = (long)P * P;
  const dim3 sg((unsigned)(B + B * (P / 16)));
  // The small kernel, whose workgroups load two rows of 16 x P each past the L2s: while that is 28 MB a product.  us per call of
  // covspec_select, sign_kernel / small, by images: order 64 40 228 / 200, 85 246 / 233; order 128 12 259 / 221, 20 277 / 250, 23 282 / 269, 24 283 / 275;
  // order 192 5 531 / 487, 7 556 / 517, 8 558 / 531, 9 603 / 586, 10 612 / 609, 12 656 / 699; order 256 1 679 / 599, 3 757 / 711, 4 772 / 745, 5 850 / 835, 6 873 /
  // 891.  (The line was drawn before the pause in its fetches, which moved the meeting points to 40 MB.)  And an image's workgroups, a tile
  // each, have to be as few as above.
  const long n16 = P / 16, t16 = n16 * (n16 + 1) / 2;
  bool small = form == 0 && P <= 64 * kSmallBlocks && B * t16 * 2 * 16 * P * 8 <= 28000000;
  static_assert(kSmallBlocks == 4, "");
  const auto sk = n64 == 1 ? sign_small_kernel<1> : n64 == 2 ? sign_small_kernel<2> : n64 == 3 ? sign_small_kernel<3> : sign_small_kernel<4>;
  if (small) {
    static PerDeviceInt resident[kSmallBlocks];
    int held = 0;
    if ((e = resident_workgroups(resident[n64 - 1], sk, 256, 0, &held)) != hipSuccess) return e;
    small = t16 <= held / 8;
  }
  const bool w64 = ordered || P == 64;
  auto ck = w64 ? cut_kernel<64> : cut_kernel<SN>;
  // A wave per SIMD; an image's workgroups are an eighth of what the device holds at most, as above.  Eight windows of 64: 47 us by
  // split_kernel, 48 with half the points and 64 with two waves a SIMD.
  const int trials = w64 ? kTrials : kTrials / 2;
  const size_t window = w64 ? 64 * 65 * 8 : SN * (SN + 1) * 8;
  bool count = B <= (w64 ? kCutImages / 2 : kCutImages);
  if (count) {
    static PerDeviceInt grown[2], room[2];
    int held = 0;
    if ((e = ensure_dynamic_lds(grown[w64], (const void*)ck, window)) != hipSuccess) return e;
    if ((e = resident_workgroups(room[w64], ck, 256, window, &held)) != hipSuccess) return e;
    count = trials / 4 <= held / 8;
  }
  if (count) {
    CutArea* area = (CutArea*)((char*)scratch + split_base_bytes(B, P));
    const size_t cut_lds = window > (size_t)P * 8 ? window : (size_t)P * 8;
    const dim3 cg((unsigned)(B * (trials / 4) + B * (P / 16)));
    hipLaunchKernelGGL(ck, cg, dim3(256), cut_lds, st, H, P, stride, B, r, ordered, trials, off, link, ctl, area, epoch, skip, again, small ? X0 : nullptr,
                       X1, Y, barrier_limit_ticks());
    if (again) hipLaunchKernelGGL(split_kernel, dim3((unsigned)B), dim3(256), 0, st, H, P, stride, B, r, false, off, link, ctl, skip, again, true, X0, X1, Y);
  } else {
    hipLaunchKernelGGL(split_kernel, sg, dim3(256), 0, st, H, P, stride, B, r, !ordered, off, link, ctl, skip, again, false, small ? X0 : nullptr, X1, Y);
  }
  if (small) {
    hipLaunchKernelGGL(sk, dim3((unsigned)(B * t16)), dim3(256), 0, st, H, X0, Y, X1, P, r, (const double*)off, (const double*)link,
                       ordered, (int)t16, ctl, barrier_limit_ticks());
    return hipGetLastError();
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(B * W)), dim3(form == 1 ? 512 : 256), lds, st, H, X0, Y, X1, P, r, (const double*)off, (const double*)link,
                     ordered, (int)W, ctl, barrier_limit_ticks());
  return hipGetLastError();
}

hipError_t launch_split_finish(const double* H, const double* Pi, const double* rnorm, int rparts, const double* cpart, int cparts, int B,
                               int P, int n, int nP, int r, double tol, const void* scratch, const int* slow, int* ok, int pass_no, float* c,
                               const NextPass& next, hipStream_t st) {
  hipLaunchKernelGGL(split_finish_kernel, dim3(B), dim3(1024), 0, st, H, Pi, rnorm, rparts, cpart, cparts, P, n, nP, r, tol,
                     (const SplitCtl*)scratch, slow, ok, pass_no, c, next);
  return hipGetLastError();
}

// A matrix without a usable gap at the cut (fewer distinct tokens than the rank) pays for the attempt in front of its full solve:
// 100 and 120 rows, all copies of ten, 2.94 -> 3.06 ms; with a gap the split takes 0.25 ms where that takes 2.7.
bool split_direct(int nP) { return nP <= SN; }

hipError_t launch_direct_energy(const double* G, const double* Pi, int B, int n, int nP, int r, const void* scratch, int* done, float* c,
                                hipStream_t st) {
  hipLaunchKernelGGL(direct_energy_kernel, dim3((n + 3) / 4, B), dim3(256), 0, st, G, Pi, n, nP, r, (const SplitCtl*)scratch, done, c);
  return hipGetLastError();
}

}  // namespace covspec
