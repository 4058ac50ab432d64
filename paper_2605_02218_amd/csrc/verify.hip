// Speculative verification over the vocabulary (paper Sec. II-A: softmax of the draft and target logits,
// acceptance probability of each drafted token, residual distribution after the first rejection).
//
// Per sequence s and drafted position tau the two logit rows z_t, z_d [V] are read ONCE by the statistics
// pass (reference and sum of exponentials of both, fp32 exponentials, partial results per chunk so that a
// few rows still fill the device); the acceptance pass combines them in fp64, evaluates
// alpha = min(1, p_t(y)/p_d(y)) at the drafted token, finds the first rejection and notes that row's
// statistics; only that one row per sequence is read again, in fp64: once for the exact sums and the chunk
// masses of max(p_t - p_d, 0), then, inside the one chunk that holds u_res * (total residual mass), for the
// inverse-CDF search of the correction.  Everything is HBM-bound streaming except the fp64 exponentials of the
// residual pass (2 per word, one row per sequence).
// For a few sequences what follows the statistics is one launch (verify_few_kernel): a workgroup per chunk of the rejected row, each of
// which works out the acceptance for itself, the last one of a sequence draws.  A chain of four launches is bound by the launches
// there; beyond, the acceptance is repeated in more workgroups than the device holds at once and the draws come at the end of the longest
// launch (few_sequences).  One sequence of 5 positions and 32000 words, us: four launches 22.8, two 16.5.
#include "common.h"
#include "kernels.h"
#include "vocab.h"

namespace covspec {

namespace {

constexpr int VT = 256;            // threads of the statistics pass
constexpr int AW = 8;              // waves of the acceptance kernel
constexpr int ST = 1024;           // threads of the sampling kernel
constexpr int FT = 512;            // of the kernel for few sequences
// Sequences that kernel is taken for, by the workgroups it makes of them (a chunk of a rejected row each).  The acceptance is worked out in each
// of them, so the line lies the lower the more chunks a row has.  Device time of the two launches over that of the four, 2 to 64 positions:
// 60 to 64 chunks 0.90 to 1.01 with three sequences, 0.95 to 1.05 with four, 0.98 to 1.21 with eight; 32 chunks 0.66 to 0.99 with six, 0.91 to
// 1.04 with eight; 16 chunks 0.87 to 0.99 with twelve, 0.90 to 1.06 with sixteen; 8 chunks 0.90 to 0.96 with 32, 0.94 to 1.05 with 64; four
// 0.93 to 1.02 with 128, one 0.83 to 1.01 with 512; a single position 0.81 to 1.05, median 0.91, up to 512 workgroups (8 to 151936 words,
// bf16).
inline bool few_sequences(long S, int L, int chunks) { return S * chunks <= (L == 1 || chunks <= 4 ? 512 : chunks <= 8 ? 256 : 192); }

// stats[(row * chunks + c) * 4 + {0,1,2,3}] = ref_t, sum_t, ref_d, sum_d (base-2 domain) over words [c*clen, min(V, (c+1)*clen))
template <int DT>
__global__ __launch_bounds__(VT) void verify_stats_kernel(const void* __restrict__ zt, const void* __restrict__ zd, int V, int clen,
                                                          int chunks, int L, double* __restrict__ stats, int* __restrict__ done) {
  constexpr int N = LogitVec<DT>::N;
  __shared__ double red[2][VT / 64][2];
  const long row = blockIdx.y;
  const int c = blockIdx.x;
  const int w0 = c * clen, w1 = min(V, w0 + clen);
  const long base = row * (long)V;
  if (c == 0 && threadIdx.x == 0 && row % L == 0) done[row / L] = 0;      // for the residual pass
  float mt = -INFINITY, st = 0.f, md = -INFINITY, sd = 0.f;
  // V, clen % N == 0: whole vectors only.  (Two vectors per trip with all loads issued first, and twice the
  // workgroups, both measured slower: the pass runs at the rate the memory system gives one resident round.)
  for (int w = w0 + threadIdx.x * N; w < w1; w += VT * N) {
    float a[N], b[N];
    LogitVec<DT>::load(zt, base + w, a);
    LogitVec<DT>::load(zd, base + w, b);
    online_add<N>(mt, st, a);
    online_add<N>(md, sd, b);
  }
  double mm, ss;
  block_combine<VT / 64>(mt, st, red[0], mm, ss);
  if (threadIdx.x == 0) { stats[(row * chunks + c) * 4] = mm; stats[(row * chunks + c) * 4 + 1] = ss; }
  block_combine<VT / 64>(md, sd, red[1], mm, ss);
  if (threadIdx.x == 0) { stats[(row * chunks + c) * 4 + 2] = mm; stats[(row * chunks + c) * 4 + 3] = ss; }
}

// The acceptance of sequence s, by the whole workgroup; `group` lanes (the smallest power of two that holds a row's chunks, at most
// 64) take a position, a wave as many positions at once as it has groups: row statistics from the chunk partials (one exponential
// per lane against the largest reference, one sum), alpha at the drafted token.  Returns the first rejected position or L (L <= 64);
// sh[t * 3 + {0,1}] = the references of row t brought back to the natural domain, i.e. its maximum logits to within rounding: the
// shift the fp64 passes below use (any value near the maximum serves, as long as every pass uses the same), [2] = the ratio of
// the two streaming sums.
// With one lane per position that folds the chunks one by one, two fp64 exponentials each, one sequence of 5 positions in 64 chunks
// took 11.5 us; now 3.4.  With a wave per position whatever the number of chunks, sixteen sequences of 64 positions in one chunk took 20 us.
template <int DT, int T>
__device__ __forceinline__ int accept(const void* __restrict__ zt, const void* __restrict__ zd, const int32_t* __restrict__ tok,
                                      const float* __restrict__ u_acc, int s, int L, int V, int chunks, int group,
                                      const double* __restrict__ stats, float* __restrict__ alpha_out, bool write, double* sh, int* sh_rej) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = lane & (group - 1), groups = 64 / group;
  for (int t0 = wv * groups; t0 < L; t0 += T / 64 * groups) {      // uniform in a wave: every lane takes part in the exchanges
    const int t = t0 + lane / group;
    const long row = (long)s * L + (t < L ? t : L - 1);
    int y = tok[row];
    y = y < 0 ? 0 : (y >= V ? V - 1 : y);     // never index outside the row
    const double xt = LogitVec<DT>::at(zt, row * V + y), xd = LogitVec<DT>::at(zd, row * V + y);
    double m[2], sum[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double mc = -INFINITY, sc = 0.0;
      if (c < chunks) {
        mc = stats[(row * chunks + c) * 4 + 2 * q];
        sc = stats[(row * chunks + c) * 4 + 2 * q + 1];
      }
      const bool has = sc > 0.0;              // a chunk of masked words has no sum
      double mm = has ? mc : -INFINITY;
      for (int o = group >> 1; o > 0; o >>= 1) mm = fmax(mm, __shfl_xor(mm, o, 64));
      m[q] = mm == -INFINITY ? 0.0 : mm;
      sum[q] = has ? sc * exp2(mc - m[q]) : 0.0;
      for (int o = group >> 1; o > 0; o >>= 1) sum[q] += __shfl_xor(sum[q], o, 64);
    }
    const double pt = exp2(xt * (double)kLog2e - m[0]) / sum[0];
    const double pd = exp2(xd * (double)kLog2e - m[1]) / sum[1];
    const double a = pd > 0.0 ? fmin(1.0, pt / pd) : 1.0;
    const float af = (float)a;
    if (c == 0 && t < L) {
      if (write && alpha_out) alpha_out[row] = af;
      sh_rej[t] = !(u_acc[row] < af) ? 1 : 0;
      sh[t * 3] = m[0] / (double)kLog2e;
      sh[t * 3 + 1] = m[1] / (double)kLog2e;
      // estimate of (sum_w exp(z_t - shift_t)) / (sum_w exp(z_d - shift_d)), good to the ~1e-6 of the streaming sums
      sh[t * 3 + 2] = sum[0] / sum[1];
    }
  }
  __syncthreads();
  const unsigned long long mask = __ballot(lane < L && sh_rej[lane < L ? lane : 0] != 0);
  return mask != 0ull ? __ffsll((long long)mask) - 1 : L;
}

// One workgroup per sequence.  rowmax[s * 4 + {0,1,2}] = what `accept` leaves of the rejected row; untouched when nothing is rejected.
template <int DT>
__global__ __launch_bounds__(64 * AW) void verify_accept_kernel(const void* __restrict__ zt, const void* __restrict__ zd,
                                                                const int32_t* __restrict__ tok, const float* __restrict__ u_acc, int L,
                                                                int V, int chunks, int group, const double* __restrict__ stats,
                                                                int32_t* __restrict__ n_acc, float* __restrict__ alpha_out,
                                                                double* __restrict__ rowmax) {
  __shared__ double sh[64 * 3];
  __shared__ int sh_rej[64];
  const int s = blockIdx.x;
  const int first = accept<DT, 64 * AW>(zt, zd, tok, u_acc, s, L, V, chunks, group, stats, alpha_out, true, sh, sh_rej);
  if (first < L && threadIdx.x < 3) rowmax[s * 4 + threadIdx.x] = sh[first * 3 + threadIdx.x];
  if (threadIdx.x == 0) n_acc[s] = first;
}

// e^x for the fp64 passes, x <= 0 to within rounding: x = n ln 2 + f with |f| <= ln 2 / 2 (Cody and Waite's two-part reduction),
// the Taylor polynomial of degree 13 (remainder below 5e-18) and a scaling by 2^n.  Beyond -800 the result is 0, a NaN stays one.  About 20 fp64 instructions.
__device__ __forceinline__ double exp_shifted(double x) {
  x = x < -800.0 ? -800.0 : x;
  const double n = rint(x * 1.4426950408889634074);
  // ln 2 in two parts, the first with trailing zeros so that n times it is exact
  double f = fma(n, -0x1.62e42feep-1, x);
  f = fma(n, -0x1.a39ef35793c76p-33, f);
  const double f2 = f * f;
  // even and odd halves side by side
  double e = fma(f2, 1.0 / 479001600.0, 1.0 / 3628800.0), o = fma(f2, 1.0 / 6227020800.0, 1.0 / 39916800.0);
  e = fma(f2, e, 1.0 / 40320.0);
  o = fma(f2, o, 1.0 / 362880.0);
  e = fma(f2, e, 1.0 / 720.0);
  o = fma(f2, o, 1.0 / 5040.0);
  e = fma(f2, e, 1.0 / 24.0);
  o = fma(f2, o, 1.0 / 120.0);
  e = fma(f2, e, 0.5);
  o = fma(f2, o, 1.0 / 6.0);
  e = fma(f2, e, 1.0);
  o = fma(f2, o, 1.0);
  return ldexp(fma(f, o, e), (int)n);
}

// The one fp64 pass over the rejected row of each sequence, per chunk: exact sums S_t, S_d of the exponentials
// (the residual is a difference of the two distributions, and the fp32 sums of the first pass, good to ~1e-6,
// would move its cumulative sums by more than a flat residual's single words) and, in the same pass, the
// chunk's residual mass (sixteen-byte loads, exp_shifted: 27 -> 24 us for 64 rows of 151936 words).  max(p_t - p_d, 0) = max(e_t - kappa e_d, 0) / S_t with kappa = S_t / S_d, which is not
// known before the pass ends; but the mass is A - kappa B with A, B the sums of e_t, e_d over the words where
// e_t > kappa e_d, and an error delta in the kappa that picks those words changes the mass only to second
// order (a word that changes sides carries a residual below delta e_d).  So the words are picked with the
// streaming estimate (delta ~ 1e-6, mass error ~ 1e-12 relative) and A, B are combined with the exact kappa
// afterwards.  rowsum[(s * rchunks + c) * 4 + {0,1,2,3}] = S_t, S_d, A, B of the chunk.
template <int DT, int T>
__device__ __forceinline__ void residual_masses(const void* __restrict__ zt, const void* __restrict__ zd, long base, int w0, int w1, double mt, double md,
                                                double kap, double* sums) {
  __shared__ double red[4][T / 64];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  constexpr int N = LogitVec<DT>::N;
  auto add = [&](double xt, double xd) {
    const double et = exp_shifted(xt - mt), ed = exp_shifted(xd - md);
    acc[0] += et;
    acc[1] += ed;
    const bool more = et > kap * ed;                             // equal rows: kap == 1 and et == ed exactly, nothing is picked
    acc[2] += more ? et : 0.0;
    acc[3] += more ? ed : 0.0;
  };
  if (w1 - w0 <= T) {
    // a word per thread: eight of them one after the other in an eighth of the threads take 4.2 us where this takes 3.3
    const int w = w0 + threadIdx.x;
    if (w < w1) add(LogitVec<DT>::at(zt, base + w), LogitVec<DT>::at(zd, base + w));
  } else {
    for (int w = w0 + threadIdx.x * N; w < w1; w += T * N) {     // V, rlen % N == 0: whole vectors only
      float a[N], c[N];
      LogitVec<DT>::load(zt, base + w, a);
      LogitVec<DT>::load(zd, base + w, c);
#pragma unroll
      for (int e = 0; e < N; ++e) add((double)a[e], (double)c[e]);
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = wave_sum(acc[q]);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) red[q][wv] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double tot = 0.0;
    for (int k = 0; k < T / 64; ++k) tot += red[threadIdx.x][k];
    store_through(sums + threadIdx.x, tot);
  }
}

template <int DT>
__global__ __launch_bounds__(VT) void verify_rowpass64_kernel(const void* __restrict__ zt, const void* __restrict__ zd, int L, int V,
                                                              int rlen, int rchunks, const int32_t* __restrict__ n_acc,
                                                              const double* __restrict__ rowmax, double* __restrict__ rowsum) {
  const int s = blockIdx.y, c = blockIdx.x;
  const int t = n_acc[s];
  if (t >= L) return;
  residual_masses<DT, VT>(zt, zd, ((long)s * L + t) * V, c * rlen, min(V, (c + 1) * rlen), rowmax[s * 4], rowmax[s * 4 + 1], rowmax[s * 4 + 2],
                          rowsum + ((long)s * rchunks + c) * 4);
}

__device__ __forceinline__ double residual_of(double zt, double zd, double mt, double ist, double md, double isd) {
  // each product rounded on its own: contracted into a fused multiply-add the difference of two EQUAL
  // probabilities would come out as rounding noise instead of zero
#pragma clang fp contract(off)
  const double a = exp_shifted(zt - mt) * ist;
  const double b = exp_shifted(zd - md) * isd;
  const double d = a - b;
  return d > 0.0 ? d : 0.0;
}

// wave 0 of a workgroup (all 64 lanes): the row's 1/sum_t and 1/sum_d from the chunk sums, into LDS.  rchunks <= 64: lane c holds
// chunk c, butterfly sums.  Returns the residual mass of chunk `lane`, A / S_t - B / S_d (0 for lanes beyond the chunks).
__device__ __forceinline__ double combine_rowstat(const double* rs, int rchunks, double* sh2) {
  const int lane = threadIdx.x & 63;
  rs += lane * 4;
  const double st_c = lane < rchunks ? rs[0] : 0.0, sd_c = lane < rchunks ? rs[1] : 0.0;
  const double a_c = lane < rchunks ? rs[2] : 0.0, b_c = lane < rchunks ? rs[3] : 0.0;
  const double st = wave_sum(st_c), sd = wave_sum(sd_c);
  const double ist = 1.0 / st, isd = 1.0 / sd;
  if (lane == 0) { sh2[0] = ist; sh2[1] = isd; }
  double mass;
  {
#pragma clang fp contract(off)
    const double x = a_c * ist, y = b_c * isd;
    mass = x - y;
  }
  return mass > 0.0 ? mass : 0.0;
}

// The correction of sequence s, by one workgroup: inverse CDF of the residual in vocabulary order.  A thread sums `per`
// neighbouring words of the chunk; the words of the one thread whose sum passes the target are evaluated once more, one by a lane.
// (With all threads walking their words again behind their prefixes, 256 of them, a chunk of 4864 words took 41 us in the kernel for few
// sequences; so, with 512, 18.)
template <int DT, int T>
__device__ __forceinline__ void sample(const void* __restrict__ zt, const void* __restrict__ zd, int s, long base, int V, int clen, int chunks,
                                       double mt, double md, const double* rowsum, float u, int32_t* __restrict__ corr) {
  constexpr int N = LogitVec<DT>::N;
  __shared__ double wsum[T / 64], before[T];
  __shared__ double sh_prefix, sh_target, sh2[2];
  __shared__ int sh_chunk, sh_cross, sh_last;
  __shared__ unsigned long long sh_best;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // lane c of a wave holds chunk c's residual mass; inclusive scan in lane order, total in lane 63
  auto scan = [&](double v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double w = __shfl_up(v, o, 64);
      if (lane >= o) v += w;
    }
    return v;
  };
  if (tid < 64) {
    const double pc = combine_rowstat(rowsum, chunks, sh2), inc = scan(pc);
    const double R = __shfl(inc, 63, 64);
    const double target = (double)u * R;
    // the first chunk whose cumulative mass passes the target; if rounding leaves the target at the total,
    // the last chunk with any mass
    const unsigned long long over = __ballot(pc > 0.0 && inc > target);
    const unsigned long long mass = __ballot(pc > 0.0);
    int cs = -1;
    if (R > 0.0) cs = over ? __ffsll((long long)over) - 1 : 63 - __clzll((long long)mass);
    if (lane == (cs < 0 ? 0 : cs)) {
      sh_chunk = cs; sh_prefix = inc - pc; sh_target = target; sh_cross = T; sh_last = -1; sh_best = 0ull;
    }
  }
  __syncthreads();
  const int cs = sh_chunk;
  if (cs < 0) {
    // no residual mass (p_t == p_d): argmax p_t, lowest index on ties
    unsigned long long best = 0ull;
    for (int w = tid * N; w < V; w += T * N) {                // V % N == 0: whole vectors only
      float a[N];
      LogitVec<DT>::load(zt, base + w, a);                     // logits are stored in at most fp32: exact
#pragma unroll
      for (int e = 0; e < N; ++e) {
        const unsigned long long key = ((unsigned long long)float_order_key(a[e]) << 32) | (0xFFFFFFFFu - (uint32_t)(w + e));
        best = key > best ? key : best;
      }
    }
    best = wave_max(best);
    if (lane == 0) atomicMax(&sh_best, best);
    __syncthreads();
    if (tid == 0) corr[s] = (int)(0xFFFFFFFFu - (uint32_t)(sh_best & 0xFFFFFFFFull));
    return;
  }
  const double ist = sh2[0], isd = sh2[1];
  const int w0 = cs * clen, w1 = min(V, w0 + clen), n = w1 - w0;
  const bool vectors = n > 2 * T;                             // one or two words per thread are spread over all of them
  const int per = vectors ? (n + T * N - 1) / (T * N) * N : (n + T - 1) / T;
  const int a0 = min(w1, w0 + tid * per), a1 = min(w1, a0 + per);
  auto residual_at = [&](int w) { return residual_of(LogitVec<DT>::at(zt, base + w), LogitVec<DT>::at(zd, base + w), mt, ist, md, isd); };
  double mine = 0.0, first = 0.0, second = 0.0;
  if (vectors) {
    for (int w = a0; w < a1; w += N) {                         // w0, w1 % N == 0: whole vectors only
      float a[N], c[N];
      LogitVec<DT>::load(zt, base + w, a);
      LogitVec<DT>::load(zd, base + w, c);
#pragma unroll
      for (int e = 0; e < N; ++e) mine += residual_of((double)a[e], (double)c[e], mt, ist, md, isd);
    }
  } else {
    if (a0 < a1) first = residual_at(a0);
    if (a0 + 1 < a1) second = residual_at(a0 + 1);
    mine = first + second;
  }
  // exclusive prefix over the threads (fp64): wave scan, then the wave totals
  const double inc = scan(mine);
  if (lane == 63) wsum[wv] = inc;
  __syncthreads();
  double run = sh_prefix;
  for (int k = 0; k < wv; ++k) run += wsum[k];
  run += inc - mine;
  before[tid] = run;
  const double target = sh_target;
  if (mine > 0.0) {
    if (run + mine > target) atomicMin(&sh_cross, tid);
    atomicMax(&sh_last, tid);
  }
  __syncthreads();
  // the first word of the crossing thread at which the running sum passes the target.  If rounding leaves the target just past
  // the chunk or the thread's words, the last word with any mass before it
  const int owner = sh_cross < T ? sh_cross : sh_last;
  if (!vectors) {
    if (tid == (owner < 0 ? 0 : owner))
      corr[s] = owner < 0 ? w1 - 1 : second > 0.0 && !(sh_cross < T && first > 0.0 && run + first > target) ? a0 + 1 : a0;
    return;
  }
  if (wv != 0) return;
  int hit = -1, last = w1 - 1;
  if (owner >= 0) {
    const int b0 = w0 + owner * per, b1 = min(w1, b0 + per);
    double sum = before[owner];
    for (int w = b0; w < b1 && hit < 0; w += 64) {
      const double r = w + lane < b1 ? residual_at(w + lane) : 0.0;
      const double upto = sum + scan(r);
      const unsigned long long over = __ballot(r > 0.0 && upto > target), mass = __ballot(r > 0.0);
      if (over) hit = w + __ffsll((long long)over) - 1;
      if (mass) last = w + 63 - __clzll((long long)mass);
      sum = __shfl(upto, 63, 64);
    }
  }
  if (lane == 0) corr[s] = hit >= 0 ? hit : last;
}

// One workgroup per sequence; 64 registers, so that a compute unit holds two of them.
template <int DT>
__global__ __launch_bounds__(ST, 8) void verify_sample_kernel(const void* __restrict__ zt, const void* __restrict__ zd, int L, int V,
                                                              int rlen, int rchunks, const int32_t* __restrict__ n_acc,
                                                              const double* __restrict__ rowmax, const double* __restrict__ rowsum,
                                                              const float* __restrict__ u_res, int32_t* __restrict__ corr) {
  const int s = blockIdx.x, t = n_acc[s];
  if (t >= L) { if (threadIdx.x == 0) corr[s] = -1; return; }
  sample<DT, ST>(zt, zd, s, ((long)s * L + t) * V, V, rlen, rchunks, rowmax[s * 4], rowmax[s * 4 + 1], rowsum + (long)s * rchunks * 4, u_res[s], corr);
}

// All of it for a few sequences, grid (rchunks, S).  The workgroup that finds the others of its sequence done draws the
// correction; nobody waits.
template <int DT>
__global__ __launch_bounds__(FT, 4) void verify_few_kernel(const void* __restrict__ zt, const void* __restrict__ zd, const int32_t* __restrict__ tok,
                                                           const float* __restrict__ u_acc, const float* __restrict__ u_res, int L, int V,
                                                           int chunks, int group, const double* __restrict__ stats, int rlen, int rchunks,
                                                           double* rowsum, int* done, int32_t* __restrict__ n_acc,
                                                           float* __restrict__ alpha_out, int32_t* __restrict__ corr) {
  __shared__ double sh[64 * 3];
  __shared__ int sh_rej[64], sh_last;
  const int s = blockIdx.y, c = blockIdx.x;
  const int t = accept<DT, FT>(zt, zd, tok, u_acc, s, L, V, chunks, group, stats, alpha_out, c == 0, sh, sh_rej);
  if (c == 0 && threadIdx.x == 0) {
    n_acc[s] = t;
    if (t >= L) corr[s] = -1;
  }
  if (t >= L) return;
  const long base = ((long)s * L + t) * V;
  const double mt = sh[t * 3], md = sh[t * 3 + 1];
  double* sums = rowsum + (long)s * rchunks * 4;
  residual_masses<DT, FT>(zt, zd, base, c * rlen, min(V, (c + 1) * rlen), mt, md, sh[t * 3 + 2], sums + 4 * c);
  if (threadIdx.x < 64) {
    __builtin_amdgcn_s_waitcnt(0x0070);              // this wave's sums are where the others see them before the count says so
    if (threadIdx.x == 0) {
      const int before = __hip_atomic_fetch_add(done + s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (before == rchunks - 1) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      sh_last = before == rchunks - 1 ? 1 : 0;
    }
  }
  __syncthreads();
  if (sh_last) sample<DT, FT>(zt, zd, s, base, V, rlen, rchunks, mt, md, sums, u_res[s], corr);
}

}  // namespace

void verify_plan(int S, int L, int V, int dtype, int* clen, int* chunks) {
  // chunks per row so that even a few rows give the streaming kernel ~1024 workgroups; chunk length a
  // multiple of what one pass of the workgroup covers
  const int vec = dtype == DT_F32 ? 4 : 8;
  const int step = VT * vec;
  long rows = (long)S * L;
  int want = (int)((1024 + rows - 1) / rows);
  if (want < 1) want = 1;
  if (want > 64) want = 64;
  int len = (V + want - 1) / want;
  len = (len + step - 1) / step * step;
  *clen = len;
  *chunks = (V + len - 1) / len;
}

// the fp64 passes read one row per sequence: their own, finer split (~2048 workgroups, at most 64 chunks a row)
static void residual_plan(int S, int V, int* rlen, int* rchunks) {
  int want = (2048 + S - 1) / S;
  if (want < 1) want = 1;
  if (want > 64) want = 64;
  int len = (V + want - 1) / want;
  len = (len + VT - 1) / VT * VT;
  *rlen = len;
  *rchunks = (V + len - 1) / len;
}

size_t verify_workspace_bytes(int S, int L, int V, int dtype) {
  int clen, chunks, rlen, rchunks;
  verify_plan(S, L, V, dtype, &clen, &chunks);
  residual_plan(S, V, &rlen, &rchunks);
  return ((size_t)S * L * chunks * 4 + (size_t)S * 4 + (size_t)S * rchunks * 4) * sizeof(double) + 512;
}

template <int DT>
static hipError_t launch_verify_t(const void* zt, const void* zd, const int32_t* tok, const float* u_acc, const float* u_res, int S,
                                  int L, int V, int32_t* n_acc, int32_t* corr, float* alpha, void* ws, hipStream_t st) {
  int clen, chunks, rlen, rchunks;
  verify_plan(S, L, V, DT, &clen, &chunks);
  residual_plan(S, V, &rlen, &rchunks);
  double* stats = (double*)ws;                               // [S*L][chunks][4]
  double* rowmax = stats + (size_t)S * L * chunks * 4;       // [S][4]; few sequences: [S] workgroups that have their sums in memory
  double* rowsum = rowmax + (size_t)S * 4;                   // [S][rchunks][4]
  int* done = (int*)rowmax;
  const double *cstats = stats, *crowmax = rowmax, *crowsum = rowsum;
  const int32_t* cn = n_acc;
  int group = 1;
  while (group < chunks) group *= 2;                         // chunks <= 64
  hipLaunchKernelGGL((verify_stats_kernel<DT>), dim3(chunks, S * L), dim3(VT), 0, st, zt, zd, V, clen, chunks, L, stats, done);
  if (few_sequences(S, L, rchunks)) {
    hipLaunchKernelGGL((verify_few_kernel<DT>), dim3(rchunks, S), dim3(FT), 0, st, zt, zd, tok, u_acc, u_res, L, V, chunks, group, cstats, rlen,
                       rchunks, rowsum, done, n_acc, alpha, corr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((verify_accept_kernel<DT>), dim3(S), dim3(64 * AW), 0, st, zt, zd, tok, u_acc, L, V, chunks, group, cstats, n_acc, alpha, rowmax);
  hipLaunchKernelGGL((verify_rowpass64_kernel<DT>), dim3(rchunks, S), dim3(VT), 0, st, zt, zd, L, V, rlen, rchunks, cn, crowmax, rowsum);
  hipLaunchKernelGGL((verify_sample_kernel<DT>), dim3(S), dim3(ST), 0, st, zt, zd, L, V, rlen, rchunks, cn, crowmax, crowsum, u_res, corr);
  return hipGetLastError();
}

hipError_t launch_verify(const void* zt, const void* zd, const int32_t* tok, const float* u_acc, const float* u_res, int S, int L,
                         int V, int dtype, int32_t* n_acc, int32_t* corr, float* alpha, void* ws, hipStream_t st) {
  if (S < 1 || L < 1 || L > 64 || V < 2 || (long)S * L > 65535) return hipErrorInvalidValue;
  if (dtype == DT_BF16) return launch_verify_t<DT_BF16>(zt, zd, tok, u_acc, u_res, S, L, V, n_acc, corr, alpha, ws, st);
  if (dtype == DT_F16) return launch_verify_t<DT_F16>(zt, zd, tok, u_acc, u_res, S, L, V, n_acc, corr, alpha, ws, st);
  return launch_verify_t<DT_F32>(zt, zd, tok, u_acc, u_res, S, L, V, n_acc, corr, alpha, ws, st);
}

}  // namespace covspec
