// HBM-bound and small per-token kernels of the token-selection path:
// activity score, row norms, format conversion and splitting, the cosine-max
// and softmax epilogues, min-max fusion, gather.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace covspec {

namespace {

// ---------------------------------------------------------------- 16-byte element loads
template <int DT> struct Vec;
template <> struct Vec<DT_BF16> {
  static constexpr int N = 8;
  __device__ static __forceinline__ void load(const void* base, long elem, float (&v)[8]) {
    u32x4_t r = *(const u32x4_t*)((const bf16_t*)base + elem);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = bf16lo_to_f32(r[i]); v[2 * i + 1] = bf16hi_to_f32(r[i]); }
  }
  __device__ static __forceinline__ float load1(const void* base, long elem) { return bf16_to_f32(((const bf16_t*)base)[elem]); }
};
template <> struct Vec<DT_F32> {
  static constexpr int N = 4;
  __device__ static __forceinline__ void load(const void* base, long elem, float (&v)[4]) {
    f32x4_t r = *(const f32x4_t*)((const float*)base + elem);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = r[i];
  }
  __device__ static __forceinline__ float load1(const void* base, long elem) { return ((const float*)base)[elem]; }
};

// ---------------------------------------------------------------- activity (paper Sec. III-A.2)
// One wave per token.  The wave walks the row in 16-byte-per-lane chunks and reads the K+1 slices of a
// chunk back to back, keeping the previous slice in registers, so every hidden element is read from
// HBM exactly once.  Squared differences accumulate in fp32 per (layer, lane) and are wave-reduced in a
// fixed order, so equal rows give bit-equal scores.  fp32 inputs accumulate in fp64, bf16 inputs in fp32
// (a difference of two bf16 values is exact in fp32).
template <int DT, int K, typename Acc>
__global__ __launch_bounds__(256) void activity_kernel(const void* __restrict__ hidden, float* __restrict__ s_act,
                                                        long tokens, int N, int d) {
  constexpr int V = Vec<DT>::N;
  const int lane = threadIdx.x & 63;
  const long token = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (token >= tokens) return;
  const long b = token / N, i = token - b * N;
  const long slice = (long)N * d;
  const long base = (b * (K + 1) * N + i) * (long)d;
  Acc acc[K];
#pragma unroll
  for (int l = 0; l < K; ++l) acc[l] = (Acc)0;
  for (int c = lane * V; c < d; c += 64 * V) {
    float prev[V], cur[V];
    Vec<DT>::load(hidden, base + c, prev);
#pragma unroll
    for (int l = 1; l <= K; ++l) {
      Vec<DT>::load(hidden, base + l * slice + c, cur);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const Acc df = (Acc)cur[e] - (Acc)prev[e];
        acc[l - 1] += df * df;
        prev[e] = cur[e];
      }
    }
  }
  double total = 0.0;
#pragma unroll
  for (int l = 0; l < K; ++l) total += sqrt((double)wave_sum(acc[l]));
  if (lane == 0) s_act[token] = (float)(total / K);
}

template <int DT>
hipError_t activity_dispatch(const void* hidden, float* s_act, long tokens, int N, int d, int K, hipStream_t st) {
  dim3 grid((unsigned)((tokens + 3) / 4)), block(256);
#define COVSPEC_ACT_CASE(KK) \
  case KK: hipLaunchKernelGGL((activity_kernel<DT, KK, typename std::conditional<DT == DT_F32, double, float>::type>), grid, block, 0, st, hidden, s_act, tokens, N, d); break;
  switch (K) {
    COVSPEC_ACT_CASE(1) COVSPEC_ACT_CASE(2) COVSPEC_ACT_CASE(3) COVSPEC_ACT_CASE(4)
    COVSPEC_ACT_CASE(5) COVSPEC_ACT_CASE(6) COVSPEC_ACT_CASE(7) COVSPEC_ACT_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef COVSPEC_ACT_CASE
  return hipGetLastError();
}

// ---------------------------------------------------------------- row norms
template <typename In> __device__ __forceinline__ double load_as_f64(const In* p, long i);
template <> __device__ __forceinline__ double load_as_f64<bf16_t>(const bf16_t* p, long i) { return (double)bf16_to_f32(p[i]); }
template <> __device__ __forceinline__ double load_as_f64<float>(const float* p, long i) { return (double)p[i]; }
template <> __device__ __forceinline__ double load_as_f64<double>(const double* p, long i) { return p[i]; }

// one wave per row; Out = float accumulates in fp32, Out = double in fp64
template <typename In, typename Out>
__global__ __launch_bounds__(256) void row_norm2_kernel(const In* __restrict__ x, Out* __restrict__ out, long rows, int d) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  Out acc = (Out)0;
  for (int c = lane; c < d; c += 64) {
    const Out v = (Out)load_as_f64<In>(x, row * d + c);
    acc += v * v;
  }
  acc = wave_sum(acc);
  if (lane == 0) out[row] = acc;
}

// ---------------------------------------------------------------- transpose
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ in0, T* __restrict__ out0, const T* __restrict__ in1, T* __restrict__ out1, int rows, int cols) {
  const T* __restrict__ in = blockIdx.z ? in1 : in0;
  T* __restrict__ out = blockIdx.z ? out1 : out0;
  __shared__ T tile[64][65];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  for (int r = ty; r < 64; r += 4)
    if (r0 + r < rows && c0 + tx < cols) tile[r][tx] = in[(long)(r0 + r) * cols + c0 + tx];
  __syncthreads();
  for (int c = ty; c < 64; c += 4)
    if (c0 + c < cols && r0 + tx < rows) out[(long)(c0 + c) * rows + r0 + tx] = tile[tx][c];
}

// The same in 16-byte pieces: a thread loads two pieces of a row into LDS and stores two pieces of a column from it.  64 x 64
// tiles of E-byte elements, rows and cols multiples of 16 / E, 16-byte aligned.  3584 x 3584 bf16: 27.5 us with an element per
// access, 11.4 here (51 MB).
template <typename T>
__global__ __launch_bounds__(256) void transpose16_kernel(const T* __restrict__ in0, T* __restrict__ out0, const T* __restrict__ in1, T* __restrict__ out1, int rows, int cols) {
  const T* __restrict__ in = blockIdx.z ? in1 : in0;
  T* __restrict__ out = blockIdx.z ? out1 : out0;
  constexpr int N = 16 / sizeof(T), PER = 64 / N;      // elements per piece, pieces per tile row
  __shared__ T tile[64][64 + 4 / sizeof(T)];           // a row is an odd number of banks
  typedef T piece_t __attribute__((ext_vector_type(N)));
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  for (int e = threadIdx.x; e < 64 * PER; e += 256) {
    const int r = e / PER, c = e % PER * N;
    if (r0 + r < rows && c0 + c < cols) {
      const piece_t v = *(const piece_t*)(in + (long)(r0 + r) * cols + c0 + c);
#pragma unroll
      for (int k = 0; k < N; ++k) tile[r][c + k] = v[k];
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * PER; e += 256) {
    const int c = e / PER, r = e % PER * N;
    if (c0 + c < cols && r0 + r < rows) {
      piece_t v;
#pragma unroll
      for (int k = 0; k < N; ++k) v[k] = tile[r + k][c];
      *(piece_t*)(out + (long)(c0 + c) * rows + r0 + r) = v;
    }
  }
}

// ---------------------------------------------------------------- conversion / splitting
template <typename In, typename Out>
__global__ void convert_kernel(const In* __restrict__ src, Out* __restrict__ dst, long n) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (Out)load_as_f64<In>(src, i);
}

__device__ __forceinline__ float sum_planes(const float* src, int planes, long plane_stride, long i) {
  float v = src[i];
  for (int p = 1; p < planes; ++p) v += src[p * plane_stride + i];
  return v;
}

// V elements of a row per thread (V = 4 when d % 4 == 0 and the planes and the output start on 16- / 8-byte boundaries:
// one 16-byte load per plane and one 8-byte store per output plane; else V = 1).  The sum over the planes is taken in
// plane order per element, the same in both widths.
template <int V>
__global__ __launch_bounds__(256) void sum_split3_kernel(const float* __restrict__ src, int planes, long plane_stride, long rows, int d,
                                                         long rpg, bf16_t* __restrict__ out) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * V;
  if (i >= rows * d) return;
  const long r = i / d;
  const int c = (int)(i - r * d);
  float v[V];
  if (V == 4) {
    const f32x4_t x = *(const f32x4_t*)(src + i);
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = x[e];
    for (int p = 1; p < planes; ++p) {
      const f32x4_t y = *(const f32x4_t*)(src + p * plane_stride + i);
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] += y[e];
    }
  } else {
    v[0] = sum_planes(src, planes, plane_stride, i);
  }
  bf16_t hi[V], mid[V], lo[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    hi[e] = f32_to_bf16_rne(v[e]);
    const float r1 = v[e] - bf16_to_f32(hi[e]);  // exact
    mid[e] = f32_to_bf16_rne(r1);
    const float r2 = r1 - bf16_to_f32(mid[e]);   // exact
    lo[e] = f32_to_bf16_rne(r2);
  }
  const long g = r / rpg, j = r - g * rpg;
  bf16_t* o0 = out + ((g * 3 + 0) * rpg + j) * d + c;
  bf16_t* o1 = out + ((g * 3 + 1) * rpg + j) * d + c;
  bf16_t* o2 = out + ((g * 3 + 2) * rpg + j) * d + c;
  if (V == 4) {
    typedef unsigned short u16x4_t __attribute__((ext_vector_type(4)));
    *(u16x4_t*)o0 = (u16x4_t){hi[0], hi[1], hi[2], hi[3]};
    *(u16x4_t*)o1 = (u16x4_t){mid[0], mid[1], mid[2], mid[3]};
    *(u16x4_t*)o2 = (u16x4_t){lo[0], lo[1], lo[2], lo[3]};
  } else {
    *o0 = hi[0];
    *o1 = mid[0];
    *o2 = lo[0];
  }
}

// What is left to do for a row of e(q): its squared length to norm2, summed by one wave in row_norm2_kernel's order (the other
// waves share the rest), and its three bf16 planes, as sum_split3_kernel writes them with one group, to eq3 (optional).  One
// workgroup per row; d % 4 == 0.
__global__ __launch_bounds__(256) void query_rows_kernel(const float* __restrict__ src, long rows, int d, bf16_t* __restrict__ eq3,
                                                         float* __restrict__ norm2) {
  const long r = blockIdx.x;
  const float* x = src + r * d;
  if (threadIdx.x < 64) {
    float acc = 0.f;
#pragma unroll 8
    for (int c = threadIdx.x; c < d; c += 64) acc = fmaf(x[c], x[c], acc);
    acc = wave_sum(acc);
    if (threadIdx.x == 0) norm2[r] = acc;
    return;
  }
  if (!eq3) return;
  for (int c = 4 * (threadIdx.x - 64); c < d; c += 768) {
    typedef unsigned short u16x4_t __attribute__((ext_vector_type(4)));
    const f32x4_t v = *(const f32x4_t*)(x + c);
    u16x4_t o[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[0][e] = f32_to_bf16_rne(v[e]);
      const float r1 = v[e] - bf16_to_f32(o[0][e]);  // exact
      o[1][e] = f32_to_bf16_rne(r1);
      o[2][e] = f32_to_bf16_rne(r1 - bf16_to_f32(o[1][e]));
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) *(u16x4_t*)(eq3 + (q * rows + r) * d + c) = o[q];
  }
}

// ---------------------------------------------------------------- cosine-max epilogue (paper Sec. III-A.1)
// s_query[token] = max_j dot_j / max(|e(v)| |e(q_j)|, 1e-30), dot_j = the sum of the logit planes of keyword j.  The
// scalar arithmetic is fp64 so that the only error left in the score is that of the fp32-accumulated contractions
// feeding it.  Four lanes per token, 64 tokens of one image per workgroup: the keywords' 1 / |e(q_j)| are formed once
// per workgroup (LDS) and a token's |e(v)| once, so that a keyword costs a token one multiplication
// (max_j dot_j / (|v| |q_j|) = (max_j dot_j / |q_j|) / |v|; a wave per token with a square root and a division per
// keyword was bound by those: 156 us for workload 5 where its 283 MB of logits are 50 us of HBM time).  Where the
// floor could bind (|v| |q_j| < 1e-30 for some keyword that is not a zero vector) the token takes the literal formula.
template <typename F>
__global__ __launch_bounds__(256) void cosine_max_kernel(const F* __restrict__ logits, int planes,
                                                          const F* __restrict__ vnorm2, int nparts,
                                                          const F* __restrict__ qnorm2, float* __restrict__ s_query,
                                                          int N, int T) {
  extern __shared__ double cm_lds[];    // [T] 1 / |e(q_j)| (0 for a zero vector), then the smallest non-zero |e(q_j)|
  double* rq = cm_lds;
  double* minq = cm_lds + T;
  const int tid = threadIdx.x, q = tid & 3;
  const int b = blockIdx.y;
  if (tid == 0) *minq = 1e300;
  __syncthreads();
  double mine = 1e300;
  for (int j = tid; j < T; j += 256) {
    const double sq = sqrt((double)qnorm2[(long)b * T + j]);
    rq[j] = sq > 0.0 ? 1.0 / sq : 0.0;
    if (sq > 0.0) mine = fmin(mine, sq);
  }
  mine = wave_min(mine);
  if ((tid & 63) == 0 && mine < 1e300) atomicMin((unsigned long long*)minq, (unsigned long long)__double_as_longlong(mine));   // positive doubles order like their bits
  __syncthreads();
  const double smallest = *minq;
  const int n = blockIdx.x * 64 + (tid >> 2);
  if (n >= N) return;      // whole quads leave together
  const long token = (long)b * N + n;
  double n2 = 0.0;
  for (int t = q; t < nparts; t += 4) n2 += (double)vnorm2[token * nparts + t];
  n2 += __shfl_xor(n2, 1, 64);
  n2 += __shfl_xor(n2, 2, 64);
  const double nv = sqrt(n2);
  const F* L = logits + token * (long)planes * T;
  double best = -INFINITY;
  if (nv * smallest >= 1e-30) {
    if (std::is_same<F, float>::value && (T & 3) == 0 && (((uintptr_t)logits) & 15) == 0) {
      for (int j0 = 4 * q; j0 < T; j0 += 16) {
        f32x4_t x = *(const f32x4_t*)((const float*)L + j0);
        double d0 = x[0], d1 = x[1], d2 = x[2], d3 = x[3];
        for (int s_ = 1; s_ < planes; ++s_) {
          x = *(const f32x4_t*)((const float*)L + (long)s_ * T + j0);
          d0 += x[0]; d1 += x[1]; d2 += x[2]; d3 += x[3];
        }
        best = fmax(best, fmax(fmax(d0 * rq[j0], d1 * rq[j0 + 1]), fmax(d2 * rq[j0 + 2], d3 * rq[j0 + 3])));
      }
    } else {
      for (int j = q; j < T; j += 4) {
        double dot = (double)L[j];
        for (int s_ = 1; s_ < planes; ++s_) dot += (double)L[(long)s_ * T + j];
        best = fmax(best, dot * rq[j]);
      }
    }
    best = best / nv;     // nv > 0 here
  } else {
    for (int j = q; j < T; j += 4) {
      double dot = (double)L[j];
      for (int s_ = 1; s_ < planes; ++s_) dot += (double)L[(long)s_ * T + j];
      const double den = nv * sqrt((double)qnorm2[(long)b * T + j]);
      best = fmax(best, dot / fmax(den, 1e-30));
    }
  }
  best = fmax(best, __shfl_xor(best, 1, 64));
  best = fmax(best, __shfl_xor(best, 2, 64));
  if (q == 0) s_query[token] = (float)best;
}

// ---------------------------------------------------------------- softmax relevance (variant)
// stats[row] = (max_i scale*S[row,i], 1 / sum_i exp(scale*S[row,i] - max)); one wave per row, one pass: every
// lane keeps a running (maximum, sum) of its elements and rescales the sum when the maximum moves.
template <typename F>
__global__ __launch_bounds__(256) void softmax_stats_kernel(const F* __restrict__ S, double2* __restrict__ stats,
                                                             long rows, int N, double scale) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const F* p = S + row * (long)N;
  F m = -INFINITY;
  double z = 0.0;
  for (int i = lane; i < N; i += 64) {
    const F v = p[i] * (F)scale;
    if (v > m) { z *= (double)exp(m - v); m = v; }      // m = -inf at first: exp(-inf) = 0
    z += (double)exp(v - m);
  }
  const F mw = wave_max(m);
  z *= (m == -INFINITY) ? 0.0 : (double)exp(m - mw);
  z = wave_sum(z);
  if (lane == 0) stats[row] = make_double2((double)mw, 1.0 / z);
}

// s_query[b,i] = (1/HT) sum_{row < HT} exp(scale*S[b,row,i] - max_row) / Z_row.  The rows of a token are cut into sixteen shares, each added up
// by itself and the shares in order, so that a token's sum is the same in both of the forms below.
constexpr int kMeanShares = 16;
// N rows of a share, all loads in flight, one after the other into acc[0], or (N = 8) into four interleaved sums.
template <int N, typename F>
__device__ __forceinline__ void softmax_mean_rows(const F* p, long pitch, const double2* st, F scale, double (&acc)[4]) {
  F v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) v[u] = p[u * pitch];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const double2 mz = st[u];
    double& a = acc[N == 8 ? u & 3 : 0];
    a = fma((double)exp(v[u] * scale - (F)mz.x), mz.y, a);
  }
}
template <typename F>
__device__ __forceinline__ double softmax_mean_share(const F* p, long pitch, const double2* st, F scale, int r, int end) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (; r + 8 <= end; r += 8) softmax_mean_rows<8>(p + r * pitch, pitch, st + r, scale, acc);
  if (r + 4 <= end) { softmax_mean_rows<4>(p + r * pitch, pitch, st + r, scale, acc); r += 4; }
  if (r + 2 <= end) { softmax_mean_rows<2>(p + r * pitch, pitch, st + r, scale, acc); r += 2; }
  if (r < end) softmax_mean_rows<1>(p + r * pitch, pitch, st + r, scale, acc);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// A workgroup has 64 tokens, each of its sixteen waves a share of the rows.  Bound by the latency of the loads: with all rows of a token in
// one thread 384 rows of 1849 tokens, six images, took 45 us on 48 workgroups, so 7 (576 fp32 tokens, four images, 512 rows:
// covspec_score 286, so 222).
template <typename F>
__global__ __launch_bounds__(64 * kMeanShares) void softmax_mean_kernel(const F* __restrict__ S, const double2* __restrict__ stats,
                                                                        float* __restrict__ s_query, int HT, int N, double scale) {
  __shared__ double part[kMeanShares][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = blockIdx.x * 64 + lane, b = blockIdx.y;
  const int share = (HT + kMeanShares - 1) / kMeanShares, end = (w + 1) * share < HT ? (w + 1) * share : HT;
  if (i < N) part[w][lane] = softmax_mean_share(S + (long)b * HT * N + i, (long)N, stats + (long)b * HT, (F)scale, w * share, end);
  __syncthreads();
  if (w != 0 || i >= N) return;
  double sum = 0.0;
#pragma unroll
  for (int g = 0; g < kMeanShares; ++g) sum += part[g][lane];
  s_query[(long)b * N + i] = (float)(sum / HT);
}

// The same with all shares of a token in one thread, 256 tokens a workgroup: for so many tokens, or so few rows, that the sixteen waves of 64
// tokens are more than it takes to hide the loads (launch_softmax_mean).
template <typename F>
__global__ __launch_bounds__(256) void softmax_mean_wide_kernel(const F* __restrict__ S, const double2* __restrict__ stats, float* __restrict__ s_query,
                                                                int HT, int N, double scale) {
  const int i = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (i >= N) return;
  const F* p = S + (long)b * HT * N + i;
  const double2* st = stats + (long)b * HT;
  const int share = (HT + kMeanShares - 1) / kMeanShares;
  double sum = 0.0;
  // shares of less than eight rows, their length a constant: whole shares at a time, up to eight rows' loads in flight
  auto few = [&](auto length) {
    constexpr int LEN = decltype(length)::value, AT_ONCE = 8 / LEN * LEN;
    auto rows = [&](auto count, int r) {
      constexpr int C = decltype(count)::value;
      F v[C];
#pragma unroll
      for (int u = 0; u < C; ++u) v[u] = p[(long)(r + u) * N];
#pragma unroll
      for (int f = 0; f < C; f += LEN) {
        double acc = 0.0;
#pragma unroll
        for (int u = f; u < C && u < f + LEN; ++u) {
          const double2 mz = st[r + u];
          acc = fma((double)exp(v[u] * (F)scale - (F)mz.x), mz.y, acc);
        }
        sum += acc;
      }
    };
    int r = 0;
    for (; r + AT_ONCE <= HT; r += AT_ONCE) rows(std::integral_constant<int, AT_ONCE>{}, r);
    if (LEN == 1 && r + 4 <= HT) { rows(std::integral_constant<int, 4>{}, r); r += 4; }
    for (; r < HT; r += LEN) sum += softmax_mean_share(p, (long)N, st, (F)scale, r, r + LEN < HT ? r + LEN : HT);
  };
  switch (share) {
    case 1: few(std::integral_constant<int, 1>{}); break;
    case 2: few(std::integral_constant<int, 2>{}); break;
    case 3: few(std::integral_constant<int, 3>{}); break;
    case 4: few(std::integral_constant<int, 4>{}); break;
    case 5: few(std::integral_constant<int, 5>{}); break;
    case 6: few(std::integral_constant<int, 6>{}); break;
    case 7: few(std::integral_constant<int, 7>{}); break;
    default:
      for (int r = 0; r < HT; r += share) sum += softmax_mean_share(p, (long)N, st, (F)scale, r, r + share < HT ? r + share : HT);
  }
  s_query[(long)b * N + i] = (float)(sum / HT);
}

// fp32 logits with N a multiple of 4 (the bf16 workloads): the same two passes with 16-byte loads, base-2
// exponentials (one v_exp_f32 each) and fp32 partial sums; fp64 only where partial results are combined.
// stats[row] = (max_i log2(e)*scale*S[row,i], 1 / sum_i 2^(log2(e)*scale*S[row,i] - max)).
constexpr float kLog2eF = 1.44269504f;

__global__ __launch_bounds__(256) void softmax_stats4_kernel(const float4* __restrict__ S, double2* __restrict__ stats, long rows,
                                                              int N4, float sl2) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float4* p = S + row * (long)N4;
  float m = -INFINITY, z = 0.f;
  for (int c = lane; c < N4; c += 64) {
    const float4 x = p[c];
    const float a = x.x * sl2, b = x.y * sl2, cc = x.z * sl2, d = x.w * sl2;
    const float mx = fmaxf(fmaxf(a, b), fmaxf(cc, d));
    if (mx > m) { z *= __builtin_amdgcn_exp2f(m - mx); m = mx; }     // m = -inf at first: 2^-inf = 0
    z += (__builtin_amdgcn_exp2f(a - m) + __builtin_amdgcn_exp2f(b - m)) + (__builtin_amdgcn_exp2f(cc - m) + __builtin_amdgcn_exp2f(d - m));
  }
  const float mw = wave_max(m);
  double zd = (m == -INFINITY) ? 0.0 : (double)z * (double)__builtin_amdgcn_exp2f(m - mw);
  zd = wave_sum(zd);
  if (lane == 0) stats[row] = make_double2((double)mw, 1.0 / zd);
}

// part[seg][b][i] = sum over the rows of segment seg of 2^(sl2*S[b,row,i] - max_row) / Z_row; a thread owns four
// neighbouring tokens and keeps four rows (64 bytes) in flight.
__global__ __launch_bounds__(256) void softmax_mean4_part_kernel(const float4* __restrict__ S, const double2* __restrict__ stats,
                                                                  double* __restrict__ part, int HT, int N4, int seg_rows, float sl2) {
  const int i4 = blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y, seg = blockIdx.z, B = gridDim.y;
  if (i4 >= N4) return;
  const int r0 = seg * seg_rows, r1 = min(HT, r0 + seg_rows);
  const float4* p = S + (long)b * HT * N4 + i4;
  const double2* st = stats + (long)b * HT;
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
  int r = r0;
  for (; r + 4 <= r1; r += 4) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[(long)(r + u) * N4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double2 mz = st[r + u];
      const float mref = (float)mz.x, rz = (float)mz.y;
      a0 = fmaf(__builtin_amdgcn_exp2f(fmaf(v[u].x, sl2, -mref)), rz, a0);
      a1 = fmaf(__builtin_amdgcn_exp2f(fmaf(v[u].y, sl2, -mref)), rz, a1);
      a2 = fmaf(__builtin_amdgcn_exp2f(fmaf(v[u].z, sl2, -mref)), rz, a2);
      a3 = fmaf(__builtin_amdgcn_exp2f(fmaf(v[u].w, sl2, -mref)), rz, a3);
    }
  }
  for (; r < r1; ++r) {
    const float4 v = p[(long)r * N4];
    const double2 mz = st[r];
    const float mref = (float)mz.x, rz = (float)mz.y;
    a0 = fmaf(__builtin_amdgcn_exp2f(fmaf(v.x, sl2, -mref)), rz, a0);
    a1 = fmaf(__builtin_amdgcn_exp2f(fmaf(v.y, sl2, -mref)), rz, a1);
    a2 = fmaf(__builtin_amdgcn_exp2f(fmaf(v.z, sl2, -mref)), rz, a2);
    a3 = fmaf(__builtin_amdgcn_exp2f(fmaf(v.w, sl2, -mref)), rz, a3);
  }
  double* out = part + (((long)seg * B + b) * N4 + i4) * 4;
  out[0] = a0; out[1] = a1; out[2] = a2; out[3] = a3;
}

// s_query[b,i] = (sum over the segments, in order, of part[seg][b][i]) / HT
__global__ __launch_bounds__(256) void softmax_mean_finish_kernel(const double* __restrict__ part, float* __restrict__ s_query, long BN,
                                                                   int segs, int HT) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= BN) return;
  double s = 0.0;
  for (int g = 0; g < segs; ++g) s += part[(long)g * BN + e];
  s_query[e] = (float)(s / HT);
}

// ---------------------------------------------------------------- min-max + fuse (paper fusion equation)
__device__ __forceinline__ void block_minmax(float& lo, float& hi, float* red) {
  lo = wave_min(lo);
  hi = wave_max(hi);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { red[w] = lo; red[32 + w] = hi; }
  __syncthreads();
  lo = red[0]; hi = red[32];
  for (int k = 1; k < nw; ++k) { lo = fminf(lo, red[k]); hi = fmaxf(hi, red[32 + k]); }
}

__global__ __launch_bounds__(1024) void fuse_kernel(const float* __restrict__ s_query, const float* __restrict__ s_act,
                                                     float* __restrict__ s_fused, int N, float lambda) {
  __shared__ float red[64];
  const long off = (long)blockIdx.x * N;
  float qlo = INFINITY, qhi = -INFINITY, alo = INFINITY, ahi = -INFINITY;
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    float q = s_query[off + i];
    qlo = fminf(qlo, q); qhi = fmaxf(qhi, q);
    if (s_act) { float a = s_act[off + i]; alo = fminf(alo, a); ahi = fmaxf(ahi, a); }
  }
  block_minmax(qlo, qhi, red);
  if (s_act) block_minmax(alo, ahi, red);
  const double lam = (double)lambda;
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    double q = (qhi == qlo) ? 0.0 : ((double)s_query[off + i] - (double)qlo) / ((double)qhi - (double)qlo);
    double f = q;
    if (s_act) {
      double a = (ahi == alo) ? 0.0 : ((double)s_act[off + i] - (double)alo) / ((double)ahi - (double)alo);
      f = lam * q + (1.0 - lam) * a;
    }
    s_fused[off + i] = (float)f;
  }
}

// ---------------------------------------------------------------- gather
__global__ __launch_bounds__(256) void gather_rows_kernel(const unsigned char* __restrict__ X, const int32_t* __restrict__ idx,
                                                           unsigned char* __restrict__ out, int N, int k, long row_bytes) {
  const long row = blockIdx.x;  // b*k + j
  const long b = row / k;
  const long src = (b * N + idx[row]) * row_bytes;
  const long dst = row * row_bytes;
  for (long o = (long)threadIdx.x * 16; o < row_bytes; o += 256 * 16)
    *(u32x4_t*)(out + dst + o) = *(const u32x4_t*)(X + src + o);
}

inline unsigned blocks_for(long n, int per) { return (unsigned)((n + per - 1) / per); }

__global__ __launch_bounds__(256) void random_scores_kernel(float* __restrict__ out, int B, int N, uint32_t seed, int image0) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long)B * N) return;
  const unsigned long long b = (unsigned long long)(e / N), i = (unsigned long long)(e - (long)b * N);
  // image0: index of this call's first image in the caller's batch (a ragged batch is worked off in runs)
  unsigned long long z = (unsigned long long)seed * 0x9E3779B97F4A7C15ull + (((b + (unsigned long long)image0) << 32) | i) + 0x632BE59BD9B4E019ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  out[e] = (float)(unsigned int)(z >> 40) * 0x1p-24f;
}

__global__ void fill_int_kernel(int* __restrict__ p, int n, int value) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

}  // namespace

hipError_t launch_transpose(const void* in, void* out, const void* in1, void* out1, int rows, int cols, int dtype, hipStream_t st) {
  const int piece = dtype == DT_BF16 ? 8 : 4;
  const auto in_pieces = [&](const void* a, const void* b) { return rows % piece == 0 && cols % piece == 0 && (((uintptr_t)a | (uintptr_t)b) & 15) == 0; };
  const bool pieces = in_pieces(in, out);
  if (in1 && in_pieces(in1, out1) != pieces) {        // a form each
    const hipError_t e = launch_transpose(in, out, nullptr, nullptr, rows, cols, dtype, st);
    return e != hipSuccess ? e : launch_transpose(in1, out1, nullptr, nullptr, rows, cols, dtype, st);
  }
  dim3 grid((cols + 63) / 64, (rows + 63) / 64, in1 ? 2 : 1), block(256);
#define COVSPEC_TRANSPOSE(kernel, T) hipLaunchKernelGGL((kernel<T>), grid, block, 0, st, (const T*)in, (T*)out, (const T*)in1, (T*)out1, rows, cols)
  if (pieces) {
    if (dtype == DT_BF16) COVSPEC_TRANSPOSE(transpose16_kernel, bf16_t);
    else COVSPEC_TRANSPOSE(transpose16_kernel, float);
  } else {
    if (dtype == DT_BF16) COVSPEC_TRANSPOSE(transpose_kernel, bf16_t);
    else COVSPEC_TRANSPOSE(transpose_kernel, float);
  }
#undef COVSPEC_TRANSPOSE
  return hipGetLastError();
}

hipError_t launch_activity(const void* hidden, float* s_act, int B, int N, int d, int K, int dtype, hipStream_t st) {
  long tokens = (long)B * N;
  return dtype == DT_BF16 ? activity_dispatch<DT_BF16>(hidden, s_act, tokens, N, d, K, st)
                          : activity_dispatch<DT_F32>(hidden, s_act, tokens, N, d, K, st);
}

hipError_t launch_row_norm2(const void* x, int in_type, void* out, bool out_f64, long rows, int d, hipStream_t st) {
  dim3 grid(blocks_for(rows, 4)), block(256);
  if (in_type == IN_BF16 && !out_f64) hipLaunchKernelGGL((row_norm2_kernel<bf16_t, float>), grid, block, 0, st, (const bf16_t*)x, (float*)out, rows, d);
  else if (in_type == IN_F32 && out_f64) hipLaunchKernelGGL((row_norm2_kernel<float, double>), grid, block, 0, st, (const float*)x, (double*)out, rows, d);
  else if (in_type == IN_F64 && out_f64) hipLaunchKernelGGL((row_norm2_kernel<double, double>), grid, block, 0, st, (const double*)x, (double*)out, rows, d);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_convert(const void* src, int in_type, void* dst, bool out_f64, long n, hipStream_t st) {
  dim3 grid(blocks_for(n, 256)), block(256);
  if (in_type == IN_BF16 && !out_f64) hipLaunchKernelGGL((convert_kernel<bf16_t, float>), grid, block, 0, st, (const bf16_t*)src, (float*)dst, n);
  else if (in_type == IN_F32 && out_f64) hipLaunchKernelGGL((convert_kernel<float, double>), grid, block, 0, st, (const float*)src, (double*)dst, n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_sum_split3(const float* src, int planes, long plane_stride, long rows, int d, long rows_per_group,
                             unsigned short* out, hipStream_t st) {
  const bool wide = d % 4 == 0 && plane_stride % 4 == 0 && ((uintptr_t)src & 15) == 0 && ((uintptr_t)out & 7) == 0;
  dim3 block(256);
  if (wide) hipLaunchKernelGGL(sum_split3_kernel<4>, dim3(blocks_for(rows * d / 4, 256)), block, 0, st, src, planes, plane_stride, rows, d, rows_per_group, out);
  else hipLaunchKernelGGL(sum_split3_kernel<1>, dim3(blocks_for(rows * d, 256)), block, 0, st, src, planes, plane_stride, rows, d, rows_per_group, out);
  return hipGetLastError();
}

hipError_t launch_query_rows(const float* src, long rows, int d, unsigned short* eq3, float* norm2, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (d % 4 != 0 || rows > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(query_rows_kernel, dim3((unsigned)rows), dim3(256), 0, st, src, rows, d, eq3, norm2);
  return hipGetLastError();
}

hipError_t launch_cosine_max(const void* logits, int planes, const void* vnorm2, int nparts, const void* qnorm2, bool f64,
                             float* s_query, int B, int N, int T, hipStream_t st) {
  if (B <= 0 || N <= 0) return hipSuccess;
  dim3 grid((unsigned)((N + 63) / 64), (unsigned)B), block(256);
  const size_t lds = (size_t)(T + 1) * sizeof(double);
  if (lds > 48 * 1024) return hipErrorInvalidValue;     // more than 6143 query keywords
  if (f64) hipLaunchKernelGGL((cosine_max_kernel<double>), grid, block, lds, st, (const double*)logits, planes, (const double*)vnorm2, nparts, (const double*)qnorm2, s_query, N, T);
  else hipLaunchKernelGGL((cosine_max_kernel<float>), grid, block, lds, st, (const float*)logits, planes, (const float*)vnorm2, nparts, (const float*)qnorm2, s_query, N, T);
  return hipGetLastError();
}

// The fast path needs fp32 logits, N % 4 == 0 and `part` scratch of softmax_scratch_bytes(B, N) bytes.
size_t softmax_scratch_bytes(int B, int N) { return (size_t)32 * B * N * sizeof(double); }

hipError_t launch_softmax_stats(const void* S, bool f64, void* stats, long rows, int N, double scale, bool base2, hipStream_t st) {
  dim3 grid(blocks_for(rows, 4)), block(256);
  if (f64) hipLaunchKernelGGL((softmax_stats_kernel<double>), grid, block, 0, st, (const double*)S, (double2*)stats, rows, N, scale);
  else if (base2) hipLaunchKernelGGL(softmax_stats4_kernel, grid, block, 0, st, (const float4*)S, (double2*)stats, rows, N / 4, (float)scale * kLog2eF);
  else hipLaunchKernelGGL((softmax_stats_kernel<float>), grid, block, 0, st, (const float*)S, (double2*)stats, rows, N, scale);
  return hipGetLastError();
}

bool softmax_base2(bool f64, int N) { return !f64 && N % 4 == 0; }

hipError_t launch_softmax_mean(const void* S, bool f64, const void* stats, float* s_query, int B, int HT, int N, double scale,
                               void* part, hipStream_t st) {
  if (softmax_base2(f64, N) && part) {
    const int N4 = N / 4, gx = (N4 + 255) / 256;
    // row segments: enough workgroups for eight waves per SIMD, at most 32 segments of at least 32 rows
    int segs = (2048 + gx * B - 1) / (gx * B);
    const int most = HT / 32 > 0 ? HT / 32 : 1;
    segs = segs > 32 ? 32 : segs;
    segs = segs > most ? most : segs;
    const int seg_rows = (HT + segs - 1) / segs;
    segs = (HT + seg_rows - 1) / seg_rows;
    hipLaunchKernelGGL(softmax_mean4_part_kernel, dim3(gx, B, segs), dim3(256), 0, st, (const float4*)S, (const double2*)stats,
                       (double*)part, HT, N4, seg_rows, (float)scale * kLog2eF);
    const long BN = (long)B * N;
    hipLaunchKernelGGL(softmax_mean_finish_kernel, dim3(blocks_for(BN, 256)), dim3(256), 0, st, (const double*)part, s_query, BN, segs, HT);
    return hipGetLastError();
  }
  // A wave has 64 tokens: from two on every SIMD, or half of them where a share is one row, the waves themselves hide the loads.  us of
  // covspec_score, sixteen waves a workgroup / a thread for all rows, bf16, width 64: 64 images of 2881 tokens (2944 waves) 1 row 95.6 / 91.6, 16 99.0 / 94.3, 64
  // 108.0 / 105.6, 128 131.5 / 126.4; 16 of 2881 (736) 4 rows 59.8 / 59.4, 16 63.0 / 61.8, 32 64.4 / 65.1, 128 66.3 / 72.2; 128 of 577 (1280) 16
  // rows 58.0 / 56.8, 64 62.4 / 63.5; 8 of 2881 (368) 16 rows 51.0 / 50.8, 64 55.7 / 62.6; 4 (184) 45.6 / 46.0 with 1 row, 47.4 / 47.8 with 16.
  const int waves = (N + 63) / 64;
  const bool wide = (long)waves * B >= (HT <= kMeanShares ? 640 : 2048);
#define COVSPEC_MEAN(kernel, F, grid, block) hipLaunchKernelGGL((kernel<F>), grid, block, 0, st, (const F*)S, (const double2*)stats, s_query, HT, N, scale)
  if (wide) {
    const dim3 grid((N + 255) / 256, B), block(256);
    if (f64) COVSPEC_MEAN(softmax_mean_wide_kernel, double, grid, block);
    else COVSPEC_MEAN(softmax_mean_wide_kernel, float, grid, block);
  } else {
    const dim3 grid(waves, B), block(64 * kMeanShares);
    if (f64) COVSPEC_MEAN(softmax_mean_kernel, double, grid, block);
    else COVSPEC_MEAN(softmax_mean_kernel, float, grid, block);
  }
#undef COVSPEC_MEAN
  return hipGetLastError();
}

hipError_t launch_fuse(const float* s_query, const float* s_act, float* s_fused, int B, int N, float lambda, hipStream_t st) {
  hipLaunchKernelGGL(fuse_kernel, dim3(B), dim3(1024), 0, st, s_query, s_act, s_fused, N, lambda);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const void* X, const int32_t* idx, void* out, int B, int N, int k, long row_bytes, hipStream_t st) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((long)B * k)), dim3(256), 0, st, (const unsigned char*)X, idx,
                     (unsigned char*)out, N, k, row_bytes);
  return hipGetLastError();
}

hipError_t launch_random_scores(float* out, int B, int N, uint32_t seed, int image0, hipStream_t stream) {
  const long total = (long)B * N;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(random_scores_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, out, B, N, seed, image0);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int n, int value, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_int_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n, value);
  return hipGetLastError();
}

}  // namespace covspec
