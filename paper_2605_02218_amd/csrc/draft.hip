// Draft-side vocabulary pass (paper Sec. III-B, margin and gating equations; Sec. III-C, fan-out equation and
// the bonus-token candidate rule): for every drafted position one read of the draft logits yields the softmax
// statistics, the two largest probabilities (margin, gate) and the F_j words with the largest logits other
// than the drafted token.
//
// Scan kernel, one workgroup per chunk of 8192 words of one row: every thread keeps its 32 logits in
// registers as loaded, accumulates the streaming softmax statistics, and the chunk's K = F_0 + 1 largest logits are
// found by a threshold instead of K rounds of a block-wide argmax: tau = the K-th largest of the 64 quad
// maxima, so at least K logits are >= tau and, for continuous data, only about K more; those few go to a list
// in LDS that one wave ranks by all-pairs comparison.  A list that overflows (many equal logits, or fewer than
// K quads with data) goes another way to the same result: the logits above the K-th largest thread maximum are ranked by
// the workgroup and the lowest words among those equal to it fill up, or, where more than 256 are above, K rounds of block-wide
// argmax.
// Bound by its vector instructions, 12 per logit, which keep the VALUs busy in two thirds or more of its cycles now that eight
// waves per SIMD cover the latencies of a workgroup's dozen phases: with the logits widened to fp32 and the overflowing
// chunks' packed keys formed ahead of their loop the kernel took 87 registers (5 waves per SIMD) and 49 us for 512 rows of 151936
// bf16 words; with the logits kept as loaded, one reference per thread instead of a running one and the few candidate
// threads' logits looked through in LDS it takes 64 registers, none spilled, and 33.6 us (4.6 TB/s; six inputs in turn, 0.93 GB.
// The same input again and again, part of which the 256 MB cache keeps: 31.8).
// Merge kernel, two waves per row: combines the chunks' statistics in fp64, merges their candidate lists,
// evaluates the margin and writes gate and candidates.
#include "common.h"
#include "kernels.h"
#include "vocab.h"

namespace covspec {

namespace {

typedef unsigned long long u64;

constexpr int DTH = 256;                  // threads of the scan kernel
constexpr int EPT = 32;                   // logits per thread
constexpr int DCL = DTH * EPT;            // words per chunk
constexpr int KMAX = 33;                  // F_0 <= 32, plus one for the drafted token
constexpr int LISTCAP = 64;               // threshold list: one entry per lane of the ranking wave
constexpr int POOL = 64;                  // threads whose logits are looked through one by one
constexpr int MAXCHUNKS = 64;             // the merge kernel keeps chunks * K keys in LDS

// (order key of the logit, ~word): larger logit first, lower word first among equal logits; never 0 for a real entry
__device__ __forceinline__ u64 pack_key(float v, int w) { return ((u64)float_order_key(v) << 32) | (u64)(0xFFFFFFFFu - (uint32_t)w); }
__device__ __forceinline__ int key_word(u64 k) { return (int)(0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull)); }
__device__ __forceinline__ float key_value(u64 k) {
  const uint32_t o = (uint32_t)(k >> 32);
  return __uint_as_float((o & 0x80000000u) ? (o ^ 0x80000000u) : ~o);
}

// rank of a key among the n distinct keys of an LDS array: the number of keys greater than its own
__device__ __forceinline__ int wave_rank(const u64* keys, int n, u64 mine) {
  int rank = 0;
  int j = 0;
  for (; j + 8 <= n; j += 8) {        // eight broadcast reads in flight
    u64 k[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) k[q] = keys[j + q];
#pragma unroll
    for (int q = 0; q < 8; ++q) rank += k[q] > mine ? 1 : 0;
  }
  for (; j < n; ++j) rank += keys[j] > mine ? 1 : 0;
  return rank;
}

struct FanTable { unsigned char f[64]; };   // F_j by position inside the drafted segment

// stats[(row * chunks + c) * 2 + {0,1}] = reference, sum (base-2 domain); top[(row * chunks + c) * KMAX + r],
// r < K: the chunk's r-th largest logit as a packed key, 0 where the chunk has fewer.
template <int DT>
__global__ __launch_bounds__(DTH, DT == DT_F32 ? 6 : 8) void draft_scan_kernel(const void* __restrict__ zd, int V, int chunks, int K,
                                                         double* __restrict__ stats, u64* __restrict__ top) {
  constexpr int N = LogitVec<DT>::N;
  constexpr int NV = EPT / N;
  __shared__ u64 gkey[64];
  __shared__ u64 list[LISTCAP];
  __shared__ u64 wbest[2][DTH / 64];
  __shared__ double red[DTH / 64][2];
  __shared__ float sh_tau;
  __shared__ int sh_cnt, sh_found, sh_above, equal[2][DTH / 64];
  __shared__ u32x4_t pool[POOL][NV];      // EPT logits of a thread, as loaded
  __shared__ int pool_id[POOL];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long row = blockIdx.y;
  const int c = blockIdx.x;
  const int w0 = c * DCL, w1 = min(V, w0 + DCL);      // V % N == 0: whole vectors only
  const long base = row * (long)V;

  // The logits stay as they were loaded (16-bit types: two per register) and are widened where they are used.  A slot without
  // a word holds NaN: like a NaN logit it compares false against every threshold and is skipped by max.
  constexpr uint32_t kNoWord = DT == DT_BF16 ? 0x7FC07FC0u : DT == DT_F16 ? 0x7E007E00u : 0x7FC00000u;
  u32x4_t raw[NV];
  int nv = 0;                          // vectors with words
  float vmax[NV];                      // per vector, NaN ignored
  float tmax = -INFINITY;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int w = w0 + (i * DTH + tid) * N;
    raw[i] = (u32x4_t){kNoWord, kNoWord, kNoWord, kNoWord};
    if (w < w1) {
      raw[i] = LogitVec<DT>::load_raw(zd, base + w);
      nv = i + 1;
    }
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    float t[N];
    LogitVec<DT>::unpack(raw[i], t);
    vmax[i] = -INFINITY;
#pragma unroll
    for (int e = 0; e < N; ++e) vmax[i] = fmaxf(vmax[i], t[e]);
    tmax = fmaxf(tmax, vmax[i]);
  }
  // streaming pair of all the thread's logits at once: they are in registers, so the reference is their maximum and no
  // partial sum is ever rescaled (see vocab.h for the base-2 domain)
  const float cref = tmax * kLog2e;
  float sum = 0.f;
  {
    const float cn = cref == -INFINITY ? 0.f : cref;      // only masked words: any finite reference gives zeros
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) {
        float t[N];
        LogitVec<DT>::unpack(raw[i], t);
#pragma unroll
        for (int e = 0; e < N; e += 2) {
          s0 += __builtin_amdgcn_exp2f(__builtin_fmaf(t[e], kLog2e, -cn));
          s1 += __builtin_amdgcn_exp2f(__builtin_fmaf(t[e + 1], kLog2e, -cn));
        }
      }
    sum = s0 + s1;
  }

  // quad maxima -> tau
  const float own = tmax;
  tmax = fmaxf(tmax, __shfl_xor(tmax, 1, 64));
  tmax = fmaxf(tmax, __shfl_xor(tmax, 2, 64));
  if ((lane & 3) == 0) gkey[tid >> 2] = ((u64)float_order_key(tmax) << 32) | (u64)(63 - (tid >> 2));
  if (tid == 0) { sh_cnt = 0; sh_found = 0; sh_above = 0; }
  {
    double mm, ss;
    block_combine<DTH / 64>(cref, sum, red, mm, ss);      // its barrier also publishes gkey and sh_cnt
    if (tid == 0) { stats[(row * chunks + c) * 2] = mm; stats[(row * chunks + c) * 2 + 1] = ss; }
  }
  // the two single-wave steps rotate over the waves with the chunk, so that no one SIMD of the compute unit
  // carries them for every resident workgroup
  const int rw = (int)((blockIdx.x + blockIdx.y) & 3u);
  if (wv == rw) {
    const u64 mine = gkey[lane];
    if (wave_rank(gkey, 64, mine) == K - 1) sh_tau = key_value(mine);     // ranks are a permutation of 0..63; K <= 64
  }
  __syncthreads();
  const float tau = sh_tau;
  // the few threads that hold a logit of tau or more (K quads and a few) put all of theirs into LDS, where the whole
  // workgroup looks through them: 32 compare-and-branch steps of every wave cost more than that
  if (nv > 0 && own >= tau) {       // a thread without words has -inf, which is tau where few quads have data
    const int pos = atomicAdd(&sh_cnt, 1);
    if (pos < POOL) {
      pool_id[pos] = tid;
#pragma unroll
      for (int i = 0; i < NV; ++i) pool[pos][i] = raw[i];
    }
  }
  __syncthreads();
  const int holders = sh_cnt;
  if (holders <= POOL) {
    for (int i = tid; i < holders * EPT; i += DTH) {
      const float x = (float)LogitVec<DT>::at(&pool[0][0], i);
      if (x >= tau) {
        const int e = i % EPT, pos = atomicAdd(&sh_found, 1);
        if (pos < LISTCAP) list[pos] = pack_key(x, w0 + ((e / N) * DTH + pool_id[i / EPT]) * N + e % N);
      }
    }
  }
  __syncthreads();
  const int n = holders <= POOL ? sh_found : LISTCAP + 1;
  u64* out = top + (row * chunks + c) * KMAX;
  if (n <= LISTCAP) {
    if (wv == ((rw + 2) & 3)) {
      const u64 mine = lane < n ? list[lane] : 0ull;
      const int rank = wave_rank(list, n, mine);
      if (lane < n && rank < K) out[rank] = mine;
      if (lane >= n && lane < K) out[lane] = 0ull;        // fewer than K logits in the chunk
    }
    return;
  }
  // Many logits of tau or more: equal ones (bf16 rows with a wide candidate list, masked words), or live words in few quads.
  // Another tau, the K-th largest of the threads' maxima; the logits above it are listed and ranked by the whole workgroup, and
  // the rest of the K are the lowest words among those equal to it.  The logits are read anew from here on (from the caches), so
  // that none is live in a register.
  auto word_at = [&](int i) { return w0 + (i * DTH + tid) * N; };
  u64* big = (u64*)&pool[0][0];       // DTH keys; the pool has been looked through
  const u64 own_key = ((u64)float_order_key(own) << 32) | (u64)(DTH - 1 - tid);
  big[tid] = own_key;
  __syncthreads();
  if (wave_rank(big, DTH, own_key) == K - 1) sh_tau = key_value(own_key);
  __syncthreads();
  const float tau2 = sh_tau;
#pragma unroll 1
  for (int i = 0; i < nv; ++i) {
    float t[N];
    LogitVec<DT>::load(zd, base + word_at(i), t);
#pragma unroll
    for (int e = 0; e < N; ++e)
      if (t[e] > tau2) {
        const int pos = atomicAdd(&sh_above, 1);
        if (pos < DTH) big[pos] = pack_key(t[e], word_at(i) + e);
      }
  }
  __syncthreads();
  const int above = sh_above;
  if (above <= DTH) {
    if (tid < above) {
      const u64 mine = big[tid];
      const int rank = wave_rank(big, above, mine);
      if (rank < K) out[rank] = mine;
    }
    const int need = K - above;
    int have = 0;                     // words equal to tau2 in the vectors before i, the same in every thread
#pragma unroll 1
    for (int i = 0; i < NV && have < need; ++i) {
      float t[N];
      int mine = 0;
      if (i < nv) {
        LogitVec<DT>::load(zd, base + word_at(i), t);
#pragma unroll
        for (int e = 0; e < N; ++e) mine += t[e] == tau2 ? 1 : 0;
      }
      int upto = mine;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(upto, o, 64);
        if (lane >= o) upto += v;
      }
      if (lane == 63) equal[i & 1][wv] = upto;
      __syncthreads();                // the other set of `equal` is free behind the next vector's
      int pos = have + upto - mine;
#pragma unroll
      for (int k = 0; k < DTH / 64; ++k) {
        const int v = equal[i & 1][k];
        if (k < wv) pos += v;
        have += v;
      }
      if (mine > 0) {
#pragma unroll
        for (int e = 0; e < N; ++e)
          if (t[e] == tau2) {
            if (pos < need) out[above + pos] = pack_key(tau2, word_at(i) + e);
            ++pos;
          }
      }
    }
    for (int p = have + tid; p < need; p += DTH) out[above + p] = 0ull;      // fewer than K logits in the chunk
    return;
  }
  // More than DTH above tau2 (in fewer than K threads): K rounds of block-wide argmax.  A thread keeps the key of its largest word that is left, and only
  // the thread that lost it looks through its words again.
  uint32_t alive = nv * N >= 32 ? 0xFFFFFFFFu : (1u << (nv * N)) - 1u;      // whole vectors: bits i*N .. i*N+N-1
  auto largest = [&]() -> u64 {
    u64 best = 0ull;
#pragma unroll 1
    for (int i = 0; i < nv; ++i) {
      const int w = word_at(i);
      float t[N];
      LogitVec<DT>::load(zd, base + w, t);
#pragma unroll
      for (int e = 0; e < N; ++e) {
        const u64 k = pack_key(t[e], w + e);
        if (((alive >> (i * N + e)) & 1u) && t[e] == t[e] && k > best) best = k;
      }
    }
    return best;
  };
  u64 mine = largest();
  for (int r = 0; r < K; ++r) {
    const u64 best = wave_max(mine);
    if (lane == 0) wbest[r & 1][wv] = best;
    __syncthreads();                  // the other set of wbest is free behind the next round's
    u64 b = wbest[r & 1][0];
#pragma unroll
    for (int k = 1; k < DTH / 64; ++k) b = wbest[r & 1][k] > b ? wbest[r & 1][k] : b;
    if (tid == 0) out[r] = b;
    if (b != 0ull && b == mine) {     // keys are distinct: one thread
      const int rel = key_word(b) - w0;                   // in [0, DCL)
      alive &= ~(1u << ((rel / N / DTH) * N + rel % N));
      mine = largest();
    }
  }
}

// The largest of a wave's keys, the same in all lanes: a prefix maximum along the rows of 16 lanes and across them, all in DPP moves.
template <int CTRL>
__device__ __forceinline__ u64 max_moved(u64 v) {
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(v & 0xFFFFFFFFull), CTRL, 0xf, 0xf, false);
  const u64 o = ((u64)hi << 32) | lo;
  return o > v ? o : v;
}
__device__ __forceinline__ u64 wave_largest(u64 v) {
  v = max_moved<0x111>(v);       // row_shr 1, 2, 4, 8
  v = max_moved<0x112>(v);
  v = max_moved<0x114>(v);
  v = max_moved<0x118>(v);
  v = max_moved<0x142>(v);       // lane 15 of a row to the next row, lane 31 to the upper half
  v = max_moved<0x143>(v);
  return ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 63) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(v & 0xFFFFFFFFull), 63);
}

// Two waves per row.  Wave 0 merges the chunks' lists, which are in descending order: lane c holds the head of chunk c's, K times the
// largest head is taken and its lane moves on.  Wave 1 combines the chunks' statistics meanwhile, all on one reference.
// A chain of latencies: with K rounds over all keys by shuffles and the statistics combined pair by pair, one after the other in one
// wave, 10 us for 512 rows of 19 chunks, 9 candidates each; so 5.2.
constexpr int MTH = 128;
__global__ __launch_bounds__(MTH) void draft_merge_kernel(const double* __restrict__ stats, const u64* __restrict__ top,
                                                         const int32_t* __restrict__ tok, int L, int V, int chunks, int K, int shift, int F0,
                                                         FanTable fan, float gamma, float* __restrict__ margin_out,
                                                         int32_t* __restrict__ gate_out, int32_t* __restrict__ cand_out) {
  extern __shared__ u64 pool[];                 // [chunks][K]
  __shared__ u64 sorted[KMAX];
  __shared__ double total[2];
  const int row = blockIdx.x, lane = threadIdx.x & 63;
  const int y = F0 > 0 ? tok[row] : 0;
  double m = 0.0, s = 0.0;
  if (threadIdx.x >= 64 && lane < chunks) {     // chunks <= 64
    m = stats[((long)row * chunks + lane) * 2];
    s = stats[((long)row * chunks + lane) * 2 + 1];
  }
  for (int i = threadIdx.x; i < chunks << shift; i += MTH) {        // K <= 2^shift
    const int c = i >> shift, r = i - (c << shift);
    if (r < K) pool[c * K + r] = top[((long)row * chunks + c) * KMAX + r];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const u64* list = pool + lane * K;
    int at = 0;
    u64 head = lane < chunks ? list[0] : 0ull;
    u64 after = lane < chunks && K > 1 ? list[1] : 0ull;            // the one behind the head, on its way while the heads are compared
    for (int r = 0; r < K; ++r) {
      const u64 best = wave_largest(head);
      if (lane == 0) sorted[r] = best;
      if (best != 0ull && head == best) {       // keys are distinct: exactly one lane
        head = after;
        ++at;
        after = at + 1 < K ? list[at + 1] : 0ull;
      }
    }
  } else {
    const double ref = wave_max(s > 0.0 ? m : -INFINITY);
    const double sum = wave_sum(s > 0.0 ? s * exp2(m - ref) : 0.0);
    if (lane == 0) { total[0] = ref; total[1] = sum; }
  }
  __syncthreads();
  if (threadIdx.x >= 64) {
    // margin = p_(1) - p_(2); V >= 2, so both exist
    const double e = lane < 2 ? exp2((double)key_value(sorted[lane]) * (double)kLog2e - total[0]) : 0.0;
    const double e2 = __shfl(e, 1, 64);
    if (lane == 0) {
      const float mf = (float)((e - e2) / total[1]);
      margin_out[row] = mf;
      gate_out[row] = mf >= gamma ? 0 : 1;
    }
    return;
  }
  if (F0 > 0) {
    const u64 mine = lane < K ? sorted[lane] : 0ull;
    const u64 hit = __ballot(mine != 0ull && key_word(mine) == y);
    const int pos_y = hit ? __ffsll((long long)hit) - 1 : K;
    const int Fj = fan.f[row % L];
    if (lane < F0) {
      const int j = lane + (lane >= pos_y ? 1 : 0);    // <= F0 = K - 1
      const u64 k = sorted[j];
      cand_out[(long)row * F0 + lane] = (lane < Fj && k != 0ull) ? key_word(k) : -1;
    }
  }
}

}  // namespace

int draft_chunks(int V) { return (V + DCL - 1) / DCL; }
int draft_max_vocab() { return MAXCHUNKS * DCL; }

size_t draft_workspace_bytes(int S, int L, int V) {
  const size_t rows = (size_t)S * L, chunks = (size_t)draft_chunks(V);
  return rows * chunks * 2 * sizeof(double) + rows * chunks * KMAX * sizeof(u64) + 512;
}

hipError_t launch_draft(const void* zd, const int32_t* tok, int S, int L, int V, int dtype, int F0, const int* fanout, float gamma,
                        float* margin, int32_t* gate, int32_t* cand, void* ws, hipStream_t st) {
  const int chunks = draft_chunks(V);
  const long rows = (long)S * L;
  if (S < 1 || L < 1 || L > 64 || V < 2 || rows > 65535 || chunks > MAXCHUNKS || F0 < 0 || F0 > KMAX - 1) return hipErrorInvalidValue;
  const int K = F0 + 1 < 2 ? 2 : F0 + 1;
  FanTable fan;
  for (int j = 0; j < 64; ++j) fan.f[j] = (unsigned char)(j < L ? fanout[j] : 0);
  double* stats = (double*)ws;
  u64* top = (u64*)(stats + (size_t)rows * chunks * 2);
  if (dtype == DT_BF16)
    hipLaunchKernelGGL((draft_scan_kernel<DT_BF16>), dim3(chunks, (unsigned)rows), dim3(DTH), 0, st, zd, V, chunks, K, stats, top);
  else if (dtype == DT_F16)
    hipLaunchKernelGGL((draft_scan_kernel<DT_F16>), dim3(chunks, (unsigned)rows), dim3(DTH), 0, st, zd, V, chunks, K, stats, top);
  else
    hipLaunchKernelGGL((draft_scan_kernel<DT_F32>), dim3(chunks, (unsigned)rows), dim3(DTH), 0, st, zd, V, chunks, K, stats, top);
  int shift = 1;
  while ((1 << shift) < K) ++shift;
  hipLaunchKernelGGL(draft_merge_kernel, dim3((unsigned)rows), dim3(MTH), (size_t)chunks * K * sizeof(u64), st, (const double*)stats,
                     (const u64*)top, tok, L, V, chunks, K, shift, F0, fan, gamma, margin, gate, cand);
  return hipGetLastError();
}

}  // namespace covspec
