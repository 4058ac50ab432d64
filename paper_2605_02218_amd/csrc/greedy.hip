// Greedy residual-update selection (a variant that is not in the paper; it replaces
// the rank-r SVD energy ranking of Sec. III-A.3 by k greedy picks).
//
// Pivoted Cholesky of the token Gram matrix G = Z Z^T in fp64: the residual squared
// norm of token i after projecting out the picked tokens is rho_i; each step picks
// argmax rho (decided on the fp32-rounded value, ties -> lower index), forms the new
// Cholesky column l = (G[:,p] - L L[p,:]^T) / sqrt(rho_p) and updates rho -= l^2.
//
// Four kernels, chosen by launch_greedy from the values each would move: the right-looking panel kernels
// (greedy_panel_kernel, the usual choice, and greedy_step_kernel for many rows), and two left-looking ones for the case that the picks are a small
// part of the rows, on several workgroups per image (greedy_kernel) or one (greedy_single_kernel).
//
// Left-looking on several workgroups (greedy_kernel).  The k steps are dependent, but inside a step the rows are
// independent, so an image is spread over nP/64 workgroups of 64 rows each: a workgroup keeps rho of its rows in
// registers, posts its best (key, rho) per step, all workgroups of the image meet at a
// barrier in global memory (one per step), read the posts, agree on the pivot p, fetch
// the pivot's Cholesky row L[p, 0..t) and extend their own 64 rows of L.  L is stored
// transposed (Lt[t][i]) so that a workgroup's part of a column is one 512-byte run.
// Inside a workgroup lanes are rows and the four waves split the dot product over t.
// Workgroups take (image, slot) from a ticket counter, so the resident ones always form
// whole images plus one partial image that is next in the dispatch order.
#include "common.h"
#include "host_cache.h"
#include "kernels.h"

namespace covspec {

namespace {

constexpr int TPB = 1024;   // finish kernel
constexpr int GR = 64;      // rows per workgroup
constexpr int GT = 256;     // threads per workgroup

struct GreedyCtl {
  ImageBarrier bar;
  unsigned int ticket;   // ctl[0] only
  unsigned int pad;
};

// posts: per image [2][W] keys (u64) then [2][W] rho (fp64), double-buffered by step parity
__global__ __launch_bounds__(GT) void greedy_kernel(const double* __restrict__ G, int n, int nP, int k, double* Lt, int32_t* __restrict__ order,
                                                     float* __restrict__ resid, GreedyCtl* ctl, unsigned long long* posts,
                                                     int* img_status, long long limit_ticks) {
  __shared__ double Lp[4096];
  __shared__ double part[4][GR];
  __shared__ unsigned long long sh_key;
  __shared__ double sh_rho;
  __shared__ int s_flag;
  const int W = nP / GR;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_flag = (int)atomicAdd(&ctl[0].ticket, 1u);
  __syncthreads();
  const int ticket = s_flag;
  __syncthreads();
  const int b = ticket / W, slot = ticket - b * W;
  GreedyCtl* cb = ctl + b;
  const double* Gb = G + (long)b * nP * nP;
  double* Ltb = Lt + (long)b * k * nP;
  unsigned long long* keys = posts + (long)b * 4 * W;       // [2][W]
  double* rhos = (double*)(keys + 2 * W);                   // [2][W]
  const int i = slot * GR + lane;                           // this lane's row (all four waves hold a copy)

  double rho = (i < n) ? Gb[(long)i * nP + i] : 0.0;
  bool picked = !(i < n);
  unsigned int target = 0;
  bool alive = true;

  for (int t = 0; t < k && alive; ++t) {
    // ---- local argmax of float(rho) over the unpicked rows, lowest index on ties (wave 0 suffices)
    if (w == 0) {
      unsigned long long key = 0ull;
      if (!picked) key = ((unsigned long long)float_order_key((float)rho) << 32) | (0xFFFFFFFFu - (uint32_t)i);
      const unsigned long long best = wave_max(key);
      const unsigned long long bal = __ballot(key == best && key != 0ull);
      if (best != 0ull && lane == (int)__ffsll((long long)bal) - 1) {
        keys[(t & 1) * W + slot] = best;
        rhos[(t & 1) * W + slot] = rho;
      }
      if (best == 0ull && lane == 0) keys[(t & 1) * W + slot] = 0ull;
    }
    target += (unsigned int)W;
    alive = image_barrier_wait(&cb->bar, target, &s_flag, limit_ticks);
    if (!alive) break;
    // ---- global argmax over the posts
    if (w == 0) {
      unsigned long long key = 0ull;
      double r = 0.0;
      for (int q = lane; q < W; q += 64) {
        const unsigned long long kq = keys[(t & 1) * W + q];
        if (kq > key) { key = kq; r = rhos[(t & 1) * W + q]; }
      }
      const unsigned long long best = wave_max(key);
      const unsigned long long bal = __ballot(key == best);
      if (lane == (int)__ffsll((long long)bal) - 1) { sh_key = best; sh_rho = r; }
    }
    __syncthreads();
    const int p = (int)(0xFFFFFFFFu - (uint32_t)(sh_key & 0xFFFFFFFFull));
    const double rp = sh_rho;
    if ((unsigned)p >= (unsigned)n) {   // cannot happen with consistent posts; never index with it
      if (tid == 0) __hip_atomic_store(&cb->bar.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      alive = false;
      break;
    }
    if (p == i) picked = true;
    for (int q = tid; q < t; q += GT) Lp[q] = Ltb[(long)q * nP + p];
    __syncthreads();
    // ---- dot products: wave w takes q = w, w+4, ...
    double d0 = 0.0, d1 = 0.0;
    {
      const double* col = Ltb + i;
      int q = w;
      // eight loads in flight per wave: the step lives on their latency
      for (; q + 28 < t; q += 32) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = col[(long)(q + 4 * u) * nP];
#pragma unroll
        for (int u = 0; u < 8; u += 2) {
          d0 = fma(v[u], Lp[q + 4 * u], d0);
          d1 = fma(v[u + 1], Lp[q + 4 * u + 4], d1);
        }
      }
      for (; q + 4 < t; q += 8) {
        d0 = fma(col[(long)q * nP], Lp[q], d0);
        d1 = fma(col[(long)(q + 4) * nP], Lp[q + 4], d1);
      }
      if (q < t) d0 = fma(col[(long)q * nP], Lp[q], d0);
    }
    part[w][lane] = d0 + d1;
    __syncthreads();
    const double piv = rp > 0.0 ? rp : 0.0;
    const double root = sqrt(piv);
    const double dot = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    const double colv = (piv > 0.0 && i < n) ? (Gb[(long)p * nP + i] - dot) / root : 0.0;
    if (w == 0) Ltb[(long)t * nP + i] = colv;
    rho -= colv * colv;
    if (slot == 0 && tid == 0) { order[(long)b * k + t] = p; resid[(long)b * k + t] = (float)rp; }
  }
  if (!alive && slot == 0) {
    // a wait ran out: leave valid (distinct) positions and poisoned residuals behind
    const float qnan = __uint_as_float(0x7fc00000u);
    for (int t = tid; t < k; t += GT) { order[(long)b * k + t] = t; resid[(long)b * k + t] = qnan; }
    if (img_status && tid == 0) img_status[b] = 1;
  }
}

// One 1024-thread workgroup per image (no barriers between workgroups), left-looking: used when the batch alone
// fills the device and the picks are a small part of the rows (see the right-looking kernel below).
constexpr int RPT = 4;  // rows per thread: n <= 4096

__global__ __launch_bounds__(TPB) void greedy_single_kernel(const double* __restrict__ G, int n, int nP, int k,
                                                      double* __restrict__ Lt, int32_t* __restrict__ order,
                                                      float* __restrict__ resid) {
  __shared__ double Lp[4096];
  __shared__ unsigned long long red[16];
  __shared__ double sh_piv;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const double* Gb = G + (long)b * nP * nP;
  double* Ltb = Lt + (long)b * k * nP;

  double rho[RPT];
  bool picked[RPT];
#pragma unroll
  for (int s = 0; s < RPT; ++s) {
    const int i = tid + TPB * s;
    rho[s] = (i < n) ? Gb[(long)i * nP + i] : 0.0;
    picked[s] = !(i < n);
  }

  for (int t = 0; t < k; ++t) {
    // ---- argmax over the unpicked rows of float(rho), lowest index on ties
    unsigned long long best = 0ull;
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
      if (!picked[s]) {
        const uint32_t i = (uint32_t)(tid + TPB * s);
        unsigned long long key = ((unsigned long long)float_order_key((float)rho[s]) << 32) | (0xFFFFFFFFu - i);
        best = key > best ? key : best;
      }
    }
    best = wave_max(best);
    if (lane == 0) red[w] = best;
    __syncthreads();
    best = red[0];
#pragma unroll
    for (int q = 1; q < TPB / 64; ++q) best = red[q] > best ? red[q] : best;
    const int p = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));
    if ((p & (TPB - 1)) == tid) {
#pragma unroll
      for (int s = 0; s < RPT; ++s)
        if (s == (p >> 10)) { sh_piv = rho[s]; picked[s] = true; }
    }
    for (int s = tid; s < t; s += TPB) Lp[s] = Ltb[(long)s * nP + p];
    __syncthreads();
    const double rp = sh_piv;
    const double piv = rp > 0.0 ? rp : 0.0;
    const double root = sqrt(piv);
    double dot[RPT];
#pragma unroll
    for (int s = 0; s < RPT; ++s) dot[s] = 0.0;
    // The columns picked so far are re-read from L2 / the memory-side cache at every step; the step lives on the
    // latency of those loads, so sixteen of them are issued before the first is used.
    {
      constexpr int UQ = 16;
      int q = 0;
      for (; q + UQ <= t; q += UQ) {
#pragma unroll
        for (int s = 0; s < RPT; ++s) {
          if (tid + TPB * s < n) {
            double v[UQ];
#pragma unroll
            for (int u = 0; u < UQ; ++u) v[u] = Ltb[(long)(q + u) * nP + tid + TPB * s];
            double d0 = 0.0, d1 = 0.0;
#pragma unroll
            for (int u = 0; u < UQ; u += 2) {
              d0 = fma(v[u], Lp[q + u], d0);
              d1 = fma(v[u + 1], Lp[q + u + 1], d1);
            }
            dot[s] += d0 + d1;
          }
        }
      }
      for (; q < t; ++q) {
        const double lp = Lp[q];
        const double* row = Ltb + (long)q * nP + tid;
#pragma unroll
        for (int s = 0; s < RPT; ++s)
          if (tid + TPB * s < n) dot[s] = fma(row[TPB * s], lp, dot[s]);
      }
    }
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
      const int i = tid + TPB * s;
      if (i < n) {
        const double col = piv > 0.0 ? (Gb[(long)p * nP + i] - dot[s]) / root : 0.0;
        Ltb[(long)t * nP + i] = col;
        rho[s] -= col * col;
      }
    }
    if (tid == 0) { order[(long)b * k + t] = p; resid[(long)b * k + t] = (float)rp; }
    __syncthreads();  // Lp, sh_piv and red are rewritten next step; Lt row t must be visible to all
  }
}

// Right-looking in blocks of 16 picks (BK in what both of these kernels use), an image of up to 960 rows spread over W workgroups of 1024 threads
// (a thread owns a row).  The residual matrix R = G - L L^T is kept in global memory IN PLACE of G and
// brought up to date once per block by a rank-BK update on the MFMA; inside a block a new column is the pivot's
// row of R minus the product with the block's earlier columns, which live in LDS.  The left-looking kernels above
// re-read every earlier column at every step (k^2 n / 2 values); this one reads one row of R per step and reads
// and writes R once per block (up to 2 n^2 k / BK values), which is less unless k is a small part of n.
// Every workgroup of the image runs the BK picks of a block redundantly (same loads, same arithmetic, hence the
// same decisions: nothing is exchanged), then the workgroups meet at the image's barrier, each brings its own
// 16-row bands of R up to date, and they meet again before the next block reads rows of R: two barriers per
// block instead of one per pick, and the device's bandwidth on the update instead of one workgroup's.
// Picks are made in runs.  A residual only ever shrinks, so while the largest residual of the 64 largest ones at the start of the
// run stays above all the others as they were then, the others need not be looked at: one wave makes the picks from the
// 64 x 64 submatrix of R in LDS, no barrier and no row of R to wait for, and the columns of the run are formed for all rows
// behind it, the rows of R requested together.  A run ends when a residual left out could be the largest (6.3 to 7 picks on the
// average on the token matrices of the workloads, 5 to 10 over their images), at the end of a block, and
// before a residual that is not finite.  Residuals are compared with their rows, so that a tie ends no run that goes on in lower rows
// (300 rows of one length, orthogonal, 150 picks, us: 414 with a step per pick, 1330 with every tie the end of a run, 340 so).
// Candidates are the 64 largest of the eight largest of each wave; ordered by (residual rounded to fp32, lower row), so that the
// first pick of a run is the largest of all whatever ties there are.
// Bound by the chain of picks: us for 463 picks of 926 rows, six images, with all rows in every step (a maximum over the
// workgroup, the pivot's row from memory and a barrier per pick) 1842, so 1470 (66 to 73
// runs of 11 us and 28 updates of R of 20, both bound by latency and the memory-side cache).
// Dynamic LDS: 16 * nP + 64 * 65 doubles; workgroups take (image, slot) from the ticket counter.

// Maximum of one 32-bit key per lane over the wave with DPP moves (no LDS round trips): quads, then shifts by 4 and
// 8 inside a row of 16 lanes, then the last lane of a row broadcast into the next row (rows 1 and 3) and lane 31
// into rows 2 and 3, which leaves the maximum in lane 63.  Lanes without a source take 0, the identity for keys.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t max_dpp(uint32_t v) {
  const uint32_t o = __builtin_amdgcn_update_dpp(0u, v, CTRL, ROW_MASK, 0xf, false);
  return o > v ? o : v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max_dpp<0xb1, 0xf>(v);       // quad_perm [1,0,3,2]
  v = max_dpp<0x4e, 0xf>(v);       // quad_perm [2,3,0,1]
  v = max_dpp<0x114, 0xf>(v);      // row_shr:4
  v = max_dpp<0x118, 0xf>(v);      // row_shr:8
  v = max_dpp<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
  v = max_dpp<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
  return __builtin_amdgcn_readlane(v, 63);
}
// Lane of the largest key, of the lowest row among equal ones.
__device__ __forceinline__ int best_lane(uint32_t key, uint32_t best, uint32_t row) {
  unsigned long long tied = __ballot(key == best);
  if (__popcll(tied) > 1) {
    const uint32_t lowest = wave_max_u32(key == best ? 0xFFFFFFFFu - row : 0u);
    tied = __ballot(key == best && 0xFFFFFFFFu - row == lowest);
  }
  return __ffsll((long long)tied) - 1;
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Key of an unpicked row; 0 is below all of them.
__device__ __forceinline__ uint32_t residual_key(double rho) {
  const uint32_t u = float_order_key((float)rho);
  return u > 1u ? u : 1u;
}
constexpr uint32_t kKeyInf = 0xFF800000u;       // of +infinity; those of NaNs with a clear sign lie above
constexpr int kWaveBest = 8;                    // keys a wave posts
constexpr int kRunBlock = 16, kCand = 64;       // picks of a block, candidates of a run

struct GreedyRun {
  unsigned long long post[TPB / 64 * kWaveBest];   // per wave its largest keys: (residual, ~row), 0 where there are no more rows
  double post_rho[TPB / 64 * kWaveBest];
  int rank[TPB / 64 * kWaveBest];
  uint32_t left[TPB / 64];                         // per wave the largest key it did not post, and the lowest row that has it
  int left_row[TPB / 64];
  unsigned long long next;                         // the largest key posted that is no candidate
  int cand[kCand];
  double cand_rho[kCand];
  double factor[kRunBlock * kRunBlock];            // [q][m]: column q of the run at the row of its pick m
  double rho[kRunBlock];                           // of the picks
  double inverse[kRunBlock];                       // of their square roots; -1: nothing left of the row, its column is zero
  int pick[kRunBlock];
  int picks;
  int flag;
};

// The lowest row of those left out that have the key `bound`, by one wave.
__device__ __forceinline__ int lowest_left_out(const GreedyRun& run, uint32_t bound) {
  const int lane = threadIdx.x & 63;
  uint32_t after = 0u;                             // all ones minus the row
  if (lane < TPB / 64 && run.left[lane] == bound) after = 0xFFFFFFFFu - (uint32_t)run.left_row[lane];
  if (lane == TPB / 64 && (uint32_t)(run.next >> 32) == bound) after = (uint32_t)run.next;
  return (int)(0xFFFFFFFFu - wave_max_u32(after));
}

// Pick m of a run and those after it, by one wave; a lane has one candidate.  col[q] is column q of the run at its row.  bound is the
// largest residual left out; it goes before a candidate of the same residual in a later row.
template <int M>
__device__ __forceinline__ int run_picks(const double* S, GreedyRun& run, int room, uint32_t bound, uint32_t row, double rho, bool open, double (&col)[kRunBlock]) {
  if constexpr (M < kRunBlock) {
    if (M >= room) return M;
    const int lane = threadIdx.x & 63;
    const uint32_t key = open ? residual_key(rho) : 0u;
    const uint32_t best = wave_max_u32(key);
    if (best == 0u || (M > 0 && (best < bound || best >= kKeyInf))) return M;
    const int at = __builtin_amdgcn_readfirstlane(best_lane(key, best, row));
    if (M > 0 && best == bound && __builtin_amdgcn_readlane((int)row, at) > lowest_left_out(run, bound)) return M;
    double c = S[at * (kCand + 1) + lane];
    const double piv = lane_value(rho, at);
    const double inverse = piv > 0.0 ? 1.0 / sqrt(piv) : -1.0;
    double taken = 0.0;
#pragma unroll
    for (int q = 0; q < M; ++q) taken = fma(col[q], lane_value(col[q], at), taken);
    if (lane == at) {
      run.pick[M] = (int)row;
      run.rho[M] = piv;
      run.inverse[M] = inverse;
#pragma unroll
      for (int q = 0; q < M; ++q) run.factor[q * 16 + M] = col[q];
      open = false;
    }
    c -= taken;
    col[M] = inverse < 0.0 ? 0.0 : c * inverse;
    rho -= col[M] * col[M];
    if (best >= kKeyInf) return M + 1;
    return run_picks<M + 1>(S, run, room, bound, row, rho, open, col);
  }
  return M;
}

// c[m] -= l factor_m for the picks m of a run, the factors in lane m of every row of 16 lanes; and the columns of the run themselves
template <int FROM, int M>
__device__ __forceinline__ void take_out(double (&c)[kRunBlock], double l, double factors) {
  if constexpr (M < kRunBlock) {
    if constexpr (M >= FROM) c[M] = fma(-l, row_lane<M>(factors), c[M]);
    take_out<FROM, M + 1>(c, l, factors);
  }
}
template <int M>
__device__ __forceinline__ void run_columns(double (&c)[kRunBlock], const GreedyRun& run, int picks, double inverses, double& rho) {
  if constexpr (M < kRunBlock) {
    if (M >= picks) return;
    const double inverse = row_lane<M>(inverses);
    c[M] = inverse < 0.0 ? 0.0 : c[M] * inverse;
    rho -= c[M] * c[M];
    if constexpr (M + 1 < kRunBlock) take_out<M + 1, 0>(c, c[M], run.factor[M * 16 + (threadIdx.x & 15)]);
    run_columns<M + 1>(c, run, picks, inverses, rho);
  }
}

// End of a block of BK picks: the workgroups of the image meet, each brings its bands of R up to date, R -= Lblk^T Lblk, and they meet
// again; Lblk is cleared.  False when a wait ran out.
template <int BK>
__device__ __forceinline__ bool update_rows(double* R, double* Lblk, int n, int nP, int W, int slot, ImageBarrier* bar, unsigned int& target, int* s_flag,
                                            long long limit_ticks) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  // every workgroup of the image has read its last row of the old R (the wait starts with a barrier of
  // the workgroup, behind which the block's columns are complete in LDS)
  target += (unsigned int)W;
  if (!image_barrier_wait<false>(bar, target, s_flag, limit_ticks)) return false;
  // ---- R -= Lblk^T Lblk on this workgroup's bands (band ti belongs to slot ti % W); a wave takes four
  //      neighbouring 16 x 16 tiles per trip and requests their 16 values of R before the first MFMA
  const int nt = (n + 15) >> 4;
  const int bands = (nt - slot + W - 1) / W;
  const int ntiles = bands * nt;
  for (int tile0 = 4 * w; tile0 < ntiles; tile0 += 4 * (TPB / 64)) {
    double* out[4];
    double r[4][4];
    int ti[4], tj[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tile = tile0 + u;
      const int tc = tile < ntiles ? tile : tile0;          // a trailing slot repeats the first tile, result unused
      const int band = tc / nt;
      ti[u] = slot + band * W;
      tj[u] = tc - band * nt;
      // lane (i16, kq), register v: row 16 ti + 4v + kq, column 16 tj + i16 (inside the nP x nP buffer: nP % 64 == 0)
      out[u] = R + (long)(16 * ti[u] + kq) * nP + 16 * tj[u] + i16;
#pragma unroll
      for (int v = 0; v < 4; ++v) r[u][v] = out[u][(long)(4 * v) * nP];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      f64x4_t d = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s4 = 0; s4 < BK / 4; ++s4)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(Lblk[(4 * s4 + kq) * nP + 16 * ti[u] + i16], Lblk[(4 * s4 + kq) * nP + 16 * tj[u] + i16], d,
                                                 0, 0, 0);
      if (tile0 + u < ntiles) {
        // through the L2, so that the barrier has nothing to write back (6 of 26 us per update of six images of 926 rows)
#pragma unroll
        for (int v = 0; v < 4; ++v) store_through(out[u] + (long)(4 * v) * nP, r[u][v] - d[v]);
      }
    }
  }
  // every band is up to date before any workgroup reads a row of R again
  target += (unsigned int)W;
  if (!image_barrier_wait<false>(bar, target, s_flag, limit_ticks)) return false;
  for (int e = tid; e < BK * nP; e += TPB) Lblk[e] = 0.0;
  __syncthreads();
  return true;
}

__global__ __launch_bounds__(TPB) void greedy_panel_kernel(double* G, int n, int nP, int k, int W, int32_t* __restrict__ order,
                                                            float* __restrict__ resid, GreedyCtl* ctl, int* img_status,
                                                            long long limit_ticks) {
  extern __shared__ double Lblk[];        // [kRunBlock][nP], then [kCand][kCand + 1]
  __shared__ GreedyRun run;
  double* S = Lblk + (size_t)kRunBlock * nP;
  constexpr int BK = kRunBlock, CAND = kCand, POSTS = TPB / 64 * kWaveBest;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  if (tid == 0) run.flag = (int)atomicAdd(&ctl[0].ticket, 1u);
  __syncthreads();
  const int ticket = run.flag;
  __syncthreads();
  const int b = ticket / W, slot = ticket - b * W;
  GreedyCtl* cb = ctl + b;
  double* R = G + (long)b * nP * nP;
  // Row of this thread.  Few rows are dealt to all waves, sixteen neighbours (a 128-byte piece of a row of R) at a time: of the rows of one
  // wave only eight become candidates.
  const int i = n <= TPB / 2 ? (lane >> 4) * (TPB / 4) + 16 * w + i16 : tid;

  double rho = i < n ? R[(long)i * nP + i] : 0.0;
  bool picked = !(i < n);
  for (int e = tid; e < BK * nP; e += TPB) Lblk[e] = 0.0;
  unsigned int target = 0;
  bool alive = true;
  // the diagonal is read above and R is first written at the end of block 0, behind a barrier

  int jj = 0;                              // columns of the block so far
  for (int t = 0; t < k;) {
    // ---- the largest keys of each wave
    {
      uint32_t key = picked ? 0u : residual_key(rho);
#pragma unroll 1
      for (int e = 0; e <= kWaveBest; ++e) {
        const uint32_t best = wave_max_u32(key);
        if (e == kWaveBest) {
          if (lane == 0) run.left[w] = best;
          if (lane == __ffsll((long long)__ballot(key == best)) - 1) run.left_row[w] = i;        // lower lanes have lower rows
        } else if (best == 0u) {
          if (lane == 0) run.post[kWaveBest * w + e] = 0ull;
        } else if (lane == best_lane(key, best, (uint32_t)i)) {
          run.post[kWaveBest * w + e] = ((unsigned long long)best << 32) | (0xFFFFFFFFu - (uint32_t)i);
          run.post_rho[kWaveBest * w + e] = rho;
          key = 0u;
        }
      }
    }
    if (tid < POSTS) run.rank[tid] = 0;
    if (tid < CAND) run.cand[tid] = -1;
    if (tid == 0) run.next = 0ull;
    __syncthreads();
    // ---- their ranks: eight threads per key, sixteen comparisons each
    const unsigned long long key = run.post[tid & (POSTS - 1)];
    {
      int above = 0;
#pragma unroll
      for (int e = 0; e < POSTS / 8; ++e) above += run.post[(tid / POSTS) * (POSTS / 8) + e] > key ? 1 : 0;
      if (above) atomicAdd(&run.rank[tid & (POSTS - 1)], above);
    }
    __syncthreads();
    if (tid < POSTS && key != 0ull) {
      const int rank = run.rank[tid];
      if (rank < CAND) {
        run.cand[rank] = (int)(0xFFFFFFFFu - (uint32_t)key);
        run.cand_rho[rank] = run.post_rho[tid];
      } else if (rank == CAND) {
        run.next = key;
      }
    }
    __syncthreads();
    // ---- R between the candidates: 16 x 16 tiles on and below the diagonal, minus what this block has already taken out
    {
      constexpr int PT = CAND / 16;
      const int ti = w / PT, tj = w % PT;
      if (w < PT * PT && tj <= ti) {
        const int cc = run.cand[16 * tj + i16], col = cc < 0 ? 0 : cc, ar = run.cand[16 * ti + i16], arow = ar < 0 ? 0 : ar;
        double r[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int cr = run.cand[16 * ti + 4 * v + kq];
          r[v] = R[(long)(cr < 0 ? 0 : cr) * nP + col];
        }
        f64x4_t d = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s4 = 0; s4 < BK / 4; ++s4)
          if (4 * s4 < jj) d = __builtin_amdgcn_mfma_f64_16x16x4f64(Lblk[(4 * s4 + kq) * nP + arow], Lblk[(4 * s4 + kq) * nP + col], d, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * ti + 4 * v + kq, c = 16 * tj + i16;
          S[a * (CAND + 1) + c] = r[v] - d[v];
          if (ti != tj) S[c * (CAND + 1) + a] = r[v] - d[v];
        }
      }
    }
    __syncthreads();
    // ---- the run
    if (w == 0) {
      uint32_t bound = lane < TPB / 64 ? run.left[lane] : lane == TPB / 64 ? (uint32_t)(run.next >> 32) : 0u;
      bound = wave_max_u32(bound);
      const int row = run.cand[lane];
      double col[BK];
      const int room = BK - jj < k - t ? BK - jj : k - t;
      const int picks = run_picks<0>(S, run, room, bound, (uint32_t)row, row < 0 ? 0.0 : run.cand_rho[lane], row >= 0, col);
      if (lane == 0) run.picks = picks;
    }
    __syncthreads();
    const int picks = run.picks;
    if (picks < 1) {                      // no row left: cannot be, k <= n
      if (tid == 0) __hip_atomic_store(&cb->bar.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      alive = false;
      break;
    }
    if (slot == 0 && tid < picks) {
      order[(long)b * k + t + tid] = run.pick[tid];
      resid[(long)b * k + t + tid] = (float)run.rho[tid];
    }
    // ---- its columns for all rows
    {
      const int mine = i16 < picks ? run.pick[i16] : run.pick[0];      // of the run's pick i16
      const double inverses = i16 < picks ? run.inverse[i16] : -1.0;
      double c[BK];
#pragma unroll
      for (int m = 0; m < BK; ++m) {
        c[m] = 0.0;
        if (m < picks) {
          const int p = __builtin_amdgcn_readlane(mine, m);
          if (i < n) c[m] = R[(long)p * nP + i];
          if (p == i) picked = true;
        }
      }
      for (int q = 0; q < jj; ++q) take_out<0, 0>(c, i < n ? Lblk[q * nP + i] : 0.0, Lblk[q * nP + mine]);
      run_columns<0>(c, run, picks, inverses, rho);
#pragma unroll
      for (int m = 0; m < BK; ++m)
        if (m < picks && i < nP) Lblk[(jj + m) * nP + i] = c[m];
    }
    t += picks;
    jj += picks;
    if (jj == BK && t < k) {
      jj = 0;
      alive = update_rows<BK>(R, Lblk, n, nP, W, slot, &cb->bar, target, &run.flag, limit_ticks);
      if (!alive) break;
    }
  }
  if (!alive && slot == 0) {
    // a wait ran out: leave valid (distinct) positions and poisoned residuals behind
    const float qnan = __uint_as_float(0x7fc00000u);
    for (int t = tid; t < k; t += TPB) { order[(long)b * k + t] = t; resid[(long)b * k + t] = qnan; }
    if (img_status && tid == 0) img_status[b] = 1;
  }
}

// The same for 64-bit keys.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned long long dpp_key(unsigned long long v) {
  const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)v, CTRL, ROW_MASK, 0xf, false);
  const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(v >> 32), CTRL, ROW_MASK, 0xf, false);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long v) {
  unsigned long long o;
  o = dpp_key<0xb1, 0xf>(v); v = o > v ? o : v;      // quad_perm [1,0,3,2]
  o = dpp_key<0x4e, 0xf>(v); v = o > v ? o : v;      // quad_perm [2,3,0,1]
  o = dpp_key<0x114, 0xf>(v); v = o > v ? o : v;     // row_shr:4
  o = dpp_key<0x118, 0xf>(v); v = o > v ? o : v;     // row_shr:8
  o = dpp_key<0x142, 0xa>(v); v = o > v ? o : v;     // row_bcast:15 into rows 1 and 3
  o = dpp_key<0x143, 0xc>(v); v = o > v ? o : v;     // row_bcast:31 into rows 2 and 3
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)v, 63), hi = __builtin_amdgcn_readlane((unsigned)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}

// The same with all rows in every step, in blocks of BK picks (dynamic LDS: BK * nP doubles), for images of up to 4096 rows (a thread owns NR of
// them, 1024 apart), whose candidates' submatrix would cost LDS that the block's columns need: see launch_greedy.
template <int BK, int NR>
__global__ __launch_bounds__(TPB) void greedy_step_kernel(double* G, int n, int nP, int k, int W, int32_t* __restrict__ order,
                                                            float* __restrict__ resid, GreedyCtl* ctl, int* img_status,
                                                            long long limit_ticks) {
  extern __shared__ double Lblk[];        // [BK][nP]
  __shared__ unsigned long long red[2][16];   // per wave: its best key and that row's residual, double-buffered by
  __shared__ double red_rho[2][16];           // step parity so that a step needs one barrier only
  __shared__ int s_flag;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_flag = (int)atomicAdd(&ctl[0].ticket, 1u);
  __syncthreads();
  const int ticket = s_flag;
  __syncthreads();
  const int b = ticket / W, slot = ticket - b * W;
  GreedyCtl* cb = ctl + b;
  double* R = G + (long)b * nP * nP;

  double rho[NR];
  bool picked[NR];
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    const int i = tid + TPB * s;
    rho[s] = (i < n) ? R[(long)i * nP + i] : 0.0;
    picked[s] = !(i < n);
  }
  for (int e = tid; e < BK * nP; e += TPB) Lblk[e] = 0.0;
  unsigned int target = 0;
  bool alive = true;
  // the diagonal is read above and R is first written at the end of block 0, behind a barrier
  __syncthreads();

  for (int t = 0; t < k; ++t) {
    const int jj = t % BK, par = t & 1;
    // ---- argmax over the unpicked rows of float(rho), lowest index on ties.  Keys are distinct, so exactly one
    //      lane of a wave holds the wave's best and posts it with its residual.  One barrier per step: what a
    //      step writes besides is read only behind the next step's barrier, and the posts alternate buffers.
    unsigned long long best = 0ull;
    double brho = 0.0;
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (!picked[s]) {
        const unsigned long long key =
            ((unsigned long long)float_order_key((float)rho[s]) << 32) | (0xFFFFFFFFu - (uint32_t)(tid + TPB * s));
        if (key > best) { best = key; brho = rho[s]; }
      }
    }
    {
      const unsigned long long wbest = wave_max_key(best);
      if (wbest == 0ull) { if (lane == 0) red[par][w] = 0ull; }
      else if (best == wbest) { red[par][w] = wbest; red_rho[par][w] = brho; }
    }
    __syncthreads();
    best = red[par][0];
    int wq = 0;
#pragma unroll
    for (int q = 1; q < TPB / 64; ++q)
      if (red[par][q] > best) { best = red[par][q]; wq = q; }
    const double rp = red_rho[par][wq];
    const int p = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));     // < n: k <= n, so an unpicked row exists
    if (best == 0ull || (unsigned)p >= (unsigned)n) {   // never index with anything else
      if (tid == 0) __hip_atomic_store(&cb->bar.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      alive = false;
      break;
    }
    if ((p & (TPB - 1)) == tid) {
#pragma unroll
      for (int s = 0; s < NR; ++s)
        if (s == (p >> 10)) picked[s] = true;
    }
    // ---- the pivot's row of R, minus what this block has already taken out (summed apart, so that the sum
    //      does not wait for the row)
    double c[NR];
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      const int i = tid + TPB * s;
      c[s] = (i < n) ? R[(long)p * nP + i] : 0.0;
    }
    {
      double taken[NR];
#pragma unroll
      for (int s = 0; s < NR; ++s) taken[s] = 0.0;
      for (int q = 0; q < jj; ++q) {
        const double lp = Lblk[q * nP + p];
#pragma unroll
        for (int s = 0; s < NR; ++s) {
          const int i = tid + TPB * s;
          if (i < n) taken[s] = fma(Lblk[q * nP + i], lp, taken[s]);
        }
      }
#pragma unroll
      for (int s = 0; s < NR; ++s) c[s] -= taken[s];
    }
    const double piv = rp > 0.0 ? rp : 0.0;
    const double root = sqrt(piv);
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      const int i = tid + TPB * s;
      const double col = (piv > 0.0 && i < n) ? c[s] / root : 0.0;
      if (i < nP) Lblk[jj * nP + i] = col;
      rho[s] -= col * col;
    }
    if (slot == 0 && tid == 0) { order[(long)b * k + t] = p; resid[(long)b * k + t] = (float)rp; }
    if (jj == BK - 1 && t + 1 < k) {
      alive = update_rows<BK>(R, Lblk, n, nP, W, slot, &cb->bar, target, &s_flag, limit_ticks);
      if (!alive) break;
    }
  }
  if (!alive && slot == 0) {
    // a wait ran out: leave valid (distinct) positions and poisoned residuals behind
    const float qnan = __uint_as_float(0x7fc00000u);
    for (int t = tid; t < k; t += TPB) { order[(long)b * k + t] = t; resid[(long)b * k + t] = qnan; }
    if (img_status && tid == 0) img_status[b] = 1;
  }
}

// idx_out[b,:] = ascending positions idx_m[b, picked]; pick_out[b,t] = idx_m[b, order[b,t]]
__global__ __launch_bounds__(TPB) void greedy_finish_kernel(const int32_t* __restrict__ order, const int32_t* __restrict__ idx_m,
                                                             int M, int k, int32_t* __restrict__ idx_out,
                                                             int32_t* __restrict__ pick_out) {
  __shared__ unsigned char flag[4096];
  __shared__ int wsum[17];
  const int b = blockIdx.x, tid = threadIdx.x;
  for (int i = tid; i < M; i += TPB) flag[i] = 0;
  __syncthreads();
  for (int t = tid; t < k; t += TPB) {
    const int p = order[(long)b * k + t];
    flag[p] = 1;
    if (pick_out) pick_out[(long)b * k + t] = idx_m[(long)b * M + p];
  }
  __syncthreads();
  const int per = (M + TPB - 1) / TPB, i0 = tid * per;
  int cnt = 0;
  for (int q = 0; q < per; ++q) { const int i = i0 + q; if (i < M && flag[i]) ++cnt; }
  int total;
  int pos = block_exscan_1024(cnt, wsum, &total);
  for (int q = 0; q < per; ++q) {
    const int i = i0 + q;
    if (i < M && flag[i]) idx_out[(long)b * k + pos++] = idx_m[(long)b * M + i];
  }
}

}  // namespace

size_t greedy_ctl_bytes(int B) { return (size_t)B * sizeof(GreedyCtl); }
size_t greedy_scratch_bytes(int B, int nP) {
  return (size_t)B * sizeof(GreedyCtl) + 256 + (size_t)B * 4 * (nP / GR) * 8;
}

// Columns of a block of BK picks and the candidates' submatrix, beside the kernel's static words.
constexpr size_t kRunLds = 160 * 1024 - sizeof(GreedyRun) - 256, kStepLds = 159 * 1024;
static size_t run_lds(int nP) { return ((size_t)kRunBlock * nP + (size_t)kCand * (kCand + 1)) * sizeof(double); }

template <typename K>
static hipError_t launch_panel(K kernel, PerDeviceInt& raised, PerDeviceInt& cache, size_t lds, size_t most, double* G, int B, int n, int nP, int k, int W,
                               int32_t* order, float* resid, GreedyCtl* ctl, int* img_status, hipStream_t st) {
  if (lds > most) return hipErrorInvalidValue;
  hipError_t e = ensure_dynamic_lds(raised, (const void*)kernel, most);
  if (e != hipSuccess) return e;
  // the workgroups of one image wait for one another, so one image has to fit the device; counted once per device
  // for the largest LDS request, which never overstates what a smaller one gets
  int capacity = 0;
  if ((e = resident_workgroups(cache, kernel, TPB, most, &capacity)) != hipSuccess) return e;
  if (W > capacity) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(B * W)), dim3(TPB), lds, st, G, n, nP, k, W, order, resid, ctl, img_status, barrier_limit_ticks());
  return hipGetLastError();
}

hipError_t launch_greedy(double* G, int B, int n, int nP, int k, double* Lt, int32_t* order, float* resid, void* scratch,
                         int* img_status, hipStream_t st) {
  if (nP % GR != 0 || n > nP || n > 4096 || k > n || k > 4096) return hipErrorInvalidValue;
  GreedyCtl* ctl = (GreedyCtl*)scratch;
  // the largest block of picks (a multiple of the MFMA's depth of 4) whose columns fit LDS
  const auto fits = [&](int bk) { return (size_t)bk * nP * sizeof(double) <= kStepLds; };
  const int BK = fits(16) ? 16 : fits(12) ? 12 : fits(8) ? 8 : 4;
  // values moved: the right-looking kernel reads and writes R once per block that is followed by another, the
  // left-looking ones read every earlier column at every step; the former also has far fewer barriers
  const double right = (double)((k - 1) / BK) * 2.0 * n * n, left = 0.5 * k * k * n;
  if (right <= 2.0 * left) {
    // workgroups per image: measured best with about 128 on the device, at most 32 and (while they fit) at least 4 per image
    const int nt = (n + 15) / 16;
    int Wp = 128 / B;
    if (Wp < 4) Wp = 256 / B < 4 ? 256 / B : 4;
    Wp = Wp < 1 ? 1 : Wp > 32 ? 32 : Wp;
    Wp = Wp > nt ? nt : Wp;
    // Runs of picks up to 960 rows, where the candidates' submatrix fits beside 16 columns.  us per selection of half of the rows, steps (before R was
    // stored through) / runs, one image and eight: 64 rows 147 / 101 and 152 / 112, 128 228 / 154 and 237 / 176, 512 751 / 567 and 910 / 677,
    // 900 1544 / 1213 and 2124 / 1594.  Beyond, runs cost the updates that a smaller block adds or most of their candidates: 1000 rows
    // 1740 / 1760 and 2400 / 2350 with 12 columns, 2160 and 2650 with 32 candidates, 2400 rows 11700 / 18900 with 4 columns.
#define COVSPEC_PANEL(kernel, lds, most)                                                                                                        \
  do {                                                                                                                                          \
    static PerDeviceInt raised, cache;                                                                                                          \
    return launch_panel(kernel, raised, cache, lds, most, G, B, n, nP, k, Wp, order, resid, ctl, img_status, st);                               \
  } while (0)
    if (run_lds(nP) <= kRunLds) COVSPEC_PANEL(greedy_panel_kernel, run_lds(nP), kRunLds);
    const size_t lds = (size_t)BK * nP * sizeof(double);
    // rows per thread: at most 1216 rows with blocks of 16, 1664 with 12, 2496 with 8
    if (BK == 16 && n <= TPB) COVSPEC_PANEL((greedy_step_kernel<16, 1>), lds, kStepLds);
    if (BK == 16) COVSPEC_PANEL((greedy_step_kernel<16, 2>), lds, kStepLds);
    if (BK == 12) COVSPEC_PANEL((greedy_step_kernel<12, 2>), lds, kStepLds);
    if (BK == 8 && n <= 2 * TPB) COVSPEC_PANEL((greedy_step_kernel<8, 2>), lds, kStepLds);
    if (BK == 8) COVSPEC_PANEL((greedy_step_kernel<8, 4>), lds, kStepLds);
    COVSPEC_PANEL((greedy_step_kernel<4, 4>), lds, kStepLds);
#undef COVSPEC_PANEL
  }
  const int W = nP / GR;
  // Left-looking: spreading an image over W workgroups costs a device-scope barrier per step; it pays while the
  // batch leaves most of the device idle.
  if ((long)B * W > 256) {
    hipLaunchKernelGGL(greedy_single_kernel, dim3(B), dim3(TPB), 0, st, G, n, nP, k, Lt, order, resid);
    return hipGetLastError();
  }
  // the workgroups of one image wait for one another, so one image has to fit the device
  static PerDeviceInt cache;
  int capacity = 0;
  const hipError_t ec = resident_workgroups(cache, greedy_kernel, GT, 0, &capacity);
  if (ec != hipSuccess) return ec;
  if (W > capacity) return hipErrorInvalidValue;
  unsigned long long* posts = (unsigned long long*)((char*)scratch + (((size_t)B * sizeof(GreedyCtl) + 255) / 256) * 256);
  hipLaunchKernelGGL(greedy_kernel, dim3((unsigned)(B * W)), dim3(GT), 0, st, G, n, nP, k, Lt, order, resid, ctl, posts,
                     img_status, barrier_limit_ticks());
  return hipGetLastError();
}

hipError_t launch_greedy_finish(const int32_t* order, const int32_t* idx_m, int B, int M, int k, int32_t* idx_out,
                                int32_t* pick_out, hipStream_t st) {
  if (M > 4096) return hipErrorInvalidValue;
  hipLaunchKernelGGL(greedy_finish_kernel, dim3(B), dim3(TPB), 0, st, order, idx_m, M, k, idx_out, pick_out);
  return hipGetLastError();
}

}  // namespace covspec
