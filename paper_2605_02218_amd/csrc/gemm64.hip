// fp64 MFMA GEMM:  C[M,N] (fp64) = A[M,K] * B[N,K]^T with A, B stored as fp64, fp32 or bf16 and every product and sum
// taken in fp64 on v_mfma_f64_16x16x4_f64.
//
// Two users.  (1) The fp32-input path: fp32 inputs carry 24-bit mantissas, so an fp32-accumulated contraction cannot deliver
// cosine scores to 1e-5 relative once the cosine is small against its natural scale; that workload is small, so its whole
// chain (embeddings, folded query matrix, inner products, norms, Gram matrix) runs here and the fp32 storage is the only
// rounding left; so does the Gram matrix of the greedy picks from bf16 rows.  (2) The low-rank stage, whose block iteration on
// the fp64 Gram matrix is a sequence of fp64 products.
//
// Five kernels:
//   gemm64_kernel        any of the storage types, row lists, any K and alignment: 64 x 64 tiles, operands converted to fp64 on
//                        their way through registers into LDS.
//   gemm64_dma_kernel    fp64 x fp64 (the block iteration) and bf16 x bf16: direct-to-LDS loads, tiles of 64 x 96 to 32 x 32.
//   gemm64_tile16_kernel fp64 products of so few 16 x 16 tiles that a compute unit gets one at most
//   gemm64_small_kernel  few tiles and an fp32 operand, row lists: 32 x 32 or 16 x 16 tiles, k over the four waves, straight from global memory.
//   gemm64_sym_kernel    the products after the spectral split, whose left operand is symmetric and whose right one is [K][N].
// gemm64_kernel: 256 threads = 4 waves (2x2); wave tile (MI*16) x (NJ*16), block tile twice that in each direction (64x64
// for <2,2>), k-tile 16; the loads of k-tile t+1 are issued before the MFMAs of tile t and parked in registers, LDS is double
// buffered, one barrier per k-tile.
// MFMA layouts: operand lane l holds (row|col = l%16, k = l/16); result lane l, register v
// holds (row 4v + l/16, col l%16).
#include <type_traits>
#include "common.h"
#include "gemm64_tiles.h"
#include "host_cache.h"
#include "kernels.h"

namespace covspec {

namespace {

constexpr int TK = 16, PITCH = TK + 1;
// 64 x 64 tiles up to which gemm64_small_kernel is taken for operands that are not both fp64: up to one workgroup per compute unit
// of the alternative, the register-staged kernel with one wave per SIMD.  us, gemm64_kernel / here: row norms of 144 tiles (576 x 1024 x 1024) 136 / 34, 256
// (2000 x 512 x 512) 64 / 30, 288 (1100 x 1024 x 1024) 148 / 52, 864 of K = 256 57 / 57, 1008 59 / 68: the small tiles would still
// win up to some 800; the line is where the sums' order was drawn.
constexpr long kSmallTiles64 = 256;

__device__ __forceinline__ double as_f64(double v) { return v; }
__device__ __forceinline__ double as_f64(float v) { return (double)v; }
__device__ __forceinline__ double as_f64(bf16_t v) { return (double)bf16_to_f32(v); }

// Workgroups are handed to the 8 XCDs round-robin; regroup the ids so that an XCD works on consecutive
// tiles (same image, same operand rows) and its L2 keeps them.
__device__ __forceinline__ int regroup_xcd(int bid, int nblocks) {
  const int per = nblocks >> 3;
  return (bid < (per << 3)) ? (bid & 7) * per + (bid >> 3) : bid;
}

template <typename TA, typename TB, int EPI, bool GATHER, int MI, int NJ>
__global__ __launch_bounds__(256) void gemm64_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int TM = 32 * MI, TN = 32 * NJ;
  constexpr int SA = TM / 16, SBn = TN / 16;       // staged elements per thread and operand
  extern __shared__ double smem[];
  double* sA = smem;                               // [2][TM * PITCH]
  double* sB = smem + 2 * TM * PITCH;              // [2][TN * PITCH]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int per = tiles_m * tiles_n;
  const int gid = regroup_xcd(blockIdx.x, gridDim.x);
  const int bidx = gid / per;
  const int pidx = gid - bidx * per;
  const int tm = pidx / tiles_n, tn = pidx - tm * tiles_n;
  const int row0 = tm * TM, col0 = tn * TN;
  const int bo = bidx / g.batch_inner, bi = bidx - bo * g.batch_inner;
  if (g.skip && g.skip[bo] > g.skip_if) return;           // uniform per workgroup
  if (g.lower_only && col0 > row0 + TM - 1) return;       // tile entirely above the diagonal
  const TA* __restrict__ A = (const TA*)g.A + (long)bo * g.strideA + (long)bi * g.strideA2;
  const TB* __restrict__ B = (const TB*)g.B + (long)bo * g.strideB + (long)bi * g.strideB2;
  const long coff = (long)bo * g.strideC + (long)bi * g.strideC2;

  // staging slots: element e = tid + 256*s -> (row e/16, k e%16).
  long aoff[SA], boff[SBn];
  bool aok[SA], bok[SBn];
  const int lk = tid & 15;
#pragma unroll
  for (int s = 0; s < SA; ++s) {
    const int ra = row0 + (tid >> 4) + 16 * s;
    aok[s] = ra < g.M;
    long ia = ra;
    if (GATHER && g.gatherA && aok[s]) ia = g.gatherA[(long)bo * g.gstrideA + ra];
    aoff[s] = ia * g.lda + lk;
  }
#pragma unroll
  for (int s = 0; s < SBn; ++s) {
    const int rb = col0 + (tid >> 4) + 16 * s;
    bok[s] = rb < g.N;
    long ib = rb;
    if (GATHER && g.gatherB && bok[s]) ib = g.gatherB[(long)bo * g.gstrideB + rb];
    boff[s] = ib * g.ldb + lk;
  }

  // bf16 x bf16, both K-contiguous, 64 x 64 tiles: a k-tile of an operand is 64 rows x 32 bytes, so the
  // element-wise staging above would issue eight 2-byte loads per thread.  When rows and K allow 16-byte
  // pieces, thread t instead loads ONE piece (operand t / 128, row (t % 128) / 2, half t % 2) and converts its
  // eight values on the way into LDS.
  constexpr bool WIDE_T = std::is_same<TA, bf16_t>::value && std::is_same<TB, bf16_t>::value && MI == 2 && NJ == 2;
  const bool wide = WIDE_T && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.K % 8 == 0 && (((uintptr_t)A | (uintptr_t)B) & 15) == 0;
  const int wop = tid >> 7, wrow = (tid & 127) >> 1, whalf = tid & 1;
  long woff = 0;
  bool wok = false;
  if (WIDE_T && wide) {
    const int rr = (wop ? col0 : row0) + wrow;
    wok = rr < (wop ? g.N : g.M);
    long ir = rr;
    const int32_t* gl = wop ? g.gatherB : g.gatherA;
    if (GATHER && gl && wok) ir = gl[(long)bo * (wop ? g.gstrideB : g.gstrideA) + rr];
    woff = ir * (wop ? g.ldb : g.lda) + 8 * whalf;
  }
  u32x4_t rw = {0u, 0u, 0u, 0u};

  double ra_[SA], rb_[SBn];
  auto fetch = [&](int k0) {
    if (WIDE_T && wide) {
      const u32x4_t z = {0u, 0u, 0u, 0u};
      const bf16_t* P = wop ? (const bf16_t*)B : (const bf16_t*)A;
      rw = (wok && k0 + 8 * whalf < g.K) ? *(const u32x4_t*)(P + woff + k0) : z;
      return;
    }
#pragma unroll
    for (int s = 0; s < SA; ++s) ra_[s] = (aok[s] && k0 + lk < g.K) ? as_f64(A[aoff[s] + k0]) : 0.0;
#pragma unroll
    for (int s = 0; s < SBn; ++s) rb_[s] = (bok[s] && k0 + lk < g.K) ? as_f64(B[boff[s] + k0]) : 0.0;
  };
  auto park = [&](int buf) {
    if (WIDE_T && wide) {
      double* dst = (wop ? sB + buf * TN * PITCH : sA + buf * TM * PITCH) + wrow * PITCH + 8 * whalf;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dst[2 * e] = (double)__uint_as_float(rw[e] << 16);
        dst[2 * e + 1] = (double)__uint_as_float(rw[e] & 0xFFFF0000u);
      }
      return;
    }
    double* a = sA + buf * TM * PITCH;
    double* b = sB + buf * TN * PITCH;
#pragma unroll
    for (int s = 0; s < SA; ++s) a[((tid >> 4) + 16 * s) * PITCH + lk] = ra_[s];
#pragma unroll
    for (int s = 0; s < SBn; ++s) b[((tid >> 4) + 16 * s) * PITCH + lk] = rb_[s];
  };

  f64x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = (f64x4_t){0.0, 0.0, 0.0, 0.0};

  const int i16 = lane & 15, kq = lane >> 4;
  const int nt = (g.K + TK - 1) / TK;
  fetch(0);
  park(0);
  __syncthreads();
  for (int t = 0; t < nt; ++t) {
    if (t + 1 < nt) fetch((t + 1) * TK);
    const double* a = sA + (t & 1) * TM * PITCH + (wm * MI * 16 + i16) * PITCH + kq;
    const double* b = sB + (t & 1) * TN * PITCH + (wn * NJ * 16 + i16) * PITCH + kq;
#pragma unroll
    for (int ks = 0; ks < TK / 4; ++ks) {
      double af[MI], bf[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) af[i] = a[i * 16 * PITCH + ks * 4];
#pragma unroll
      for (int j = 0; j < NJ; ++j) bf[j] = b[j * 16 * PITCH + ks * 4];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    if (t + 1 < nt) park((t + 1) & 1);
    __syncthreads();
  }

  if (EPI == EPI_STORE_F64) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = row0 + wm * MI * 16 + i * 16 + 4 * v + kq;
          const int c = col0 + wn * NJ * 16 + j * 16 + i16;
          if (r < g.M && c < g.N) {
            double* out = (double*)g.C + coff + (long)r * g.ldc + c;
            *out = acc[i][j][v];
            // lanes of equal i16 hold four consecutive rows r: the transposed store goes out in 32-byte pieces
            if (g.mirror && tn != tm) ((double*)g.C)[coff + (long)c * g.ldc + r] = acc[i][j][v];
          }
        }
  } else {  // EPI_ROWNORM2: per-row sum over this tile's columns of C^2 (fp64)
    double* red = smem;   // [2][TM], reuses the operand buffers (all reads of them are behind the last barrier)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) s += acc[i][j][v] * acc[i][j][v];
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (i16 == 0) red[wn * TM + wm * MI * 16 + i * 16 + 4 * v + kq] = s;
      }
    __syncthreads();
    if (tid < TM) {
      const int r = row0 + tid;
      if (r < g.M) ((double*)g.C)[coff + (long)r * g.ldc + tn] = red[tid] + red[TM + tid];
    }
  }
}

// ---- fp64 x fp64, both K-contiguous, fp64 result (the products of the low-rank stage).  TM x TN tile, 2 x 2 waves, k-tile 16,
// operand tiles loaded straight into LDS as whole 128-byte rows (a ring of four stages, three k-tiles in flight, one barrier per
// k-tile), rows swizzled by their low three bits so that the 16-byte fragment reads (two k values per lane: any order of k serves as
// long as both operands have it) are conflict-free, the fragments of the next half k-tile read while the current one is
// multiplied.  KS = 2: a second group of four waves takes the other half of k in a ring of its own and the halves are added at the
// end, for problems with no more tiles than compute units, where one wave per SIMD cannot hide its own waits.
// Bound by the fp64 MFMA: a 64 x 64 tile keeps a compute unit busy for K / 32 us, so what decides is how evenly the tiles go into the
// compute units (launch_plain).  us with the tiles chosen there, and the time at the rate of a loop of nothing but these MFMAs (67.6
// TFLOP/s): 192 x 1664 x 1664, batch 4 72 (63; on tiles of 32 x 32, which read their operands at 20 TB/s from the L2s, 83); 384 x 1152 x
// 1152, batch 8 139 (121); 256 x 640 x 640, batch 64 218 (199); 192 x 1280 x 1280, batch 4 50 (37).
// A symmetric product (lower_only, frag; TM = TN) has a workgroup for each tile on and below its diagonal only.
// TS = bf16 (the Gram matrix of the greedy picks, row lists): the same 128-byte pieces of a row are 64 k, converted between LDS and
// MFMA, which the MFMAs hide.  Staged through registers and converted into LDS, one k-tile of 16 in flight, six of
// 926 x 926 x 2048 took 308 us, so 230.
// Requires whole k-tiles (16 or 64), pitches of whole pieces, 16-byte aligned bases.  Rows beyond M / N are clamped when loading.
// A Chebyshev step (GemmArgs::cheb) is scale * (A B + start): the accumulators begin with the terms that are not the product,
// whose loads are over before the first operands have landed (read behind the product they cost 30 of 260 us).
__device__ __forceinline__ double cheb_scale(const GemmArgs& g, double t) { return t == 0.0 ? 1.0 : g.cheb_step == 0 ? t : 2.0 * t; }
__device__ __forceinline__ double cheb_start(const GemmArgs& g, const double* A, const double* C, double rt, int r, int c) {   // rt = 1 / t
  const double a = A[(long)r * g.lda + c];
  return -rt * (g.cheb_step == 0 ? a : fma(0.5, C[(long)r * g.ldc + c], a));
}

// Bytes of a stage: whole loads of eight rows, as many for each wave.
constexpr int dma_stage(int TM, int TN) { return ((TM + TN) / 8 + 3) / 4 * 4 * 1024; }

// A 16-byte piece of a row and its elements as fp64.
template <typename TS> struct Piece;
template <> struct Piece<double> {
  typedef f64x2_t type;
  static __device__ __forceinline__ double at(const type& v, int e) { return v[e]; }
};
template <> struct Piece<bf16_t> {
  typedef u32x4_t type;
  static __device__ __forceinline__ double at(const type& v, int e) { return (double)__uint_as_float(e & 1 ? v[e >> 1] & 0xFFFF0000u : v[e >> 1] << 16); }
};

// WM: waves along the rows of the tile (the others along its columns).
template <typename TS, int KS, int TM, int TN, int WM>
__global__ __launch_bounds__(256 * KS, 2) void gemm64_dma_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int GROUPS = (TM + TN) / 8, LOADS = (GROUPS + 3) / 4;      // of eight rows, a load each: of a stage, and of a wave
  constexpr int NST = 4, STAGE = dma_stage(TM, TN);                    // bytes: A tile, then B tile, then what fills up the waves' loads
  constexpr int WN = 4 / WM, MI = TM / (16 * WM), NJ = TN / (16 * WN); // 16 x 16 tiles of a wave
  static_assert(TM % (16 * WM) == 0 && TN % (16 * WN) == 0 && TM % 8 == 0, "");
  constexpr int PE = 16 / sizeof(TS), KT = 8 * PE;  // elements of a piece and of a k-tile
  constexpr bool F64 = std::is_same<TS, double>::value;
  typedef typename Piece<TS>::type piece_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
  const int tid = threadIdx.x & 255, grp = threadIdx.x >> 8, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN, i16 = lane & 15, kq = lane >> 4;
  const bool triangle = TM == TN && (g.lower_only || g.frag);
  const int per = triangle ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int gid = regroup_xcd(blockIdx.x, gridDim.x);
  const int b = gid / per, pidx = gid - b * per;
  if (g.skip && g.skip[b] > g.skip_if) return;            // uniform per workgroup
  int tm, tn;
  if (triangle) {                                         // tile (x, y <= x) of the triangle; frag: its mirror image, see the store
    int x = (int)((sqrtf(8.0f * (float)pidx + 1.0f) - 1.0f) * 0.5f);
    while (x * (x + 1) / 2 > pidx) --x;
    while ((x + 1) * (x + 2) / 2 <= pidx) ++x;
    const int y = pidx - x * (x + 1) / 2;
    tm = g.frag ? y : x;
    tn = g.frag ? x : y;
  } else {
    tm = pidx / tiles_n;
    tn = pidx - tm * tiles_n;
  }
  const int row0 = tm * TM, col0 = tn * TN;
  const bool moved = g.sel && g.sel[b];
  const TS* A = (const TS*)g.A + (long)b * g.strideA + (moved ? g.selA : 0);
  const TS* B = (const TS*)g.B + (long)b * g.strideB + (moved ? g.selB : 0);
  const int nk = g.K / KT, nk0 = (nk + KS - 1) / KS, kt0 = grp * nk0;
  const int mine = nk - kt0 < nk0 ? (nk - kt0 > 0 ? nk - kt0 : 0) : nk0;      // k-tiles of this group

  // load j of wave w fills the eight rows of group LOADS w + j of the stage: lane l -> row l / 8, 16-byte slot l % 8, which holds the row's
  // piece (l % 8) ^ (row % 8)
  const TS* src[LOADS];
  const int lr = lane >> 3, lc = PE * ((lane & 7) ^ (lane >> 3));
  auto row_of = [&](int r, int rows, const int32_t* list, long stride) -> long {
    const int at = min(r, rows - 1);
    return !F64 && list ? (long)list[(long)b * stride + at] : (long)at;
  };
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int r = 8 * (LOADS * wave + j) + lr;
    src[j] = r < TM ? A + row_of(row0 + r, g.M, g.gatherA, g.gstrideA) * g.lda : B + row_of(col0 + r - TM, g.N, g.gatherB, g.gstrideB) * g.ldb;
    src[j] += lc + KT * (long)kt0;
  }
  unsigned char* base = ring + grp * (NST * STAGE);
  const int last = mine > 0 ? mine - 1 : 0;
  auto issue = [&](int kt) {
    // past the end: the last k-tile again (a group without any: the one before it), into a stage that is never read
    const long at = KT * (long)(mine == 0 ? -1 : kt < last ? kt : last);
    unsigned char* st = base + (kt & (NST - 1)) * STAGE + wave * (LOADS * 1024);
#pragma unroll
    for (int j = 0; j < LOADS; ++j)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + at),
                                       (__attribute__((address_space(3))) void*)(st + j * 1024), 16, 0, 0);
  };
  double* C = (double*)g.C + (long)b * g.strideC + (moved ? g.selC : 0);
  const double t = F64 && g.cheb ? g.cheb[(long)b * g.cheb_stride] : 0.0, scale = cheb_scale(g, t), rt = 1.0 / t;
  f64x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      acc[i][j] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
      if constexpr (F64) if (t != 0.0 && grp == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          acc[i][j][v] = cheb_start(g, A, C, rt, min(row0 + wm * (16 * MI) + i * 16 + 4 * v + kq, g.M - 1), min(col0 + wn * (16 * NJ) + j * 16 + i16, g.N - 1));
      }
    }
  // fragment of row R, half h: piece kq + 4h, i.e. k = PE (kq + 4h) + 0 .. PE - 1; R % 8 == i16 % 8 for every fragment row
  int offA[2], offB[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int piece = ((kq + 4 * h) ^ (i16 & 7)) * 16;
    offA[h] = (wm * (16 * MI) + i16) * 128 + piece;
    offB[h] = TM * 128 + (wn * (16 * NJ) + i16) * 128 + piece;
  }
  auto frags = [&](int kt, int h, piece_t (&fa)[MI], piece_t (&fb)[NJ]) {
    const unsigned char* st = base + (kt & (NST - 1)) * STAGE;
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[i] = *(const piece_t*)(st + offA[h] + i * 2048);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb[j] = *(const piece_t*)(st + offB[h] + j * 2048);
  };
  auto mma = [&](const piece_t (&fa)[MI], const piece_t (&fb)[NJ]) {
#pragma unroll
    for (int e = 0; e < PE; ++e)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(Piece<TS>::at(fa[i], e), Piece<TS>::at(fb[j], e), acc[i][j], 0, 0, 0);
  };
  // Per k-tile: wait until the next one has landed (only the loads of the one after it may be outstanding), barrier,
  // start the loads three ahead into the stage that held the previous one (every wave's reads of it are complete before it
  // arrives at the barrier).
  piece_t a0[MI], b0[NJ], a1[MI], b1[NJ];
  issue(0);
  issue(1);
  issue(2);
  __builtin_amdgcn_s_waitcnt(0x0070 + 2 * LOADS);       // vmcnt: the loads of two stages, lgkmcnt(0): k-tile 0 has landed
  __builtin_amdgcn_s_barrier();
  frags(0, 0, a0, b0);
  for (int kt = 0; kt < nk0; ++kt) {
    __builtin_amdgcn_s_waitcnt(0x0070 + LOADS);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    frags(kt, 1, a1, b1);
    issue(kt + 3);
    if (KS == 1 || kt < mine) mma(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    frags(kt + 1, 0, a0, b0);
    if (KS == 1 || kt < mine) mma(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);

  if constexpr (KS == 2) {                                // the second group's sums come second
    __syncthreads();
    double* x = (double*)ring + wave * (MI * NJ * 256) + lane;
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) x[((i * NJ + j) * 4 + v) * 64] = acc[i][j][v];
    }
    __syncthreads();
    if (grp == 1) return;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] += x[((i * NJ + j) * 4 + v) * 64];
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (g.frag) {
      // the product is symmetric: what this lane holds of tile (row, column) is the fragment of tile (column, row)
      const int per16 = g.N >> 4, ct = (row0 + wm * (16 * MI)) / 16 + i;
#pragma unroll
      for (int j = 0; j < NJ; ++j) frag_store(C + ((long)((col0 + wn * (16 * NJ)) / 16 + j) * per16 + ct) * kFragTile, lane, acc[i][j]);
      continue;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = row0 + wm * (16 * MI) + i * 16 + 4 * v + kq, c = col0 + wn * (16 * NJ) + j * 16 + i16;
        if (r < g.M && c < g.N) {
          C[(long)r * g.ldc + c] = scale * acc[i][j][v];
          if (g.mirror && tn != tm) C[(long)c * g.ldc + r] = acc[i][j][v];
        }
      }
  }
}

// Four consecutive elements as fp64 (aligned to an element; the loads are 16 bytes wide all the same).
typedef double f64x4_any __attribute__((ext_vector_type(4), aligned(8)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f64x4_t load4_f64(const double* p) { return *(const f64x4_any*)p; }
__device__ __forceinline__ f64x4_t load4_f64(const float* p) {
  const f32x4_any v = *(const f32x4_any*)p;
  return (f64x4_t){(double)v[0], (double)v[1], (double)v[2], (double)v[3]};
}

// The products of gemm64_dma_kernel where 16 x 16 tiles are one per compute unit at most: the four waves take a quarter of k each, operands straight from global memory, the partial
// tiles added in order by the first wave.  Bound by latency (192 x 320 x 320 is 0.5 us of MFMAs): no ring to fill, no barriers but one, a quarter of
// the MFMAs in a chain.
__global__ __launch_bounds__(256) void gemm64_tile16_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int DEPTH = 8;
  __shared__ double part[3 * 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), i16 = lane & 15, kq = lane >> 4;
  const bool triangle = g.lower_only || g.frag;
  const int per = triangle ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int gid = regroup_xcd(blockIdx.x, gridDim.x);
  const int b = gid / per, pidx = gid - b * per;
  if (g.skip && g.skip[b] > g.skip_if) return;
  int tm, tn;
  if (triangle) {
    int x = (int)((sqrtf(8.0f * (float)pidx + 1.0f) - 1.0f) * 0.5f);
    while (x * (x + 1) / 2 > pidx) --x;
    while ((x + 1) * (x + 2) / 2 <= pidx) ++x;
    const int y = pidx - x * (x + 1) / 2;
    tm = g.frag ? y : x;
    tn = g.frag ? x : y;
  } else {
    tm = pidx / tiles_n;
    tn = pidx - tm * tiles_n;
  }
  const int row0 = tm * 16, col0 = tn * 16, kn = g.K >> 2, nc = kn >> 4;
  const bool moved = g.sel && g.sel[b];
  const double* A = (const double*)g.A + (long)b * g.strideA + (moved ? g.selA : 0);
  const double* B = (const double*)g.B + (long)b * g.strideB + (moved ? g.selB : 0);
  const double* ar = A + (long)min(row0 + i16, g.M - 1) * g.lda + w * kn + 4 * kq;
  const double* br = B + (long)min(col0 + i16, g.N - 1) * g.ldb + w * kn + 4 * kq;
  f64x4_t fa[DEPTH], fb[DEPTH];
  auto load = [&](int s, int c) {
    if (c < nc) {
      fa[s] = load4_f64(ar + 16 * c);
      fb[s] = load4_f64(br + 16 * c);
    }
  };
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) load(s, s);
  double* C = (double*)g.C + (long)b * g.strideC + (moved ? g.selC : 0);
  const double t = g.cheb ? g.cheb[(long)b * g.cheb_stride] : 0.0, scale = cheb_scale(g, t), rt = 1.0 / t;
  f64x4_t acc = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  if (t != 0.0 && w == 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = cheb_start(g, A, C, rt, min(row0 + 4 * v + kq, g.M - 1), min(col0 + i16, g.N - 1));
  }
#pragma unroll 1
  for (int c = 0; c < nc; c += DEPTH) {
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      if (c + s < nc) {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][k], fb[s][k], acc, 0, 0, 0);
        load(s, c + s + DEPTH);
      }
    }
  }
  if (w > 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) part[((w - 1) * 4 + v) * 64 + lane] = acc[v];
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] += part[(q * 4 + v) * 64 + lane];
  if (g.frag) {
    frag_store(C + ((long)tn * (g.N >> 4) + tm) * kFragTile, lane, acc);
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = row0 + 4 * v + kq, c = col0 + i16;
    if (r < g.M && c < g.N) {
      C[(long)r * g.ldc + c] = scale * acc[v];
      if (g.mirror && tn != tm) C[(long)c * g.ldc + r] = acc[v];
    }
  }
}

// Problems of few tiles with an fp32 operand and optional row lists: 32 x 32 tile, the four waves take a
// quarter of k each, operands straight from global memory (rows in pieces of 16 elements, three such groups in flight), the
// partial tiles added through LDS in a fixed order.  Twice the operand traffic of a 64 x 64 tile but four times the
// workgroups and a sixteenth of the dependent MFMAs.  us, 64 x 64 register-staged -> here: 16 x 1024 x 1024 106 -> 15.7,
// 576 x 16 x 1024 96 -> 15.4, 128 x 128 x 1024 with row lists 138 -> 16.6, 576 x 1024 x 1024 row norms 145 -> 34.  Requires K % 64 == 0.
// A 32 x 32 tile is K / 64 us of its compute unit's MFMAs: where that leaves units idle the tiles are 16 x 16 (X = 1), eight groups in flight, every
// sum in the same order (128 x 128 x 1024 14.1 -> 7.0).
// EPI: EPI_STORE_F64, or EPI_ROWNORM2 with one partial per 32 columns.
template <typename TA, typename TB, int EPI, int X = 2>
__global__ __launch_bounds__(256) void gemm64_small_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int TILE = 16 * X, ROW = TILE + 1, PART = TILE * ROW;
  __shared__ double part[4 * PART];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  const int per = tiles_m * tiles_n;
  const int b = blockIdx.x / per, pidx = blockIdx.x - b * per, tm = pidx / tiles_n, tn = pidx - tm * tiles_n;
  if (g.skip && g.skip[b] > g.skip_if) return;
  if (g.lower_only && tn > tm) return;
  const int row0 = tm * TILE, col0 = tn * TILE, kn = g.K >> 2;
  const TA* Ab = (const TA*)g.A + (long)b * g.strideA;
  const TB* Bb = (const TB*)g.B + (long)b * g.strideB;
  const TA* ar[X];
  const TB* br[X];
#pragma unroll
  for (int x = 0; x < X; ++x) {
    long ra = min(row0 + 16 * x + i16, g.M - 1), rb = min(col0 + 16 * x + i16, g.N - 1);
    if (g.gatherA) ra = g.gatherA[(long)b * g.gstrideA + ra];
    if (g.gatherB) rb = g.gatherB[(long)b * g.gstrideB + rb];
    ar[x] = Ab + ra * g.lda + w * kn + 4 * kq;
    br[x] = Bb + rb * g.ldb + w * kn + 4 * kq;
  }
  constexpr int DEPTH = X == 1 ? 8 : 3;
  double* C = (double*)g.C + (long)b * g.strideC;
  f64x4_t acc[X][X], fa[DEPTH][X], fb[DEPTH][X];
#pragma unroll
  for (int x = 0; x < X; ++x)
#pragma unroll
    for (int y = 0; y < X; ++y) acc[x][y] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  const int nc = kn >> 4;
  auto load = [&](int s, int c) {
    if (c < nc) {
#pragma unroll
      for (int x = 0; x < X; ++x) {
        fa[s][x] = load4_f64(ar[x] + 16 * c);
        fb[s][x] = load4_f64(br[x] + 16 * c);
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
          for (int x = 0; x < X; ++x)
#pragma unroll
            for (int y = 0; y < X; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][x][k], fb[s][y][k], acc[x][y], 0, 0, 0);
        load(s, c + s + DEPTH);
      }
    }
  }
  double* out = part + w * PART;
#pragma unroll
  for (int x = 0; x < X; ++x)
#pragma unroll
    for (int y = 0; y < X; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(16 * x + 4 * v + kq) * ROW + 16 * y + i16] = acc[x][y][v];
  __syncthreads();
  auto sum = [&](int i, int j) {
    const double* q = part + i * ROW + j;
    return (q[0] + q[PART]) + (q[2 * PART] + q[3 * PART]);
  };
  if (EPI == EPI_ROWNORM2) {                              // eight lanes per row, four columns each; columns beyond N count as zero
    const int i = tid >> 3, j0 = (tid & 7) * 4;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (col0 + j0 + j < g.N) { const double v = sum(i, j0 + j); s = fma(v, v, s); }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((tid & 7) == 0 && row0 + i < g.M) C[(long)(row0 + i) * g.ldc + tn] = s;
    return;
  }
#pragma unroll
  for (int q = 0; q < X * X; ++q) {
    const int e = tid + 256 * q, i = e / TILE, j = e % TILE;
    if (row0 + i < g.M && col0 + j < g.N) C[(long)(row0 + i) * g.ldc + col0 + j] = sum(i, j);
    if (g.mirror && tn != tm && row0 + j < g.M && col0 + i < g.N) C[(long)(col0 + i) * g.ldc + row0 + j] = sum(j, i);
  }
}

// The products that follow the split (launch_gemm64_store_dot, launch_gemm64_rownorm_dual): 32 x 32 tile, the four
// waves take a quarter of k each, straight from global memory.  B is stored [K][N] and A is symmetric, so that both operands are
// read by rows of k, sixteen neighbouring doubles per quarter wave.  DUAL: the second product's k follows the first one's with
// A2 negated.  All dimensions are multiples of 64.  gemm64_kernel staged B's tiles through registers and walked all of k in
// every wave; us, residual / energies: one image of P = 192, nP = 320 47 -> 8.8 / 20 -> 6.1, four of 192, 1280 48 -> 23 / 22 -> 15,
// eight of 384, 1152 215 -> 133 / 85 -> 68, sixty-four of 256, 640 359 -> 276 / 160 -> 155.  Bound by the fp64 MFMA at the large end.
template <bool DUAL>
__global__ __launch_bounds__(256) void gemm64_sym_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  __shared__ double part[4 * 32 * 33];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i16 = lane & 15, kq = lane >> 4;
  const int per = tiles_m * tiles_n;
  const int b = blockIdx.x / per, pidx = blockIdx.x - b * per, tm = pidx / tiles_n, tn = pidx - tm * tiles_n;
  if (g.skip && g.skip[b] > g.skip_if) return;
  const int row0 = tm * 32, col0 = tn * 32;
  const int groups = g.K >> 6, total = DUAL ? 2 * groups : groups;      // steps of 16 k per wave
  const bool moved = g.sel && g.sel[b];
  const long abase = (long)b * g.strideA + row0 + i16, bbase = (long)b * g.strideB + col0 + i16, bmoved = moved ? g.selB : 0;
  f64x4_t acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[x][y][v] = 0.0;
  double fa[2][4][2], fb[2][4][2];
  auto load = [&](int t, double (&a)[4][2], double (&bb)[4][2]) {
    const bool second = DUAL && t >= groups;
    const double* A = (const double*)(second ? g.A2 : g.A) + abase;
    const double* B = second ? (const double*)g.B2 + bbase : (const double*)g.B + bbase + bmoved;
    const long k0 = (long)(second ? t - groups : t) * 64 + 16 * w + kq;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const double av = A[(k0 + 4 * q) * g.lda + 16 * x];
        a[q][x] = second ? -av : av;
        bb[q][x] = B[(k0 + 4 * q) * g.ldb + 16 * x];
      }
  };
  auto mul = [&](const double (&a)[4][2], const double (&bb)[4][2]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q][x], bb[q][y], acc[x][y], 0, 0, 0);
  };
  load(0, fa[0], fb[0]);
#pragma unroll 1
  for (int t = 0; t < total; t += 2) {
    if (t + 1 < total) load(t + 1, fa[1], fb[1]);
    mul(fa[0], fb[0]);
    if (t + 1 >= total) break;
    if (t + 2 < total) load(t + 2, fa[0], fb[0]);
    mul(fa[1], fb[1]);
  }
  double* out = part + w * (32 * 33);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(16 * x + 4 * v + kq) * 33 + 16 * y + i16] = acc[x][y][v];
  __syncthreads();
  auto sum = [&](int i, int j) {
    const double* q = part + i * 33 + j;
    return (q[0] + q[32 * 33]) + (q[2 * 32 * 33] + q[3 * 32 * 33]);
  };
  const long coff = (long)b * g.strideC;
  if (DUAL) {                                             // eight lanes per row, four columns each
    const int i = tid >> 3, j0 = (tid & 7) * 4;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) { const double v = sum(i, j0 + j); s = fma(v, v, s); }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((tid & 7) == 0) ((double*)g.C)[coff + (long)(row0 + i) * g.ldc + tn] = s;
    return;
  }
  double dot = 0.0;                                       // eight threads per column, four rows each
  const int j = tid & 31, i0 = tid >> 5;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double v = sum(i0 + 8 * q, j);
    const long o = coff + (long)(row0 + i0 + 8 * q) * g.ldc + col0 + j;
    ((double*)g.C)[o] = v;
    dot = fma(v, ((const double*)g.D)[o + (moved ? g.selD : 0)], dot);
  }
  __syncthreads();
  part[i0 * 33 + j] = dot;
  __syncthreads();
  if (tid < 32) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s += part[q * 33 + tid];
    g.dots[((long)b * tiles_m + tm) * g.N + col0 + tid] = s;
  }
}

// Can gemm64_small_kernel take the product?
inline bool small_fits(const GemmArgs& g) { return g.batch > 0 && g.batch_inner == 1 && g.K >= 64 && g.K % 64 == 0; }

template <typename TA, typename TB, int EPI>
hipError_t launch_small(const GemmArgs& g, hipStream_t stream) {
  const long m32 = (g.M + 31) / 32, n32 = (g.N + 31) / 32, blocks = m32 * n32 * g.batch;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  if constexpr (EPI == EPI_STORE_F64) {
    // 16 x 16 tiles while a compute unit gets one.  us, 32 x 32 / here: 36 (576 x 16 x 1024) 13.3 / 8.2, 64 (16 x 1024 x 1024) 13.2 / 8.3, 171 (288 x 288
    // x 1024, the lower ones) 14.4 / 11.1, 256 (64 x 1024 x 1024) 14.7 / 8.6, 256 of K = 4096 51 / 28; 296 (577 x 32 x 768, batch 4) 12.1 / 11.7, 384
    // 14.9 / 14.8, 380 (300 x 300 x 1024, batch 2, the lower ones) 14.8 / 16.0, 640 15.2 / 20.6.
    const long m16 = (g.M + 15) / 16, n16 = (g.N + 15) / 16;
    if ((g.lower_only ? m16 * (m16 + 1) / 2 : m16 * n16) * g.batch <= kUnits) {
      hipLaunchKernelGGL((gemm64_small_kernel<TA, TB, EPI, 1>), dim3((unsigned)(m16 * n16 * g.batch)), dim3(256), 0, stream, g, (int)m16, (int)n16);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((gemm64_small_kernel<TA, TB, EPI>), dim3((unsigned)blocks), dim3(256), 0, stream, g, (int)m32, (int)n32);
  return hipGetLastError();
}

inline long tiles64(const GemmArgs& g) { return (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.batch; }

template <typename TS, int KS, int TM, int TN, int WM = 2>
hipError_t launch_dma(const GemmArgs& g, hipStream_t stream) {
  const long tm = (g.M + TM - 1) / TM, tn = (g.N + TN - 1) / TN;
  const bool triangle = g.lower_only || g.frag;
  if (triangle && TM != TN) return hipErrorInvalidValue;
  const long blocks = (triangle ? tm * (tm + 1) / 2 : tm * tn) * g.batch;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  constexpr size_t kRing = (size_t)KS * 4 * dma_stage(TM, TN);
  if (kRing > 64 * 1024) {
    static PerDeviceInt raised;
    const hipError_t e = ensure_dynamic_lds(raised, (const void*)gemm64_dma_kernel<TS, KS, TM, TN, WM>, kRing);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((gemm64_dma_kernel<TS, KS, TM, TN, WM>), dim3((unsigned)blocks), dim3(256 * KS), kRing, stream, g, (int)tm, (int)tn);
  return hipGetLastError();
}

template <typename TS>
hipError_t launch_plain(const GemmArgs& g, hipStream_t stream) {
  constexpr bool F64 = std::is_same<TS, double>::value;
  const bool triangle = g.lower_only || g.frag;
  if ((triangle && g.M != g.N) || (g.frag && g.N % 64 != 0)) return hipErrorInvalidValue;
  const Gemm64Tile tile = plain_tile(g.M, g.N, g.K, g.batch, triangle, F64);
  if constexpr (F64) {
    if (tile == TILE_16x16) {
      const int m16 = (g.M + 15) / 16, n16 = (g.N + 15) / 16;
      const unsigned blocks = (triangle ? m16 * (m16 + 1) / 2 : m16 * n16) * g.batch;
      hipLaunchKernelGGL(gemm64_tile16_kernel, dim3(blocks), dim3(256), 0, stream, g, m16, n16);
      return hipGetLastError();
    }
    if (tile == TILE_64x96) return launch_dma<TS, 1, 64, 96>(g, stream);
    if (tile == TILE_64x80) return launch_dma<TS, 1, 64, 80, 4>(g, stream);
    if (tile == TILE_64x48) return launch_dma<TS, 1, 64, 48, 4>(g, stream);
  }
  if (tile == TILE_64x64) return launch_dma<TS, 1, 64, 64>(g, stream);
  if (tile == TILE_64x32) return launch_dma<TS, 1, 64, 32>(g, stream);
  const long m32 = (g.M + 31) / 32, n32 = (g.N + 31) / 32, t32 = (triangle ? m32 * (m32 + 1) / 2 : m32 * n32) * g.batch;
  return t32 <= kUnits && g.K >= (int)(256 / sizeof(TS)) ? launch_dma<TS, 2, 32, 32>(g, stream) : launch_dma<TS, 1, 32, 32>(g, stream);
}

// Products gemm64_dma_kernel takes.
template <typename TS>
inline bool plain(const GemmArgs& g) {
  constexpr int PE = 16 / sizeof(TS);
  return g.batch > 0 && g.batch_inner == 1 && g.K >= 8 * PE && g.K % (8 * PE) == 0 && g.lda % PE == 0 && g.ldb % PE == 0 && g.strideA % PE == 0 &&
         g.strideB % PE == 0 && (((uintptr_t)g.A | (uintptr_t)g.B) & 15) == 0;
}

template <typename TA, typename TB, int EPI, bool GATHER, int MI, int NJ>
hipError_t launch_cfg(const GemmArgs& g, hipStream_t stream) {
  constexpr int TM = 32 * MI, TN = 32 * NJ;
  const int tiles_m = (g.M + TM - 1) / TM, tiles_n = (g.N + TN - 1) / TN;
  const long nblocks = (long)tiles_m * tiles_n * g.batch;
  if (nblocks <= 0) return hipSuccess;
  if (nblocks > 0x7fffffffL) return hipErrorInvalidValue;
  const size_t lds = (size_t)2 * (TM + TN) * PITCH * sizeof(double);
  auto kern = gemm64_kernel<TA, TB, EPI, GATHER, MI, NJ>;
  if (lds > 64 * 1024) {
    static PerDeviceInt raised;   // per instantiation
    const hipError_t e = ensure_dynamic_lds(raised, (const void*)kern, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(256), lds, stream, g, tiles_m, tiles_n);
  return hipGetLastError();
}

// Row norms are decided by sizes alone: the number of partials is part of a plan.
inline bool rownorm_small(long M, int N, int K) { return ((M + 63) / 64) * ((N + 63) / 64) <= kSmallTiles64 && K >= 64 && K % 64 == 0; }

template <typename TA, typename TB>
hipError_t launch_ab(const GemmArgs& g, hipStream_t stream) {
  const bool gather = g.gatherA || g.gatherB;
  constexpr bool f64x2 = std::is_same<TA, double>::value && std::is_same<TB, double>::value;
  if constexpr (!f64x2 && !std::is_same<TA, bf16_t>::value) {
    if (g.epilogue == EPI_STORE_F64 && tiles64(g) <= kSmallTiles64 && small_fits(g)) return launch_small<TA, TB, EPI_STORE_F64>(g, stream);
  }
  if (g.epilogue == EPI_STORE_F64) {
    if constexpr (std::is_same<TA, bf16_t>::value) {
      if (plain<bf16_t>(g) && (!g.lower_only || g.M == g.N)) return launch_plain<bf16_t>(g, stream);
    }
    if (gather) return launch_cfg<TA, TB, EPI_STORE_F64, true, 2, 2>(g, stream);
    if constexpr (f64x2) {
      if (plain<double>(g)) return launch_plain<double>(g, stream);
    }
    if (g.frag || g.sel || g.cheb) return hipErrorInvalidValue;
    return launch_cfg<TA, TB, EPI_STORE_F64, false, 2, 2>(g, stream);
  }
  if (gather) return hipErrorInvalidValue;
  if constexpr (std::is_same<TA, float>::value && std::is_same<TB, float>::value) {
    // one product of stored rows and weights: the only form whose number of partials gemm64_tiles_n states
    if (g.epilogue == EPI_ROWNORM2 && g.batch == 1 && g.batch_inner == 1)
      return rownorm_small(g.M, g.N, g.K) ? launch_small<TA, TB, EPI_ROWNORM2>(g, stream) : launch_cfg<TA, TB, EPI_ROWNORM2, false, 2, 2>(g, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int gemm64_tiles_n(long M, int N, int K) { return rownorm_small(M, N, K) ? (N + 31) / 32 : (N + 63) / 64; }

template <bool DUAL>
static hipError_t launch_sym(const GemmArgs& g, hipStream_t stream) {
  if (g.gatherA || g.gatherB || g.M != g.K || g.M % 64 != 0 || g.N % 64 != 0 || g.batch < 1 || g.batch_inner != 1) return hipErrorInvalidValue;
  const long m32 = g.M / 32, n32 = g.N / 32, blocks = m32 * n32 * g.batch;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm64_sym_kernel<DUAL>, dim3((unsigned)blocks), dim3(256), 0, stream, g, (int)m32, (int)n32);
  return hipGetLastError();
}

hipError_t launch_gemm64_store_dot(const GemmArgs& g, hipStream_t stream) {
  return g.D && g.dots ? launch_sym<false>(g, stream) : hipErrorInvalidValue;
}

hipError_t launch_gemm64_rownorm_dual(const GemmArgs& g, hipStream_t stream) {
  return g.A2 && g.B2 ? launch_sym<true>(g, stream) : hipErrorInvalidValue;
}

hipError_t launch_gemm64_bf16(const GemmArgs& g, hipStream_t stream) { return launch_ab<bf16_t, bf16_t>(g, stream); }

hipError_t launch_gemm64_nt(const GemmArgs& g, bool a_is_f64, bool b_is_f64, hipStream_t stream) {
  if (a_is_f64) return b_is_f64 ? launch_ab<double, double>(g, stream) : launch_ab<double, float>(g, stream);
  return b_is_f64 ? launch_ab<float, double>(g, stream) : launch_ab<float, float>(g, stream);
}

}  // namespace covspec
