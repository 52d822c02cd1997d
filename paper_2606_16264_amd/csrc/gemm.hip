// gemm.hip -- bf16 matrix-core GEMM for gfx950: C[M][N] = A[M][K] * B[N][K]^T
// with fp32 accumulation and fused epilogues (plain store, + residual, SwiGLU,
// and the QKV projection's RoPE + KV-cache append).
//
// Design:
//  - workgroup tile BM x BN, K step 64; waves of 64 lanes each own a WM x WN
//    sub-tile computed with v_mfma_f32_16x16x32_bf16 (one product per 16 x 16
//    block and 32-wide K slice: under the chip's power limit it sustains a
//    higher rate than the 32 x 32 x 16 form, for the same LDS reads);
//  - K is consumed in 32-wide slices through an LDS ring (4 stages, 3 in the last
//    shape, 6 in the read-once 64 x 128 tiles) filled by the DMA path
//    (global_load_lds): the other slices are in flight while the matrix cores
//    work on one, and no registers are spent on staging;
//  - B is addressed through block, row and K-slice strides: row-major, or the
//    packed weights' 16 x 32 tiles of 1 KB, where each DMA instruction reads
//    one contiguous kilobyte;
//  - a slice runs in two phases (the two halves of the wave's A blocks against
//    all its B blocks); each phase's MFMAs are issued one at a time, with the
//    slice's DMA issues (first phase) and the next slice's fragment reads
//    (second phase) spread between them, so that a wave keeps the matrix core
//    fed while it issues its memory instructions; one barrier per slice;
//  - LDS rows are 64 bytes (32 bf16 of K); the 16-byte chunk c of row r is
//    stored at c ^ swz(r), which makes the 16 lanes that the LDS serves at a
//    time hit 16 distinct bank groups (see swz);
//  - tile order is XCD-aware: workgroup b runs on XCD b % 8, and each XCD is
//    handed a contiguous run of tiles taken in M-grouped order, so that the
//    tiles sharing an L2 also share A and B panels;
//  - a K split runs over a second grid dimension (split z of S takes the
//    64-wide K chunks [z C / S, (z + 1) C / S) of the C in K, so S need not
//    divide C) and finishes in a deterministic reduce-and-epilogue kernel;
//  - a cost model picks tile shape and K split per problem (a per-CU feed
//    estimate for few rows, rounds of tile-units for more), and may run the
//    rows in two launches: the first in whole rounds of tiles, the rest as a
//    GEMM of their own (split over K), so that a problem a little over a whole
//    number of rounds does not pay for a mostly empty last round.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <tuple>

#include "gemm_tile.h"
#include "mx_device.h"
#include "mx_kernels.h"

namespace mx {

namespace {

template <int BM, int BN, int WM, int WN, int NS, int EPI, bool SPLIT>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void gemm_kernel(GemmArgs a, int tiles_m,
                                                                           int tiles_n,
                                                                           int k_chunks) {
  gemm_tile<BM, BN, WM, WN, NS, EPI, SPLIT, false>(a, tiles_m, tiles_n, k_chunks);
}

// Plain or residual reduce, four columns per thread (N, ldc and ldr multiples
// of 4): 16-byte partial loads, 8-byte residual loads and stores, and every
// load of a thread's iteration issued before its store.
template <bool RESIDUAL>
__global__ __launch_bounds__(256) void splitk_reduce4_kernel(GemmArgs a, int ksplit) {
  const int nq4 = a.N / 4;
  const int64_t total = (int64_t)a.M * nq4;
  const f32x4* part = reinterpret_cast<const f32x4*>(a.partial);
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(idx / nq4), col = (int)(idx % nq4) * 4;
    f32x4 v = part[idx];
    for (int z = 1; z < ksplit; z++) {
      const f32x4 pz = part[z * total + idx];
      v[0] += pz[0]; v[1] += pz[1]; v[2] += pz[2]; v[3] += pz[3];
    }
    if constexpr (RESIDUAL) {
      const u32x2 r = *reinterpret_cast<const u32x2*>(a.R + (int64_t)row * a.ldr + col);
      v[0] += __uint_as_float(r[0] << 16);
      v[1] += __uint_as_float(r[0] & 0xFFFF0000u);
      v[2] += __uint_as_float(r[1] << 16);
      v[3] += __uint_as_float(r[1] & 0xFFFF0000u);
    }
    u32x2 w;
    w[0] = pack_bf16x2(v[0], v[1]);
    w[1] = pack_bf16x2(v[2], v[3]);
    *reinterpret_cast<u32x2*>(a.C + (int64_t)row * a.ldc + col) = w;
  }
}

// Sum of the K splits in fixed order, then the epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a, int ksplit) {
  const int ncols = (EPI == EPI_SWIGLU || EPI == EPI_QKV) ? a.N / 2 : a.N;
  const int64_t total = (int64_t)a.M * ncols;
  const int64_t plane = (int64_t)a.M * a.N;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(idx / ncols), col = (int)(idx % ncols);
    if constexpr (EPI == EPI_QKV) {
      const int c = (col / 32) * 64 + col % 32;
      const int64_t li = (int64_t)row * a.N + c, hi = li + 32;
      float lo = 0.f, hv = 0.f;
      for (int z = 0; z < ksplit; z++) {
        lo += a.partial[z * plane + li];
        hv += a.partial[z * plane + hi];
      }
      const QkvEpilogue& e = a.qkv;
      qkv_pair_store(e.q_out, e.k_pool, e.v_pool, e.nq, e.nkv, e.head_dim, row, c, lo, hv,
                     e.tok_slot[row], e.rope_cs[rope_index(row, c, e.head_dim)]);
    } else if constexpr (EPI == EPI_SWIGLU) {
      const int fb = col / 32, w = col % 32;
      const int64_t gi = (int64_t)row * a.N + fb * 64 + w, ui = gi + 32;
      float g = 0.f, u = 0.f;
      for (int z = 0; z < ksplit; z++) {
        g += a.partial[z * plane + gi];
        u += a.partial[z * plane + ui];
      }
      a.C[a.c_tiled ? tile_index(row, col, a.ldc) : (int64_t)row * a.ldc + col] =
          f32_to_bf16(silu(g) * u);
    } else {
      const int64_t pi = (int64_t)row * a.N + col;
      float v = 0.f;
      for (int z = 0; z < ksplit; z++) v += a.partial[z * plane + pi];
      if constexpr (EPI == EPI_RESIDUAL) v += bf16_to_f32(a.R[(int64_t)row * a.ldr + col]);
      a.C[(int64_t)row * a.ldc + col] = f32_to_bf16(v);
    }
  }
}

struct Shape {
  int BM, BN;
  // time of one round of tile-units on the chip: a + b * (K slice length),
  // microseconds (least-squares fit over measured layer-shape GEMMs, all tile
  // shapes and K splits; the main loop is bound by its global->LDS feed, so a
  // unit's time grows with the bytes it streams)
  double a_us, b_us_per_k;
  int per_cu;       // tile-units one round holds per CU
  double feed_gbs;  // bytes a CU streams per microsecond (x1e3) with cold weights
};
// 256x256 and 128x256 run eight waves (2 per SIMD), the smaller shapes four.
// The last shape is 128x256 with a three-stage ring (72 KB of LDS), meant for
// two workgroups per CU; with the 16 x 16 x 32 main loop a 128x256 wave needs
// more than the 128 registers that four waves per SIMD leave, so it runs one
// per CU, and its figures (a fourth stage missing against the 128x256 shape)
// keep the model from choosing it where it prices at all (see choose_one).
constexpr Shape kShapes[] = {{256, 256, 3.471, 0.02443, 1, 44.3},
                             {128, 256, 0.978, 0.01544, 1, 56.7},
                             {128, 128, 2.5, 0.0194, 2, 45.7},
                             {64, 128, 0.0, 0.00729, 1, 55.7},
                             {128, 256, 0.978, 0.0287, 1, 50.0}};
constexpr int kNumShapes = 5;
constexpr int kFeedMaxM = 256;  // rows up to which the feed estimate is used
constexpr double kCUs = 256.0;
// Two 128x128 workgroups share a CU; one alone takes 0.75 of the pair's time
// (1003 x 4096 x 4096, 256 tiles: 53 us; 1003 x 6144 x 4096, 384 tiles, one pair on
// half of the CUs: 71).  Priced as two rounds of single tiles, O of a 1003-token
// 8B prompt ran 128x128 tiles, 54 us, not 128x256 split in two, 47 with the reduce
// (the layer 447 -> 436 us).
constexpr double kLoneUnit = 0.75;
// One round of 128x256 tiles takes 0.94 of what their rounds take in larger
// problems (its tiles have the chip's power and memory paths to themselves for
// their last part): 400 x 4096 x 14336 split in four 61.5 us (256x256 split in eight
// 69.8), 576 x 10240 x 8192 unsplit 101 (256x256 split in two 107), 400 x 4096 x 4096
// in four 30.8 (64x128 unsplit 35.3), 1028 x 4096 x 4096 unsplit 47.7 (256x256 split in
// three 52.7), 2048 x 4096 x 11008 unsplit 144 (256x256 split in two 159).
constexpr double kOneRound = 0.94;

// Estimated time (us) of one GEMM launch with tile shape c and K split ks, in
// two regimes, or a negative value when the choice is not allowed.  Few rows
// (M <= kFeedMaxM): the layer's weights arrive cold from HBM and the busiest
// CU's feed bounds the time: its tile-units (ceil(units / 256)) times the
// bytes one unit streams (its A and B rows over its K slice) at the shape's
// per-CU fetch rate, plus a fixed cost; the weights' stream bounds it from below
// (the 8.2e6 bytes per us of that bound belong to the fit with the fixed 5.76 us
// beside them, and are no rate of the memory, which gives 6.7e6).  More rows: the
// busiest CU's ceil(units / 256) units run in rounds of per_cu, a last single one
// of a pair's shape at kLoneUnit of a round, and nothing beats streaming the
// operands from HBM once.  A K split adds the fp32 partial round trip and the
// reduce launch.  Both fitted on cold timings of the layer GEMMs of the four layer
// shapes, every tile shape and every K split from 1 to 8.  Few rows (15 GEMMs at
// 24, 40, 64, 96, 128, 160, 200 and 256 rows, timed with read-once kernels for
// every single row of tiles): the picks are 0.3% above the best measured on
// average, 5% at most (4.9% on average with the constants fitted before those
// kernels).  More rows (320 to 3200): 0.8% on average.
double estimate(int c, int ks, int M, int N, int K) {
  const double hbm = 5.0e12;
  if ((K / BK) / ks < 4) return -1.0;  // every split at least four 64-wide K chunks
  if (ks > 1 && (double)ks * M * N > (double)kMaxSplitFloats) return -1.0;
  const int BM = kShapes[c].BM, BN = kShapes[c].BN;
  const double tiles = (double)((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const double split_mb = ((double)ks * M * N * 8.0 + 2.0 * M * N) / 1e6;
  const double k_unit = (double)((K / BK + ks - 1) / ks * BK);  // the longest split
  if (M <= kFeedMaxM) {
    const double per_cu = std::ceil(tiles * ks / kCUs);
    // (rows past M are copied too, from row M - 1: 0.63 of a row's cost)
    const double rows = M < BM ? M + 0.63 * (BM - M) : BM;
    const double unit_bytes = (BN + rows) * k_unit * 2.0;
    const double t_feed = per_cu * unit_bytes / (kShapes[c].feed_gbs * 1e3);
    return std::max(t_feed, 2.0 * N * K / 8.2e6) + 5.76 + (ks > 1 ? 0.222 * split_mb + 0.39 : 0.0);
  }
  const double per_cu = std::ceil(tiles * ks / kCUs);  // tile-units of the busiest CU
  const double full = std::floor(per_cu / kShapes[c].per_cu);
  const double rounds = full + (per_cu > full * kShapes[c].per_cu ? kLoneUnit : 0.0);
  const double one = c == 1 && per_cu == 1.0 ? kOneRound : 1.0;
  const double t_units = one * rounds * (kShapes[c].a_us + kShapes[c].b_us_per_k * k_unit);
  const double t_mem = 2.0 * ((double)N * K + (double)M * K) / hbm * 1e6;
  return std::max(t_units, t_mem) + (ks > 1 ? 0.197 * split_mb + 3.39 : 0.0);
}

struct Pick {
  int cfg, ksplit;
  double t;
};

// The best (tile shape, K split) of one launch over all M rows.  K below 256, which
// estimate() does not price, runs the last shape.
Pick choose_one(int M, int N, int K) {
  Pick best{kNumShapes - 1, 1, 1e30};
  for (int c = 0; c < kNumShapes; c++)
    for (int ks = 1; ks <= 8; ks++) {
      const double t = estimate(c, ks, M, N, K);
      if (t < 0.0) break;
      if (t < best.t * 0.98) best = {c, ks, t};
    }
  return best;
}

// Launch plan of one GEMM.  Rows [0, m_main) run with tile shape cfg and K
// split ksplit; when m_main < M, the remaining rows run as a second GEMM of
// their own (tile shape tail_cfg, K split tail_ksplit) after the first.  The
// row split removes the last, mostly empty round of a problem whose tiles
// fill a few rounds and a little more (70B-shaped down projection at 8448
// rows: 1056 tiles of 256 x 256, 4.125 rounds of 256 CUs, run as 1024 tiles in
// four full rounds plus 256 rows split eight ways over K).
struct Plan {
  int cfg, ksplit;
  int m_main;
  int tail_cfg, tail_ksplit;
  double t;  // estimated time (us) of a plan without a row split
};

Plan plan_uncached(int M, int N, int K) {
  const Pick whole = choose_one(M, N, K);
  Plan best{whole.cfg, whole.ksplit, M, -1, 0, whole.t};
  if (M <= 2 * kFeedMaxM) return best;
  double best_t = whole.t;
  // first part: whole rounds of one tile shape without a K split; second part:
  // the remaining rows, planned as a launch of their own (plus a launch gap)
  for (int c = 0; c < kNumShapes; c++) {
    const int BM = kShapes[c].BM, BN = kShapes[c].BN;
    const double slots = kCUs * kShapes[c].per_cu;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    for (int j = tiles_m - 1; j >= 1 && M - j * BM <= 4 * kFeedMaxM; j--) {
      const double tiles = (double)j * tiles_n;
      const double frac = tiles / slots - std::floor(tiles / slots);
      if (frac > 0.0 && frac < 0.75) continue;  // only (nearly) full last rounds
      const double t_main = estimate(c, 1, j * BM, N, K);
      if (t_main < 0.0) continue;
      const Pick tail = choose_one(M - j * BM, N, K);
      const double t = t_main + tail.t + 4.0;
      if (t < best_t * 0.97) {
        best_t = t;
        best = {c, 1, j * BM, tail.cfg, tail.ksplit, 0.0};
      }
    }
  }
  // ... unless the rows are one round of 256 x 256 tiles that leaves CUs free: its
  // tiles have the chip's power and memory paths to themselves and take less than the
  // full round that estimate() prices: with 0.55-0.8 of the CUs at work 0.69-0.75 of
  // it on one card and 0.76-0.83 on another, more power-bound one, against 0.87 and
  // 0.89 of their prices for the row splits.  At 0.84 the choice is 1.1 and 1.0% above
  // the better of the two on average (317 and 348 problems measured on each), always
  // splitting 5.2 and 0.9%, never splitting 2.4 and 6.0% (608 x 15360 x 5120, 180
  // tiles: 92 us whole on the first card, 108 as 512 + 96 rows; 768 x 12288 x 4096, 144
  // tiles: 76 and 88).
  const double tiles = (double)((M + 255) / 256) * ((N + 255) / 256);
  if (best.m_main < M && tiles <= kCUs) {
    const double t = estimate(0, 1, M, N, K);
    if (t > 0.0 && 0.84 * t < best_t) best = {0, 1, M, -1, 0, t};
  }
  return best;
}

// Plans are cached per problem: the layer step plans four GEMMs per call.
Plan plan_gemm(int M, int N, int K) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int>, Plan> cache;
  const auto key = std::make_tuple(M, N, K);
  {
    std::lock_guard<std::mutex> g(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
  }
  const Plan p = plan_uncached(M, N, K);
  std::lock_guard<std::mutex> g(mu);
  if (cache.size() > 4096) cache.clear();
  cache[key] = p;
  return p;
}

// Scratch (fp32 elements) that a plan's K split needs.
size_t plan_scratch(const Plan& p, int M, int N) {
  if (p.m_main < M) return p.tail_ksplit > 1 ? (size_t)p.tail_ksplit * (M - p.m_main) * N : 0;
  return p.ksplit > 1 ? (size_t)p.ksplit * M * N : 0;
}

// The GEMM of rows [m0, M) of a: every row-indexed operand moves by m0 rows
// (A, C, R and, for the QKV epilogue, the rotary table, the token slots and
// q_out; the pools are addressed through the slots).  In the tile layout row
// m0 starts a tile row only when m0 % 16 == 0, which the callers ensure.
GemmArgs rows_from(const GemmArgs& a, int m0) {
  GemmArgs t = a;
  t.M = a.M - m0;
  t.A = a.A + (a.a_tiled ? (int64_t)(m0 / 16) * tile_row_pitch(a.lda) : (int64_t)m0 * a.lda);
  if (t.C)
    t.C = a.C + (a.c_tiled ? (int64_t)(m0 / 16) * tile_row_pitch(a.ldc) : (int64_t)m0 * a.ldc);
  if (t.R) t.R = a.R + (int64_t)m0 * a.ldr;
  if (a.epilogue == EPI_QKV) {
    t.qkv.rope_cs = a.qkv.rope_cs + (int64_t)m0 * (a.qkv.head_dim / 2);
    t.qkv.tok_slot = a.qkv.tok_slot + m0;
    t.qkv.q_out = a.qkv.q_out + (int64_t)m0 * a.qkv.nq * a.qkv.head_dim;
  }
  return t;
}

template <int BM, int BN, int WM, int WN, int NS, int EPI, bool SPLIT>
hipError_t run(const GemmArgs& a, int ksplit, hipStream_t stream) {
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int threads = (BM / WM) * (BN / WN) * 64;
  const size_t lds = (size_t)NS * (BM + BN) * BKS * 2;
  dim3 grid(tiles_m * tiles_n, ksplit);
  gemm_kernel<BM, BN, WM, WN, NS, EPI, SPLIT><<<grid, threads, lds, stream>>>(a, tiles_m, tiles_n,
                                                                          a.K / BK);
  return hipGetLastError();
}

// Whether a GEMM of one row of tiles over weights that come from HBM runs in the
// read-once kernels.  Weights of less than 16 MB may well be in the caches (a tiny
// GEMM, 132 x 1024 x 256, took 9.0 us with the deep ring against 7.7).  A K split's
// fp32 planes go out to the caches and back meanwhile, and beside many of them the
// non-temporal reads gain nothing: in the layer step (four layer shapes, 23 row counts
// from 17 to 256, cold weights) the read-once kernels take 0.77-0.95 of the ordinary
// ones' time unsplit, 0.86-1.03 with planes of up to a quarter of the weights' bytes,
// 0.98-1.05 beyond (8B qkv at 72 rows split in eight, 0.28, 26.0 us against 24.8).
bool reads_once(int M, int N, int K, int BM, int ksplit) {
  return M <= BM && (int64_t)N * K * 2 >= (int64_t)16 << 20 &&
         (ksplit == 1 || (int64_t)8 * ksplit * M <= K);
}

// reduce = false: a K split leaves its fp32 planes at a.partial for the caller
// to reduce.
template <int BM, int BN, int WM, int WN, int NS>
hipError_t run_shape(const GemmArgs& a, int ksplit, bool reduce, hipStream_t stream) {
  // (they stand for the four-stage shapes: the three-stage one runs as itself)
  const bool once = NS == 4 && has_gemm_once(BM, BN) && reads_once(a.M, a.N, a.K, BM, ksplit);
  if (ksplit > 1) {
    hipError_t e = once ? launch_gemm_once(a, BM, ksplit, stream)
                        : run<BM, BN, WM, WN, NS, EPI_STORE, true>(a, ksplit, stream);
    if (e != hipSuccess || !reduce) return e;
    const bool paired = a.epilogue == EPI_SWIGLU || a.epilogue == EPI_QKV;
    const int64_t total = (int64_t)a.M * (paired ? a.N / 2 : a.N);
    const int blocks = (int)std::min<int64_t>((total + 255) / 256, 4096);
    const bool by4 = !paired && a.N % 4 == 0 && a.ldc % 4 == 0 &&
                     (a.epilogue != EPI_RESIDUAL || a.ldr % 4 == 0);
    if (by4) {
      const int blocks4 = (int)std::min<int64_t>((total / 4 + 255) / 256, 4096);
      if (a.epilogue == EPI_RESIDUAL)
        splitk_reduce4_kernel<true><<<blocks4, 256, 0, stream>>>(a, ksplit);
      else
        splitk_reduce4_kernel<false><<<blocks4, 256, 0, stream>>>(a, ksplit);
      return hipGetLastError();
    }
    if (a.epilogue == EPI_QKV)
      splitk_reduce_kernel<EPI_QKV><<<blocks, 256, 0, stream>>>(a, ksplit);
    else if (a.epilogue == EPI_SWIGLU)
      splitk_reduce_kernel<EPI_SWIGLU><<<blocks, 256, 0, stream>>>(a, ksplit);
    else if (a.epilogue == EPI_RESIDUAL)
      splitk_reduce_kernel<EPI_RESIDUAL><<<blocks, 256, 0, stream>>>(a, ksplit);
    else
      splitk_reduce_kernel<EPI_STORE><<<blocks, 256, 0, stream>>>(a, ksplit);
    return hipGetLastError();
  }
  if (once) return launch_gemm_once(a, BM, 1, stream);
  switch (a.epilogue) {
    case EPI_QKV: return run<BM, BN, WM, WN, NS, EPI_QKV, false>(a, 1, stream);
    case EPI_SWIGLU: return run<BM, BN, WM, WN, NS, EPI_SWIGLU, false>(a, 1, stream);
    case EPI_RESIDUAL: return run<BM, BN, WM, WN, NS, EPI_RESIDUAL, false>(a, 1, stream);
    default: return run<BM, BN, WM, WN, NS, EPI_STORE, false>(a, 1, stream);
  }
}

template <int BM, int BN, int WM, int WN, int NS>
hipError_t set_lds_attr() {
  const int lds = NS * (BM + BN) * BKS * 2;
  hipError_t e;
#define MX_SET(EPI, SPLIT)                                                                  \
  e = hipFuncSetAttribute((const void*)gemm_kernel<BM, BN, WM, WN, NS, EPI, SPLIT>,             \
                          hipFuncAttributeMaxDynamicSharedMemorySize, lds);                 \
  if (e != hipSuccess) return e;
  MX_SET(EPI_STORE, false)
  MX_SET(EPI_RESIDUAL, false)
  MX_SET(EPI_SWIGLU, false)
  MX_SET(EPI_QKV, false)
  MX_SET(EPI_STORE, true)
#undef MX_SET
  return hipSuccess;
}

}  // namespace

hipError_t gemm_init() {
  hipError_t e = set_lds_attr<256, 256, 128, 64, 4>();
  if (e != hipSuccess) return e;
  e = set_lds_attr<128, 256, 64, 64, 4>();
  if (e != hipSuccess) return e;
  e = set_lds_attr<128, 128, 64, 64, 4>();
  if (e != hipSuccess) return e;
  e = set_lds_attr<64, 128, 32, 64, 4>();
  if (e != hipSuccess) return e;
  e = set_lds_attr<128, 256, 64, 64, 3>();
  if (e != hipSuccess) return e;
  return gemm_once_init();
}

size_t gemm_scratch_floats(int M, int N, int K) {
  return plan_scratch(plan_gemm(M, N, K), M, N);
}

void gemm_plan(int M, int N, int K, int out[5]) {
  const Plan p = plan_gemm(M, N, K);
  out[0] = p.cfg;
  out[1] = p.ksplit;
  out[2] = p.m_main;
  out[3] = p.tail_cfg;
  out[4] = p.tail_ksplit;
}

hipError_t launch_gemm(const GemmArgs& a, size_t ws_floats, hipStream_t stream) {
  return launch_gemm_config(a, ws_floats, -1, 0, stream);
}

int gemm_num_configs() { return kNumShapes; }

namespace {
hipError_t launch_shape(const GemmArgs& a, int cfg, int ksplit, bool reduce, hipStream_t stream) {
  switch (cfg) {
    case 0: return run_shape<256, 256, 128, 64, 4>(a, ksplit, reduce, stream);
    case 1: return run_shape<128, 256, 64, 64, 4>(a, ksplit, reduce, stream);
    case 2: return run_shape<128, 128, 64, 64, 4>(a, ksplit, reduce, stream);
    case 3: return run_shape<64, 128, 32, 64, 4>(a, ksplit, reduce, stream);
    default: return run_shape<128, 256, 64, 64, 3>(a, ksplit, reduce, stream);
  }
}

// A plan whose K split needs more scratch than there is runs that part unsplit.
Plan fit_scratch(Plan p, int M, int N, size_t ws_floats) {
  if (plan_scratch(p, M, N) > ws_floats) {
    if (p.m_main < M)
      p.tail_ksplit = 1;
    else
      p.ksplit = 1;
  }
  return p;
}

// reduce = false: the K split of the last part (the tail rows, or all rows
// without a row split) leaves its fp32 planes at a.partial for the caller.
hipError_t launch_plan(const GemmArgs& a, const Plan& p, bool reduce, hipStream_t stream) {
  if (p.m_main >= a.M) return launch_shape(a, p.cfg, p.ksplit, reduce, stream);
  GemmArgs head = a;
  head.M = p.m_main;
  hipError_t e = launch_shape(head, p.cfg, p.ksplit, true, stream);
  if (e != hipSuccess) return e;
  return launch_shape(rows_from(a, p.m_main), p.tail_cfg, p.tail_ksplit, reduce, stream);
}
}  // namespace

namespace {
// Estimated time (us) of the streaming kernel (gemm_stream.hip): its workgroups read
// whole strips of the weights, so a number of them that leaves CUs out, or out of a
// last round, or a long K for a few of them, costs what a K split of the tiles fills;
// and every strip reads the activations again, up to as many bytes as the weights.
// Fitted to 521 cold problems of 1 to 16 rows (N 1024-57344, K 2048-28672), 7.7% off
// each on average.
double stream_estimate(int M, int N, int K, bool paired) {
  const double strips = paired ? 2 : 1, weights = strips * 32.0 * K;  // bytes of a workgroup
  const double bytes = weights + 0.42 * M * 2.0 * K;
  const double units = N / (16.0 * strips), r = units / kCUs, full = std::floor(r);
  const double rounds = full + (r > full ? 0.57 + 0.43 * (r - full) : 0.0);
  return std::max({rounds * bytes / 33.1e3, bytes / 65.5e3, units * weights / 7.14e6}) + 4.04;
}

// Few rows in the layer's layouts stream the weights where that is faster.  Whole
// 64-column groups keep the paired epilogues' strips inside N; strips are addressed
// with 32-bit byte offsets.  The plans' prices are low at so few rows: against 1.15 of
// them the choice is 0.9% above the best measured on average, always streaming 4.4%,
// never 15% (16 rows: 13B down 38 us streamed, 27 in tiles, 70B qkv 38 and 31, 7B down
// 18.5 and 20.7; one row: 70B qkv 33.6 and 29.3, 13B qkv 25.3 and 28.4).
bool streams(const GemmArgs& a) {
  const bool paired = a.epilogue == EPI_SWIGLU || a.epilogue == EPI_QKV;
  return a.M <= kStreamMaxM && a.a_tiled && a.b_row == 32 && a.N % (paired ? 64 : 16) == 0 &&
         a.K <= (1 << 24) &&
         stream_estimate(a.M, a.N, a.K, paired) <= 1.15 * plan_gemm(a.M, a.N, a.K).t;
}
}  // namespace

hipError_t launch_gemm_config(const GemmArgs& a, size_t ws_floats, int cfg, int ksplit,
                              hipStream_t stream) {
  if (a.M == 0) return hipSuccess;
  if (cfg < 0 && streams(a)) return launch_gemm_stream(a, stream);
  Plan p = plan_gemm(a.M, a.N, a.K);
  if (cfg >= 0 && cfg < kNumShapes) {
    p = Plan{cfg, ksplit >= 1 ? ksplit : 1, a.M, -1, 0, 0.0};
    if (a.K / BK < p.ksplit) return hipErrorInvalidValue;
  }
  return launch_plan(a, fit_scratch(p, a.M, a.N, ws_floats), true, stream);
}

hipError_t launch_gemm_rows(const GemmArgs& a, size_t ws_floats, int m_main, int cfg,
                            int tail_cfg, int tail_ksplit, hipStream_t stream) {
  if (a.M == 0) return hipSuccess;
  if (m_main < 1 || m_main >= a.M || cfg < 0 || cfg >= kNumShapes || tail_cfg < 0 ||
      tail_cfg >= kNumShapes || tail_ksplit < 1 || a.K / BK < tail_ksplit)
    return hipErrorInvalidValue;
  if ((a.a_tiled || a.c_tiled) && m_main % 16) return hipErrorInvalidValue;
  const Plan p{cfg, 1, m_main, tail_cfg, tail_ksplit, 0.0};
  if (plan_scratch(p, a.M, a.N) > ws_floats) return hipErrorInvalidValue;
  return launch_plan(a, p, true, stream);
}

hipError_t launch_gemm_unreduced(const GemmArgs& a, size_t ws_floats, int* split_row, int* ksplit,
                                 hipStream_t stream) {
  *split_row = a.M;
  *ksplit = 1;
  if (a.M == 0) return hipSuccess;
  if (streams(a)) return launch_gemm_stream(a, stream);
  const Plan p = fit_scratch(plan_gemm(a.M, a.N, a.K), a.M, a.N, ws_floats);
  const int ks = p.m_main < a.M ? p.tail_ksplit : p.ksplit;
  if (ks > 1) {
    *split_row = p.m_main < a.M ? p.m_main : 0;
    *ksplit = ks;
  }
  return launch_plan(a, p, false, stream);
}

}  // namespace mx
