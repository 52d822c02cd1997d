// gemm_tile.h -- the workgroup tile of the LDS-tiled GEMM: operand copies, main
// loop and epilogues, as described at the head of gemm.hip.
#pragma once

#include <type_traits>

#include "mx_device.h"
#include "mx_kernels.h"

namespace mx {

constexpr int BK = 64;    // K granularity of a split (and of the problem)
constexpr int BKS = 32;   // K per LDS stage
constexpr int kGroupM = 8;

// LDS ring discipline: the K slices are copied global -> LDS by the DMA path
// and the MFMA fragments read by inline-assembly ds_read_b128, with every wait
// placed by hand (the helpers in mx_device.h).

// Chunk swizzle of LDS row r: 16-byte chunk c is stored at c ^ swz(r).  The
// LDS serves a 16-byte read for 16 lanes at a time from 64 banks, and those are
// not 16 consecutive lanes but {0-3, 12-15, 20-23, 24-27} (then the same + 4 - 8
// ... within the 32, and the upper 32 likewise): in a fragment read they hold
// rows 0-3 and 12-15 at chunk c and rows 4-11 at chunk c ^ 1.  Row r sits in bank
// group 4 (r % 4) + stored chunk, and with (r >> 1) & 3 those 16 are distinct: a
// read takes 4.2 clocks (256 bytes per clock; measured with eight waves reading
// back to back).  The swizzle that is conflict-free for 16 consecutive lanes,
// ((r >> 1) & 3) ^ ((r >> 3) & 1), takes 8.0 clocks, and the 128 x 256 tiles, whose
// 64 x 64 wave tiles read 64 KB per slice, were bound by it: 576 x 12288 x 4096
// 64.3 -> 59.4 us, 2304 x 6144 x 4096 with 128 x 256 tiles 114 -> 106 us, 256 x 256
// tiles (96 KB per slice of twice the products) 0-1%.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 3; }

__device__ __forceinline__ void tile_coords(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int nt = tiles_m * tiles_n;
  const int xcd = bid & 7, local = bid >> 3;
  const int q = nt >> 3, r = nt & 7;
  const int t = xcd * q + min(xcd, r) + local;
  const int group = kGroupM * tiles_n;
  const int gid = t / group;
  const int first_m = gid * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int in_group = t - gid * group;
  tm = first_m + in_group % gm;
  tn = in_group / gm;
}

// Fused QKV epilogue for one rotary pair: packed columns c and c + 32 (c in the
// low 32-column block of a 64-column group) of token row t, fp32 values lo,
// hi, with the token's KV slot and the pair's (cos, sin) already read.  q and k
// heads are rotated (rotate-half pairing, dims d_lo and d_lo + hd/2) and
// rounded once; q goes to q_out, k and v to their slots in the pools.
__device__ __forceinline__ void qkv_pair_store(uint16_t* __restrict__ q_out,
                                               uint16_t* __restrict__ k_pool,
                                               uint16_t* __restrict__ v_pool, int nq, int nkv,
                                               int hd, int t, int c, float lo, float hi,
                                               int64_t slot, float2 cs) {
  const int head = c / hd, within = c % hd;
  if (head < nq + nkv) {
    const int d_lo = 32 * (within / 64) + (within % 32);
    const float rlo = lo * cs.x - hi * cs.y;
    const float rhi = hi * cs.x + lo * cs.y;
    uint16_t* dst;
    int step;  // element distance from dim d_lo to dim d_lo + hd/2
    if (head < nq) {
      dst = q_out + ((int64_t)t * nq + head) * hd + d_lo;
      step = hd / 2;
    } else {
      // key pages blocked by 32 dims: [d / 32][16 slots][32]
      const int64_t page = slot / 16;
      dst = k_pool + (page * nkv + (head - nq)) * 16 * hd + (d_lo / 32) * 512 + (slot % 16) * 32 +
            d_lo % 32;
      step = 8 * hd;
    }
    dst[0] = f32_to_bf16(rlo);
    dst[step] = f32_to_bf16(rhi);
  } else {
    const int64_t page = slot / 16;
    uint16_t* dst = v_pool + ((page * nkv + (head - nq - nkv)) * hd) * 16 + slot % 16;
    dst[(int64_t)within * 16] = f32_to_bf16(lo);
    dst[(int64_t)(within + 32) * 16] = f32_to_bf16(hi);
  }
}

// The (cos, sin) of packed column c (any column of a 64-column group) of
// token t; in bounds for every c (v heads read a row of the table too).
__device__ __forceinline__ int rope_index(int t, int c, int hd) {
  const int within = c % hd;
  return t * (hd / 2) + 32 * (within / 64) + (within % 32);
}

// QKV epilogue of one wave's block (rows r0.., the 64 columns c0..: one
// 64-column group of one head, i.e. the two 32-column halves of its rotary
// pairs).  q and k heads are rotated and rounded once; q goes to q_out, k to
// its pool slot ([d / 32][16 slots][32] pages), v to the transposed value
// pages [page][kv head][dim][16 slots].  Per 32-row block the rounded values
// are staged in LDS, like the outputs of the other epilogues, and written in
// 16-byte runs: q and k read back token-major (8 consecutive dims of one
// token per run), v dim-major, 8 consecutive tokens of one dim per run
// wherever they fill 8 consecutive slots starting at a multiple of 8, in any
// position in the block (a chunk's start need not line up with the rows); the
// tokens left over are stored one value at a time.  Each block first issues
// its reads (this lane's token slot, the rotary cos/sin), so that no wait on
// them also waits for a store (one counter tracks both).
constexpr int kQkRow = 64 + 8;  // bf16 per staged token row (q, k)
constexpr int kVRow = 32 + 8;   // bf16 per staged dim row (v)
constexpr int kQkvStageHalves = 64 * kVRow > 32 * kQkRow ? 64 * kVRow : 32 * kQkRow;

__device__ __forceinline__ int64_t lane_slot(int64_t s, int l) {  // s of lane l (uniform l)
  const int lo = __builtin_amdgcn_readlane((int)(uint32_t)s, l);
  const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)s >> 32), l);
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

template <int MA, int NQ>
__device__ __forceinline__ void qkv_epilogue(const f32x4 (&acc)[MA][NQ], int M, int N, int r0,
                                             int c0, int lane, const float2* __restrict__ rope_cs,
                                             const int64_t* __restrict__ tok_slot,
                                             uint16_t* __restrict__ q_out,
                                             uint16_t* __restrict__ k_pool,
                                             uint16_t* __restrict__ v_pool, int nq, int nkv,
                                             int hd, MX_LDS uint16_t* st) {
  static_assert(NQ == 4, "one 64-column group per wave");
  if (c0 >= N) return;  // (wave-uniform)
  // accumulator layout: block (a, j) holds rows 16 a + crow .. + 3 of column
  // 16 j + ccol in this lane
  const int ccol = lane & 15, crow = 4 * (lane >> 4);
  const int head = c0 / hd, within0 = c0 % hd;
  const bool is_v = head >= nq + nkv, is_q = head < nq;
  // dims of the low and high 32-column blocks (q / k: the packed rotary halves)
  const int d_lo = is_v ? within0 : 32 * (within0 / 64);
  const int d_hi = is_v ? within0 + 32 : d_lo + hd / 2;
#pragma unroll
  for (int i = 0; i < MA / 2; i++) {  // 32-row blocks: accumulator rows 2 i, 2 i + 1
    const int rb = r0 + i * 32;
    // 1. reads: the slot of token rb + lane % 32, the (cos, sin) of this lane's
    // elements (rows 16 h + crow + v, low columns 16 j + ccol, h, j < 2)
    const int64_t myslot = tok_slot[min(rb + (lane & 31), M - 1)];
    float2 cs[16];
    if (!is_v) {
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int h = e >> 3, j = (e >> 2) & 1, v = e & 3;
        const int row = min(rb + 16 * h + crow + v, M - 1);
        cs[e] = rope_cs[(int64_t)row * (hd / 2) + d_lo + 16 * j + ccol];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!is_v) {
      // 2. rotate, round, stage token-major: [token][low 32 dims, high 32 dims]
      // (a pair's halves are columns c and c + 32: blocks j and j + 2, same lane)
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int h = e >> 3, j = (e >> 2) & 1, v = e & 3;
        const int t = 16 * h + crow + v, c = 16 * j + ccol;
        const float lo = acc[2 * i + h][j][v], hi = acc[2 * i + h][j + 2][v];
        st[t * kQkRow + c] = f32_to_bf16(lo * cs[e].x - hi * cs[e].y);
        st[t * kQkRow + 32 + c] = f32_to_bf16(hi * cs[e].x + lo * cs[e].y);
      }
      lgkm_wait<0>();  // (and no access below moves above the staging)
      // 3. read back token (lane / 8) + 8 q, dims 8 (lane % 8) .. + 7 of the 64
      u32x4 out[4];
#pragma unroll
      for (int q = 0; q < 4; q++)
        out[q] = *reinterpret_cast<const MX_LDS u32x4*>(st + ((lane >> 3) + 8 * q) * kQkRow +
                                                        8 * (lane & 7));
      lgkm_wait<0>();  // the block is read back before the next one is staged
      const int p = lane & 7;
      const int dim = (p < 4 ? d_lo : d_hi) + 8 * (p & 3);
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int t = (lane >> 3) + 8 * q;
        const int64_t slot = __shfl(myslot, t);  // (every lane takes part)
        if (rb + t >= M) continue;
        uint16_t* dst;
        if (is_q) {
          dst = q_out + ((int64_t)(rb + t) * nq + head) * hd + dim;
        } else {
          dst = k_pool + ((slot >> 4) * nkv + (head - nq)) * 16 * hd + (dim >> 5) * 512 +
                (slot & 15) * 32 + (dim & 31);
        }
        *reinterpret_cast<u32x4*>(dst) = out[q];
      }
    } else {
      // 2. stage dim-major: [dim (low 32, high 32)][token]; this lane's four
      // consecutive tokens of a block are one 8-byte write
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const f32x4 a = acc[2 * i + h][j];
          u32x2 w;
          w[0] = pack_bf16x2(a[0], a[1]);
          w[1] = pack_bf16x2(a[2], a[3]);
          *reinterpret_cast<MX_LDS u32x2*>(st + (16 * j + ccol) * kVRow + 16 * h + crow) = w;
        }
      lgkm_wait<0>();
      // runs: token t starts one where its slot is a multiple of 8 and token
      // t + 7 holds the slot 7 further (then the eight tokens are consecutive
      // positions of one request: a page belongs to one request)
      const int tl = lane & 31;
      const int64_t s7 = __shfl(myslot, min(tl + 7, 31));
      const bool start = tl + 7 < 32 && rb + tl + 7 < M && (myslot & 7) == 0 && s7 == myslot + 7;
      uint32_t starts = (uint32_t)__ballot(start);
      const int nrow = min(32, M - rb);
      uint32_t single = nrow >= 32 ? ~0u : ((1u << nrow) - 1u);
      for (uint32_t m = starts; m; m &= m - 1) single &= ~(0xFFu << __builtin_ctz(m));
      const int vh = head - nq - nkv;
      const int dim = within0 + lane;  // lane l writes dim row l of the staging
      const MX_LDS uint16_t* srow = st + lane * kVRow;
      for (; starts; starts &= starts - 1) {
        const int t = __builtin_ctz(starts);
        const int64_t slot = lane_slot(myslot, t);
        u32x4 v;
        if ((t & 7) == 0) {
          v = *reinterpret_cast<const MX_LDS u32x4*>(srow + t);
        } else {
#pragma unroll
          for (int e = 0; e < 4; e++) v[e] = (uint32_t)srow[t + 2 * e] | ((uint32_t)srow[t + 2 * e + 1] << 16);
        }
        *reinterpret_cast<u32x4*>(v_pool + (((slot >> 4) * nkv + vh) * hd + dim) * 16 + (slot & 15)) = v;
      }
      for (; single; single &= single - 1) {
        const int t = __builtin_ctz(single);
        const int64_t slot = lane_slot(myslot, t);
        v_pool[(((slot >> 4) * nkv + vh) * hd + dim) * 16 + (slot & 15)] = srow[t];
      }
      lgkm_wait<0>();
    }
  }
}

// Output staging of the plain, residual and SwiGLU epilogues.  The
// matrix-core layout gives a lane one column of four rows per 32 x 32 block, so
// writing it out directly takes one 2-byte store (and one 2-byte residual load)
// per element: 64-128 store instructions per lane per tile, and a CU issues
// about one vector memory instruction per 16 cycles, so the epilogue of a
// 256 x 256 tile cost 5-15 us.  Instead each wave stages one 32-row block of
// its fp32 results at a time in LDS (the operand ring, free once the main loop
// is done) and reads it back as runs of 8 consecutive columns of one row: a
// lane then moves 8 outputs, and 8 residuals, per 16-byte access.  The sums
// and roundings are the same as unstaged.  Staged rows are padded by 4 floats
// so that the rows 4 apart, which one write instruction covers, fall on other
// banks.
constexpr int kStageRow = 64 + 4;              // floats per staged row (64 columns)
constexpr int kStageFloats = 32 * kStageRow;   // one wave's 32-row block
constexpr int kStageRowSw = 32 + 4;            // SwiGLU: 32 output columns per wave

// Plain or residual epilogue of one wave's block (rows r0.., columns c0..,
// 64 columns).  Every residual read (indices clamped into range) is issued
// first, then per 32-row block the staging, the sums rounded to bf16 and the
// stores.  Rows whose stride is not a multiple of 8 elements, and the columns
// at the N edge, take 2-byte accesses.  R must not overlap C.
template <int MA, int NQ, bool RESIDUAL>
__device__ __forceinline__ void store_epilogue(const f32x4 (&acc)[MA][NQ], int M, int N, int r0,
                                               int c0, int lane, const uint16_t* __restrict__ R,
                                               int ldr, uint16_t* __restrict__ C, int ldc,
                                               MX_LDS float* st) {
  static_assert(NQ == 4, "the staging holds 64 columns per wave");
  constexpr int MB = MA / 2;  // 32-row blocks
  const int ccol = lane & 15, crow = 4 * (lane >> 4);  // accumulator layout
  const int rq = lane >> 3, col = c0 + 8 * (lane & 7);  // read-back: rows rq + 8 q, 8 columns
  const bool vec = ldc % 8 == 0 && (!RESIDUAL || ldr % 8 == 0) && col + 8 <= N;
  u32x4 res[MB][4];
#pragma unroll
  for (int i = 0; i < MB; i++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      res[i][q] = u32x4{0, 0, 0, 0};
      if constexpr (RESIDUAL) {
        const uint16_t* rp = R + (int64_t)min(r0 + i * 32 + rq + 8 * q, M - 1) * ldr;
        if (vec) {
          res[i][q] = *reinterpret_cast<const u32x4*>(rp + col);
        } else {
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const uint32_t lo = rp[min(col + e, N - 1)], hi = rp[min(col + e + 1, N - 1)];
            res[i][q][e / 2] = lo | (hi << 16);
          }
        }
      }
    }
#pragma unroll
  for (int i = 0; i < MB; i++) {
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int v = 0; v < 4; v++)
#pragma unroll
        for (int j = 0; j < NQ; j++)
          st[(16 * h + crow + v) * kStageRow + 16 * j + ccol] = acc[2 * i + h][j][v];
    lgkm_wait<0>();  // (and no access below moves above the staging)
    u32x4 out[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const MX_LDS f32x4* sp =
          reinterpret_cast<const MX_LDS f32x4*>(st + (rq + 8 * q) * kStageRow + 8 * (lane & 7));
      const f32x4 lo = sp[0], hi = sp[1];
#pragma unroll
      for (int e = 0; e < 2; e++) {
        out[q][e] = pack_bf16x2(lo[2 * e] + __uint_as_float(res[i][q][e] << 16),
                                lo[2 * e + 1] + __uint_as_float(res[i][q][e] & 0xFFFF0000u));
        out[q][2 + e] = pack_bf16x2(hi[2 * e] + __uint_as_float(res[i][q][2 + e] << 16),
                                    hi[2 * e + 1] + __uint_as_float(res[i][q][2 + e] & 0xFFFF0000u));
      }
    }
    lgkm_wait<0>();  // the block is read back before the next one is staged
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int row = r0 + i * 32 + rq + 8 * q;
      if (row >= M || col >= N) continue;
      uint16_t* cp = C + (int64_t)row * ldc + col;
      if (vec) {
        *reinterpret_cast<u32x4*>(cp) = out[q];
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (col + e < N) cp[e] = (uint16_t)(out[q][e / 2] >> (16 * (e & 1)));
      }
    }
  }
}

// The fp32 partial sums of one K split, through the same staging: 8
// consecutive columns of one row per lane and run, two 16-byte stores (rows
// of N % 4 != 0 floats, and the columns at the N edge, take 4-byte stores).
template <int MA, int NQ>
__device__ __forceinline__ void split_epilogue(const f32x4 (&acc)[MA][NQ], int M, int N, int r0,
                                               int c0, int lane, float* __restrict__ P,
                                               MX_LDS float* st) {
  static_assert(NQ == 4, "the staging holds 64 columns per wave");
  const int ccol = lane & 15, crow = 4 * (lane >> 4);  // accumulator layout
  const int rq = lane >> 3, col = c0 + 8 * (lane & 7);
  const bool vec = N % 4 == 0 && col + 8 <= N;
#pragma unroll
  for (int i = 0; i < MA / 2; i++) {
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int v = 0; v < 4; v++)
#pragma unroll
        for (int j = 0; j < NQ; j++)
          st[(16 * h + crow + v) * kStageRow + 16 * j + ccol] = acc[2 * i + h][j][v];
    lgkm_wait<0>();
    f32x4 lo[4], hi[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const MX_LDS f32x4* sp =
          reinterpret_cast<const MX_LDS f32x4*>(st + (rq + 8 * q) * kStageRow + 8 * (lane & 7));
      lo[q] = sp[0];
      hi[q] = sp[1];
    }
    lgkm_wait<0>();
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int row = r0 + i * 32 + rq + 8 * q;
      if (row >= M || col >= N) continue;
      float* pp = P + (int64_t)row * N + col;
      if (vec) {
        reinterpret_cast<f32x4*>(pp)[0] = lo[q];
        reinterpret_cast<f32x4*>(pp)[1] = hi[q];
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (col + e < N) pp[e] = e < 4 ? lo[q][e] : hi[q][e - 4];
      }
    }
  }
}

// SwiGLU epilogue of one wave's block: packed columns c0.. hold 32-column
// blocks of gate and up of the same 32 features; the 32 outputs (columns
// c0 / 2 ..) go to C row-major or, c_tiled, in the projection-input tile
// layout, through the same staging as above (ldc a multiple of 32).
template <int MA, int NQ>
__device__ __forceinline__ void swiglu_epilogue(const f32x4 (&acc)[MA][NQ], int M, int N, int r0,
                                                int c0, int lane, uint16_t* __restrict__ C,
                                                int ldc, bool c_tiled, MX_LDS float* st) {
  static_assert(NQ == 4, "one gate/up pair per wave");
  // accumulator layout; gate column c pairs with up column c + 32 (blocks j, j + 2)
  const int ccol = lane & 15, crow = 4 * (lane >> 4);
  const int rq = lane >> 2, col = c0 / 2 + 8 * (lane & 3);  // read-back: rows rq + 16 q
  if (c0 >= N) return;  // (wave-uniform)
#pragma unroll
  for (int i = 0; i < MA / 2; i++) {
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int v = 0; v < 4; v++)
#pragma unroll
        for (int j = 0; j < 2; j++)
          st[(16 * h + crow + v) * kStageRowSw + 16 * j + ccol] =
              silu(acc[2 * i + h][j][v]) * acc[2 * i + h][j + 2][v];
    lgkm_wait<0>();
    u32x4 out[2];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const MX_LDS f32x4* sp =
          reinterpret_cast<const MX_LDS f32x4*>(st + (rq + 16 * q) * kStageRowSw + 8 * (lane & 3));
      const f32x4 lo = sp[0], hi = sp[1];
      out[q] = u32x4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]),
                     pack_bf16x2(hi[2], hi[3])};
    }
    lgkm_wait<0>();
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int row = r0 + i * 32 + rq + 16 * q;
      if (row >= M) continue;
      *reinterpret_cast<u32x4*>(C + (c_tiled ? tile_index(row, col, ldc) : (int64_t)row * ldc + col)) =
          out[q];
    }
  }
}

// One workgroup's tile (grid: tiles_m * tiles_n x K splits).  ONCE: B is read
// non-temporally, for launches with one row of tiles, which read it once.
template <int BM, int BN, int WM, int WN, int NS, int EPI, bool SPLIT, bool ONCE>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, int tiles_m, int tiles_n,
                                          int k_chunks) {
  constexpr int WAVES_N = BN / WN;
  constexpr int NWAVES = (BM / WM) * WAVES_N;
  // 16 x 16 output blocks of v_mfma_f32_16x16x32_bf16: MA rows of them per
  // wave, NQ columns; a slice (32 of K) is one product per block
  constexpr int MA = WM / 16, NQ = WN / 16, MH = MA / 2;
  constexpr int ROWB = BKS * 2;                // bytes of one tile row in a stage (64)
  constexpr int STAGE = (BM + BN) * ROWB;      // bytes per LDS stage
  constexpr int L = STAGE / 1024 / NWAVES;     // DMA instructions per wave per stage
  static_assert(L * NWAVES * 1024 == STAGE, "stage does not split into whole DMA rows");
  constexpr int VM_KEEP = (NS - 2) * L;        // in flight after the oldest stage landed
  constexpr int NR0 = NQ + MH;                 // fragment reads of phase 0 (B, first A half)
  constexpr int NR1 = MH;                      // fragment reads of phase 1 (second A half)
  static_assert(MA % 2 == 0 && NQ == 4, "two A halves; 64 columns per wave");
  static_assert(NR0 + NR1 <= 15, "lgkmcnt range");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const unsigned sbase = (unsigned)(size_t)(MX_LDS char*)smem;

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  int tm, tn;
  tile_coords(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int kz = blockIdx.y;
  const int c_beg = kz * k_chunks / (int)gridDim.y, c_end = (kz + 1) * k_chunks / (int)gridDim.y;
  const int kbeg = c_beg * BK;
  const int nk = (c_end - c_beg) * (BK / BKS);

  // DMA: an instruction fills the 16 rows of one block of the stacked A|B tile;
  // lane l lands at row l / 4 of it, stored chunk l % 4, which holds logical chunk
  // (l % 4) ^ swz(row).  Instructions 0 .. LA - 1 of a wave copy A blocks, the
  // others B blocks, so that which operand one reads is known at compile time
  // (ONCE: B is read non-temporally).  Each lane keeps a pointer to its 16 bytes
  // of the next slice to issue, advanced by a scalar step after every issue (no
  // per-slice address multiply), and the LDS destination is scalar arithmetic on
  // the wave index.
  constexpr int LA = BM / 16 / NWAVES, LB = L - LA;
  static_assert(LA * NWAVES * 16 == BM && LB * NWAVES * 16 == BN, "whole blocks per wave");
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const uint16_t* dsrc[L];
  // A element (m, k) at A + (m / 16) a_blk + (m % 16) a_row + (k / 32) a_kstep
  // + k % 32: row-major (16 lda, lda, 32) or the activation tiles
  // (tile_row_pitch(lda), 32, 512), where the 16 rows of an instruction are one
  // contiguous kilobyte
  const int64_t a_blk = a.a_tiled ? tile_row_pitch(a.lda) : 16 * (int64_t)a.lda;
  const int a_row = a.a_tiled ? 32 : a.lda;
  const int64_t a_kstep = a.a_tiled ? 512 : BKS;
  // block of instruction i in the stacked tile
  auto dma_block = [&](int i) { return i < LA ? wave_s * LA + i : BM / 16 + wave_s * LB + i - LA; };
#pragma unroll
  for (int i = 0; i < L; i++) {
    const int row = dma_block(i) * 16 + (lane >> 2);
    const int c = (lane & 3) ^ swz(row);
    if (i < LA) {
      const int m = min(m0 + row, a.M - 1);
      dsrc[i] = a.A + (int64_t)(m >> 4) * a_blk + (int64_t)(m & 15) * a_row +
                (int64_t)(kbeg >> 5) * a_kstep + c * 8;
    } else {
      const int n = min(n0 + row - BM, a.N - 1);
      dsrc[i] = a.B + (int64_t)(n >> 4) * a.b_blk + (int64_t)(n & 15) * a.b_row +
                (int64_t)(kbeg >> 5) * a.b_kstep + c * 8;
    }
  }
  // DMA instruction i of slice st into its LDS slot; slices are issued in
  // order, and past the end the last slice is fetched again (never read)
  auto dma_one = [&](int i, int st) {
    const unsigned slot = sbase + (unsigned)((st % NS) * STAGE);
    if (i >= LA && ONCE)
      dma16<kNonTemporal>(dsrc[i], slot + (unsigned)(dma_block(i) * 1024));
    else
      dma16(dsrc[i], slot + (unsigned)(dma_block(i) * 1024));
    if (st < nk - 1) dsrc[i] += i < LA ? a_kstep : a.b_kstep;
  };

  f32x4 acc[MA][NQ];
#pragma unroll
  for (int i = 0; i < MA; i++)
#pragma unroll
    for (int j = 0; j < NQ; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A fragment of 16-row block a: lane l holds row 16 a + l % 16, logical
  // chunk l / 16 (8 of the slice's 32 K values); B likewise for its columns
  const int frow = lane & 15, fk = lane >> 4;
  unsigned aoff[MA], boff[NQ];
#pragma unroll
  for (int i = 0; i < MA; i++) {
    const int r = wave_m * WM + i * 16 + frow;
    aoff[i] = r * ROWB + (((unsigned)fk ^ swz(r)) << 4);
  }
#pragma unroll
  for (int j = 0; j < NQ; j++) {
    const int r = wave_n * WN + j * 16 + frow;
    boff[j] = (BM + r) * ROWB + (((unsigned)fk ^ swz(r)) << 4);
  }
  // A slice runs in two phases, the first and second half of the wave's A
  // blocks against all its B blocks: fa0 and fa1 hold the two halves, fb[p]
  // the B fragments of slices of parity p (the next slice's arrive while the
  // second phase still uses this one's).
  u32x4 fa0[MH], fa1[MH], fb[2][NQ];
  // phase-0 fragment r of slice st (B first, then the first A half), into fb[p]
  auto read0 = [&](int p, int st, int r) {
    const unsigned slot = sbase + (unsigned)((st % NS) * STAGE);
    if (r < NQ)
      fb[p][r] = lds_read16(slot + boff[r]);
    else
      fa0[r - NQ] = lds_read16(slot + aoff[r - NQ]);
  };
  // phase-1 fragment r of slice st (the second A half)
  auto read1 = [&](int st, int r) {
    const unsigned slot = sbase + (unsigned)((st % NS) * STAGE);
    fa1[r] = lds_read16(slot + aoff[MH + r]);
  };
  constexpr int NM = MH * NQ;  // MFMAs per phase
  auto mfma0 = [&](int p, int idx) {
    const int i = idx / NQ, j = idx % NQ;
    acc[i][j] = mfma16(as_bf16x8(fa0[i]), as_bf16x8(fb[p][j]), acc[i][j]);
  };
  auto mfma1 = [&](int p, int idx) {
    const int i = idx / NQ, j = idx % NQ;
    acc[MH + i][j] = mfma16(as_bf16x8(fa1[i]), as_bf16x8(fb[p][j]), acc[MH + i][j]);
  };

  // One slice (p = kt % 2, a constant at every call): its two phases.  The
  // MFMAs of each phase go out one at a time, with the slice's memory
  // instructions spread between them (the DMA of slice kt + NS - 1 among the
  // first phase's, the next slice's phase-0 fragment reads among the
  // second's), so that a wave keeps the matrix core fed while it issues them:
  // with the instructions in bursts, the two waves of a SIMD, lined up by the
  // barrier, issued theirs at the same time and the matrix core idled
  // meanwhile.  `more` issues the fragment reads of the next slice's first
  // phase.  The last slice must not: the compiler sees the result of a read
  // that is never consumed as dead and may hand its registers to the epilogue
  // while the read is still in flight, and the landing data would then
  // overwrite them.
  auto slice = [&](int kt, bool more, auto parity) {
    constexpr int p = decltype(parity)::value;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < NR1; r++) read1(kt, r);
    lgkm_wait<NR1>();  // the phase-0 fragments (older reads) have landed
    pin(fa0);
    pin(fb[p]);
    // slot (kt + NS - 1) % NS was last read in slice kt - 1, before its barrier
#pragma unroll
    for (int idx = 0; idx < NM; idx++) {
      mfma0(p, idx);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < L; i++)
        if (i * NM / L == idx) dma_one(i, kt + NS - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // (every fragment buffer of a phase stays live across it, so that no
    // read's destination is a register an MFMA of the phase took as a source)
    pin(fa0);
    pin(fb[p]);
    // own DMA of stage kt + 1 landed, own reads of stage kt done; after the
    // barrier everyone's are, so stage kt + 1 is readable and slot kt % NS free
    vm_wait<VM_KEEP>();
    lgkm_wait<0>();
    pin(fa1);
    pin(fb[p]);
    wg_barrier();
#pragma unroll
    for (int idx = 0; idx < NM; idx++) {
      mfma1(p, idx);
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
#pragma unroll
        for (int r = 0; r < NR0; r++)
          if (r * NM / NR0 == idx) read0(p ^ 1, kt + 1, r);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(fa1);
    pin(fb[p]);
  };
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;

#pragma unroll
  for (int st = 0; st < NS - 1; st++)
#pragma unroll
    for (int i = 0; i < L; i++) dma_one(i, st);
  vm_wait<VM_KEEP>();
  wg_barrier();
#pragma unroll
  for (int r = 0; r < NR0; r++) read0(0, 0, r);
  // nk is even (K is a multiple of 64), so slices pair up by parity
  for (int kt = 0; kt < nk - 2; kt += 2) {
    slice(kt, true, P0{});
    slice(kt + 1, true, P1{});
  }
  slice(nk - 2, true, P0{});
  slice(nk - 1, false, P1{});
  // drain: no DMA may still target this workgroup's LDS when it exits (no
  // fragment read is outstanding: the last slice waited for all of them)
  vm_wait<0>();

  // epilogue
  if constexpr (EPI == EPI_QKV && !SPLIT) {
    static_assert(NWAVES * kQkvStageHalves * 2 <= NS * STAGE, "the staging does not fit the ring");
    wg_barrier();  // every wave is done reading the ring
    MX_LDS uint16_t* st =
        reinterpret_cast<MX_LDS uint16_t*>((MX_LDS char*)smem) + wave_s * kQkvStageHalves;
    const QkvEpilogue& e = a.qkv;
    qkv_epilogue<MA, NQ>(acc, a.M, a.N, m0 + wave_m * WM, n0 + wave_n * WN, lane, e.rope_cs,
                         e.tok_slot, e.q_out, e.k_pool, e.v_pool, e.nq, e.nkv, e.head_dim, st);
    return;
  }
  if constexpr (!SPLIT && (EPI == EPI_STORE || EPI == EPI_RESIDUAL || EPI == EPI_SWIGLU)) {
    static_assert(NWAVES * kStageFloats * 4 <= NS * STAGE, "the staging does not fit the ring");
    wg_barrier();  // every wave is done reading the ring
    MX_LDS float* st = reinterpret_cast<MX_LDS float*>((MX_LDS char*)smem) + wave_s * kStageFloats;
    if constexpr (EPI == EPI_SWIGLU)
      swiglu_epilogue<MA, NQ>(acc, a.M, a.N, m0 + wave_m * WM, n0 + wave_n * WN, lane, a.C, a.ldc,
                              a.c_tiled != 0, st);
    else
      store_epilogue<MA, NQ, EPI == EPI_RESIDUAL>(acc, a.M, a.N, m0 + wave_m * WM,
                                                  n0 + wave_n * WN, lane, a.R, a.ldr, a.C, a.ldc,
                                                  st);
    return;
  }
  if constexpr (SPLIT) {  // this split's fp32 plane, [M][N]
    static_assert(NWAVES * kStageFloats * 4 <= NS * STAGE, "the staging does not fit the ring");
    wg_barrier();
    MX_LDS float* st = reinterpret_cast<MX_LDS float*>((MX_LDS char*)smem) + wave_s * kStageFloats;
    split_epilogue<MA, NQ>(acc, a.M, a.N, m0 + wave_m * WM, n0 + wave_n * WN, lane,
                           a.partial + (int64_t)kz * a.M * a.N, st);
  }
}

}  // namespace mx
