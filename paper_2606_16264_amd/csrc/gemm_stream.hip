// gemm_stream.hip -- the projections of a few rows (M <= kStreamMaxM = 16, where
// streams() in gemm.hip prices it below the tiled kernels): the weights stream from
// HBM once and bound the time, so nothing is shared through LDS and no K split
// leaves the kernel.  Operands in the layer's own layouts
// (packed weights and activations in 16 x 32 tiles of 1 KB), where one load
// instruction of a wave reads one whole tile in the register layout of
// v_mfma_f32_16x16x32_bf16.
//
//  - A workgroup owns NT 16-row strips of the weights over all of K.  Its four
//    waves take every fourth 32-wide K step and add up their sums through LDS at
//    the end, in wave order, before the epilogue: no partial planes and no
//    reduce launch.
//  - Per step a wave loads its NT weight tiles and the activation tile (from L2,
//    where every workgroup finds it) straight into registers, kDepth = 8 steps
//    ahead.
//  - Buffer loads bound every strip by its own end: steps past K return zeros and
//    move nothing, so the loop has no tail and no branch around a load.
//  - The product is taken transposed (weights as the A operand): a lane holds
//    four consecutive columns of one token, one 8-byte store.
//
// Measured with cold weights in the layer, one row and 16, against the tiled kernels
// with their K split's reduce: 7B qkv 26.1 -> 21.8 and 28.0 -> 24.4 us, gate/up 39.7 ->
// 31.8 and 42.1 -> 33.8, down 21.7 -> 17.5 and 22.8 -> 20.3; 8B qkv 19.5 -> 12.3 and 17.2
// -> 14.0; 70B o 25.7 -> 23.1.  Where the strips do not fill the CUs evenly, or at 16
// rows over a long K, the tiles win and run instead: 70B qkv 36.3 against 34.4 at one
// row, 40.7 against 34.2 at 16, 13B down 31.5 against 28.3 and 40.3 against 29.6.  Eight
// waves per workgroup or a depth of 16 are slower wherever the strips do not fill the
// CUs evenly (7B qkv 24.2, 13B qkv 42.8), a shallower ring at large K (70B qkv 44).
// Two activation tiles per step (17-32 rows) cost 5-10 us more each and lose to
// the tiled kernels, whose LDS tile reads the activations once per 128 rows (13B
// qkv 45.7 against 32.7 us).
#include "mx_device.h"
#include "mx_kernels.h"

namespace mx {

namespace {

constexpr int kBufferWord3 = 0x00020000;  // raw buffer descriptor, 32-bit data format

constexpr int kWaves = 4, kDepth = 8;

// 16 bytes at byte offset `off` of the resource, zeros past its end.
template <int POLICY>
__device__ __forceinline__ u32x4 buffer_read16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POLICY));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t resource(const uint16_t* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, bytes, kBufferWord3);
}

template <int NT, int EPI>
__global__ __launch_bounds__(kWaves * 64) void gemm_stream_kernel(GemmArgs a) {
  constexpr bool PAIRED = EPI == EPI_SWIGLU || EPI == EPI_QKV;
  static_assert(!PAIRED || NT == 2, "a pair of strips 32 columns apart");
  __shared__ __attribute__((aligned(16))) f32x4 red[kWaves][NT][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x;
  auto strip = [&](int i) { return PAIRED ? 4 * (unit >> 1) + (unit & 1) + 2 * i : unit * NT + i; };
  const int steps = a.K / 32;
  // a strip, and the tile row of the activations: a step is 1 KB further in either
  __amdgpu_buffer_rsrc_t wr[NT];
#pragma unroll
  for (int i = 0; i < NT; i++) wr[i] = resource(a.B + (int64_t)strip(i) * 16 * a.K, 32 * a.K);
  const __amdgpu_buffer_rsrc_t xr = resource(a.A, 32 * a.K);
  const int lane_off = (lane & 15) * 64 + (lane >> 4) * 16;  // this lane's 16 bytes of a tile
  // activation rows past M lie in the padding of the tile row: their products
  // stay in their own columns, which are not written; row M - 1 stands in
  const int x_off = min(lane & 15, a.M - 1) * 64 + (lane >> 4) * 16;

  f32x4 acc[NT];
#pragma unroll
  for (int i = 0; i < NT; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 wf[kDepth][NT], xf[kDepth];
  // (the loads stay in step order, so that the wait before a step's products
  // covers that step alone)
  auto load = [&](int slot, int step) {
#pragma unroll
    for (int i = 0; i < NT; i++)
      wf[slot][i] = buffer_read16<kNonTemporal>(wr[i], lane_off + step * 1024);
    xf[slot] = buffer_read16<0>(xr, x_off + step * 1024);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int j = 0; j < kDepth; j++) load(j, wave + j * kWaves);
  for (int s = wave; s < steps; s += kDepth * kWaves) {
#pragma unroll
    for (int j = 0; j < kDepth; j++) {
#pragma unroll
      for (int i = 0; i < NT; i++) acc[i] = mfma16(as_bf16x8(wf[j][i]), as_bf16x8(xf[j]), acc[i]);
      __builtin_amdgcn_sched_barrier(0);
      load(j, s + (j + kDepth) * kWaves);
    }
  }

#pragma unroll
  for (int i = 0; i < NT; i++) red[wave][i][lane] = acc[i];
  __syncthreads();
  // wave 0 finishes: this lane's sums of strip i are columns 16 strip(i) + 4 (lane
  // / 16) .. + 3 of token lane % 16
  if (wave != 0) return;
  auto total = [&](int i) {
    f32x4 v = red[0][i][lane];
#pragma unroll
    for (int w = 1; w < kWaves; w++) v += red[w][i][lane];
    return v;
  };
  const int t = lane & 15;
  if (t >= a.M) return;
  const int quad = 4 * (lane >> 4);
  if constexpr (PAIRED) {
    const f32x4 lo = total(0), hi = total(1);
    const int c = 16 * strip(0) + quad;  // packed column; its partner is c + 32
    if constexpr (EPI == EPI_SWIGLU) {
      const int f = 32 * (c / 64) + c % 64;  // feature: the gate block's own column
      u32x2 w;
      w[0] = pack_bf16x2(silu(lo[0]) * hi[0], silu(lo[1]) * hi[1]);
      w[1] = pack_bf16x2(silu(lo[2]) * hi[2], silu(lo[3]) * hi[3]);
      *reinterpret_cast<u32x2*>(
          a.C + (a.c_tiled ? tile_index(t, f, a.ldc) : (int64_t)t * a.ldc + f)) = w;
    } else {
      const QkvEpilogue& e = a.qkv;
      const int hd = e.head_dim, head = c / hd, within = c % hd;
      const int64_t slot = e.tok_slot[t];
      if (head < e.nq + e.nkv) {
        const int d_lo = 32 * (within / 64) + within % 32;
        const f32x4* cs =
            reinterpret_cast<const f32x4*>(e.rope_cs + (int64_t)t * (hd / 2) + d_lo);
        const f32x4 c01 = cs[0], c23 = cs[1];  // (cos, sin) of four dims
        const float co[4] = {c01[0], c01[2], c23[0], c23[2]};
        const float si[4] = {c01[1], c01[3], c23[1], c23[3]};
        float rl[4], rh[4];
#pragma unroll
        for (int v = 0; v < 4; v++) {
          rl[v] = lo[v] * co[v] - hi[v] * si[v];
          rh[v] = hi[v] * co[v] + lo[v] * si[v];
        }
        uint16_t* dst;
        int step;  // from dim d_lo to dim d_lo + hd / 2
        if (head < e.nq) {
          dst = e.q_out + ((int64_t)t * e.nq + head) * hd + d_lo;
          step = hd / 2;
        } else {
          dst = e.k_pool + ((slot >> 4) * e.nkv + (head - e.nq)) * 16 * hd + (d_lo / 32) * 512 +
                (slot & 15) * 32 + d_lo % 32;
          step = 8 * hd;
        }
        *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16x2(rl[0], rl[1]), pack_bf16x2(rl[2], rl[3])};
        *reinterpret_cast<u32x2*>(dst + step) =
            u32x2{pack_bf16x2(rh[0], rh[1]), pack_bf16x2(rh[2], rh[3])};
      } else {
        uint16_t* dst = e.v_pool +
                        (((slot >> 4) * e.nkv + (head - e.nq - e.nkv)) * hd + within) * 16 +
                        (slot & 15);
#pragma unroll
        for (int v = 0; v < 4; v++) {
          dst[v * 16] = f32_to_bf16(lo[v]);
          dst[(v + 32) * 16] = f32_to_bf16(hi[v]);
        }
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NT; i++) {
      f32x4 v = total(i);
      const int c = 16 * strip(i) + quad;
      if constexpr (EPI == EPI_RESIDUAL) {
        const u32x2 r = *reinterpret_cast<const u32x2*>(a.R + (int64_t)t * a.ldr + c);
        v[0] += __uint_as_float(r[0] << 16);
        v[1] += __uint_as_float(r[0] & 0xFFFF0000u);
        v[2] += __uint_as_float(r[1] << 16);
        v[3] += __uint_as_float(r[1] & 0xFFFF0000u);
      }
      *reinterpret_cast<u32x2*>(a.C + (int64_t)t * a.ldc + c) =
          u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    }
  }
}

}  // namespace

hipError_t launch_gemm_stream(const GemmArgs& a, hipStream_t stream) {
  constexpr int threads = kWaves * 64;
  switch (a.epilogue) {
    case EPI_QKV: gemm_stream_kernel<2, EPI_QKV><<<a.N / 32, threads, 0, stream>>>(a); break;
    case EPI_SWIGLU: gemm_stream_kernel<2, EPI_SWIGLU><<<a.N / 32, threads, 0, stream>>>(a); break;
    case EPI_RESIDUAL: gemm_stream_kernel<1, EPI_RESIDUAL><<<a.N / 16, threads, 0, stream>>>(a); break;
    default: gemm_stream_kernel<1, EPI_STORE><<<a.N / 16, threads, 0, stream>>>(a); break;
  }
  return hipGetLastError();
}

}  // namespace mx
