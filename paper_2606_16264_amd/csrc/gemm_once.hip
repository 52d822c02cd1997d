// gemm_once.hip -- the tiled GEMM where M fits one tile, so that every weight is
// read once: non-temporal weight copies, and for 64 x 128 tiles a ring of six
// slices instead of four.  Such launches are bound by the weights' way from HBM.
// Measured with cold weights, each launch by itself (four-slice ring and ordinary
// copies before): 7B gate/up at 64 rows 41.1 -> 34.9 us (38.0 with the ring alone),
// QKV unsplit 36.9 -> 31.1, split in two 27.0 -> 24.9, 13B gate/up at 128 rows 71.6
// -> 65.7, 70B gate/up at 256 rows 223 -> 219.  A K split with many planes gains
// less in the layer than by itself; reads_once() in gemm.hip leaves it out.
#include "gemm_tile.h"
#include "mx_device.h"
#include "mx_kernels.h"

namespace mx {

namespace {

template <int BM, int BN, int WM, int WN, int NS, int EPI, bool SPLIT>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void gemm_once_kernel(GemmArgs a,
                                                                                int tiles_n,
                                                                                int k_chunks) {
  gemm_tile<BM, BN, WM, WN, NS, EPI, SPLIT, true>(a, 1, tiles_n, k_chunks);
}

template <int BM, int BN, int NS>
constexpr size_t lds_bytes() { return (size_t)NS * (BM + BN) * BKS * 2; }

template <int BM, int BN, int WM, int WN, int NS>
hipError_t run(const GemmArgs& a, int ksplit, hipStream_t stream) {
  const int tiles_n = (a.N + BN - 1) / BN, threads = (BM / WM) * (BN / WN) * 64;
  const dim3 grid(tiles_n, ksplit);
  constexpr size_t lds = lds_bytes<BM, BN, NS>();
#define MX_RUN(EPI, SPLIT) \
  gemm_once_kernel<BM, BN, WM, WN, NS, EPI, SPLIT><<<grid, threads, lds, stream>>>(a, tiles_n, a.K / BK)
  if (ksplit > 1)
    MX_RUN(EPI_STORE, true);
  else if (a.epilogue == EPI_QKV)
    MX_RUN(EPI_QKV, false);
  else if (a.epilogue == EPI_SWIGLU)
    MX_RUN(EPI_SWIGLU, false);
  else if (a.epilogue == EPI_RESIDUAL)
    MX_RUN(EPI_RESIDUAL, false);
  else
    MX_RUN(EPI_STORE, false);
#undef MX_RUN
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int NS>
hipError_t init() {
  const void* kernels[] = {
      (const void*)gemm_once_kernel<BM, BN, WM, WN, NS, EPI_STORE, true>,
      (const void*)gemm_once_kernel<BM, BN, WM, WN, NS, EPI_QKV, false>,
      (const void*)gemm_once_kernel<BM, BN, WM, WN, NS, EPI_SWIGLU, false>,
      (const void*)gemm_once_kernel<BM, BN, WM, WN, NS, EPI_RESIDUAL, false>,
      (const void*)gemm_once_kernel<BM, BN, WM, WN, NS, EPI_STORE, false>};
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)lds_bytes<BM, BN, NS>());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t gemm_once_init() {
  hipError_t e = init<64, 128, 32, 64, 6>();
  if (e == hipSuccess) e = init<128, 256, 64, 64, 4>();
  if (e == hipSuccess) e = init<256, 256, 128, 64, 4>();
  return e;
}

bool has_gemm_once(int BM, int BN) { return BN == (BM == 64 ? 128 : 256); }

hipError_t launch_gemm_once(const GemmArgs& a, int BM, int ksplit, hipStream_t stream) {
  switch (BM) {
    case 64: return run<64, 128, 32, 64, 6>(a, ksplit, stream);
    case 128: return run<128, 256, 64, 64, 4>(a, ksplit, stream);
    default: return run<256, 256, 128, 64, 4>(a, ksplit, stream);
  }
}

}  // namespace mx
