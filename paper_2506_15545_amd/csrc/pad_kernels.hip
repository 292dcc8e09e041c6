// The rows of dO past the last whole tile, for the matrix-core backward kernels.
#include "common.hpp"
#include "kernels.hpp"

namespace rattn {

namespace {

// One thread per 16 bytes of the [B,128,H,D] tail buffer (hv vectors per head row): rows Tfull + r of the [B,T,H,D] bf16
// tensor, zero where Tfull + r >= T.
__global__ __launch_bounds__(256) void tail_rows_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int B, int T,
                                                        int Tfull, int H, int hv) {
  const long long total = (long long)B * 128 * H * hv;
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long long)gridDim.x * 256) {
    long long r = e / ((long long)H * hv);
    const int c = (int)(e - r * H * hv);
    const int row = (int)(r & 127), b = (int)(r >> 7);
    dst[e] = Tfull + row < T ? src[((long long)b * T + Tfull + row) * H * hv + c] : make_uint4(0u, 0u, 0u, 0u);
  }
}

}  // namespace

void gather_tail(const void* src, void* tail, int B, int T, int H, int D, hipStream_t st) {
  const int hv = D / 8;
  const long long n = ((long long)B * 128 * H * hv + 255) / 256;
  ProfScope ps("tail_rows_kernel(gather)", st);
  tail_rows_kernel<<<(unsigned)(n < 16384 ? n : 16384), 256, 0, st>>>((const uint4*)src, (uint4*)tail, B, T, T / 128 * 128, H, hv);
}

}  // namespace rattn
