// Chunked prefill: the layer's forward for the next Tc tokens of sequences whose first pos0 tokens are only
// present as what the decode path keeps (Sec. 2.1: a ring of the last W keys/values; Sec. 2.2 / Eq. 4: the state
// S0 = sum over s < pos0 - W of phi(k_s)^T v_s).
//
// The sequence that the forward kernels see is [ring tokens in time order ; the new chunk]: every new query then
// finds its whole window, and every key that has left some query's window but is still in the ring, in the
// tensor.  What the tensor does not hold is the contribution of the keys before the ring: the carried state, which is
// the initial value of the forward state scan.  These kernels put the ring rows in time order in front of the chunk.
#include "common.hpp"
#include "kernels.hpp"

namespace rattn {

namespace {

// General kernels: [B, R + Tc, Hkv, D] copies of K and V.  Rows j < R come from the rings (token pos0 - R + j sits in slot
// (pos0 - R + j) % W), rows j >= R from the chunk.  One thread per 16 bytes; `row_vecs` = 16-byte pieces per head row.
__global__ __launch_bounds__(256) void chunk_concat_kernel(const uint4* __restrict__ k, const uint4* __restrict__ v,
                                                           const uint4* __restrict__ k_ring, const uint4* __restrict__ v_ring,
                                                           uint4* __restrict__ kc, uint4* __restrict__ vc, int B, int Tc,
                                                           int R, int Hkv, int W, int pos0, int row_vecs) {
  const int L = R + Tc;
  const long long nkv = (long long)B * L * Hkv * row_vecs;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < nkv; i += (long long)gridDim.x * 256) {
    const int c = (int)(i % row_vecs);
    long long r = i / row_vecs;
    const int g = (int)(r % Hkv); r /= Hkv;
    const int j = (int)(r % L);
    const int b = (int)(r / L);
    if (j < R) {
      const int slot = (pos0 - R + j) % W;
      const size_t src = (((size_t)b * Hkv + g) * W + slot) * row_vecs + c;
      kc[i] = k_ring[src];
      vc[i] = v_ring[src];
    } else {
      const size_t src = ((size_t)(b * Tc + j - R) * Hkv + g) * row_vecs + c;
      kc[i] = k[src];
      vc[i] = v[src];
    }
  }
}

// Matrix-core kernels: only the ring rows, as the whole 128-row tiles [B, P, Hkv, D] that precede the chunk's; the P - R
// rows in front of a ring that does not fill its tiles are zero.
__global__ __launch_bounds__(256) void chunk_ring_kernel(const uint4* __restrict__ k_ring, const uint4* __restrict__ v_ring,
                                                         uint4* __restrict__ kf, uint4* __restrict__ vf, int B, int P, int R,
                                                         int Hkv, int W, int slot0, int row_vecs) {
  // rows a quarter of P apart: four independent pairs of 16-byte copies per thread
  const long long n = (long long)B * Hkv * (P / 4) * row_vecs, i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int c = (int)(i % row_vecs);
  long long r = i / row_vecs;
  const int g = (int)(r % Hkv); r /= Hkv;
  const int j0 = (int)(r % (P / 4)), b = (int)(r / (P / 4));
  uint4 x[4], y[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = j0 + P / 4 * u - (P - R);  // ring row, oldest first
    int slot = slot0 + j;
    slot = slot < W ? slot : slot - W;
    const size_t src = (((size_t)b * Hkv + g) * W + slot) * row_vecs + c;
    x[u] = j >= 0 ? k_ring[src] : make_uint4(0u, 0u, 0u, 0u);
    y[u] = j >= 0 ? v_ring[src] : make_uint4(0u, 0u, 0u, 0u);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const size_t dst = (((size_t)b * P + j0 + P / 4 * u) * Hkv + g) * row_vecs + c;
    kf[dst] = x[u];
    vf[dst] = y[u];
  }
}

}  // namespace

void chunk_concat(const LayerDims& dmc, int dtype, int Tc, int R, int pos0, const void* k, const void* v,
                  const void* k_ring, const void* v_ring, void* kc, void* vc, hipStream_t st) {
  const int row_vecs = dmc.D * (dtype == 0 ? 4 : 2) / 16;
  const long long total = (long long)dmc.B * (R + Tc) * dmc.Hkv * row_vecs;
  const int blocks = (int)((total + 255) / 256 < 16384 ? (total + 255) / 256 : 16384);
  ProfScope ps("chunk_concat_kernel", st);
  chunk_concat_kernel<<<blocks, 256, 0, st>>>((const uint4*)k, (const uint4*)v, (const uint4*)k_ring, (const uint4*)v_ring,
                                              (uint4*)kc, (uint4*)vc, dmc.B, Tc, R, dmc.Hkv, dmc.W, pos0, row_vecs);
}

void chunk_ring(const LayerDims& dmc, int P, int R, int pos0, const void* k_ring, const void* v_ring, void* k_front,
                void* v_front, hipStream_t st) {
  const int row_vecs = dmc.D * 2 / 16;
  const long long n = (long long)dmc.B * dmc.Hkv * (P / 4) * row_vecs;
  ProfScope ps("chunk_ring_kernel", st);
  chunk_ring_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const uint4*)k_ring, (const uint4*)v_ring, (uint4*)k_front, (uint4*)v_front,
                                                     dmc.B, P, R, dmc.Hkv, dmc.W, (pos0 - R) % dmc.W, row_vecs);
}

}  // namespace rattn
