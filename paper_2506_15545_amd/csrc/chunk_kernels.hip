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
#include "mfma.hpp"
#include "segment_state.hpp"

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
// rows in front of a ring that does not fill its tiles are zero.  One thread per four pairs of 16-byte copies, of rows a
// quarter of P apart.
struct RingGather {
  const uint4 *k_ring, *v_ring;
  uint4 *kf, *vf;
  int B, P, R, Hkv, W, slot0, row_vecs;
  int blocks() const { return (int)(((long long)B * Hkv * (P / 4) * row_vecs + 255) / 256); }
};
__device__ __forceinline__ void gather_ring(const RingGather& a, int block) {
  const long long n = (long long)a.B * a.Hkv * (a.P / 4) * a.row_vecs, i = (long long)block * 256 + threadIdx.x;
  if (i >= n) return;
  const int c = (int)(i % a.row_vecs);
  long long r = i / a.row_vecs;
  const int g = (int)(r % a.Hkv); r /= a.Hkv;
  const int j0 = (int)(r % (a.P / 4)), b = (int)(r / (a.P / 4));
  uint4 x[4], y[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = j0 + a.P / 4 * u - (a.P - a.R);  // ring row, oldest first
    int slot = a.slot0 + j;
    slot = slot < a.W ? slot : slot - a.W;
    const size_t src = (((size_t)b * a.Hkv + g) * a.W + slot) * a.row_vecs + c;
    x[u] = j >= 0 ? a.k_ring[src] : make_uint4(0u, 0u, 0u, 0u);
    y[u] = j >= 0 ? a.v_ring[src] : make_uint4(0u, 0u, 0u, 0u);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const size_t dst = (((size_t)b * a.P + j0 + a.P / 4 * u) * a.Hkv + g) * a.row_vecs + c;
    a.kf[dst] = x[u];
    a.vf[dst] = y[u];
  }
}
__global__ __launch_bounds__(256) void chunk_ring_kernel(RingGather a) { gather_ring(a, blockIdx.x); }

// Chunk products and hand-over in one: the states that the forward's query tiles read and the state that the call leaves
// are prefix sums over the same keys, so they come out of the same products (in the precision of the hand-over, which the
// forward's states profit from) and one scan.
// Bound: HBM for large batches, the launches for small ones.  Three launches with the forward instead of six (gather, products,
// scan, forward, products of the hand-over, their sum): 4 x 2048 tokens after 2048, 8 KV heads, W = 512 154 -> 130 us (products
// with the gather 21, scan 12 by the trace), 700 tokens after 1531, 32/8 heads 52.8 -> 41.0 us (9 + 6).

// One-dimensional grid: block i < nprod * Hkv * B forms product i % nprod of (b, kv head) i / nprod, U[..][d][f]; the others
// gather the ring for the forward.  Product 0 of a plan with a head covers rows [0, 64), all others ckeys rows, ended by row
// `end`; rows in front of kmin do not exist.  PIECES: a product of 128 rows is the sum of two of 64.
template <int PHI, bool PIECES>
__global__ __launch_bounds__(256, 2) void chunk_products_kernel(RingRows<128> k, RingRows<128> v, float* __restrict__ U, ChunkPlan pl,
                                                                int nstate, RingGather ga) {
  constexpr int D = 128;
  __shared__ __align__(16) unsigned char smem[5 * TileGeom<D>::KT];
  if ((int)blockIdx.x >= nstate) {
    gather_ring(ga, blockIdx.x - nstate);
    return;
  }
  const int c = blockIdx.x % pl.nprod, bg = blockIdx.x / pl.nprod;
  k.b = v.b = bg / k.H;
  k.g = v.g = bg % k.H;
  const int lo = c < pl.head ? 0 : 64 * pl.head + pl.ckeys * (c - pl.head);
  const int hi = min(c < pl.head ? 64 : lo + pl.ckeys, pl.end);
  segment_state<D, PHI, true, PIECES>(smem, lo, k.kmin, hi, k, v, U + (size_t)blockIdx.x * (D * D), 64);
}

// Block i < nscan: one 32 x 32 tile of (b, kv head): the running sum starts from the carried state (or zero), is stored as
// bf16 [d][f] in front of product head + per i for state i, and after the last product in fp32 [f][d] where the carried
// state was (each element by the thread that read it; both go through LDS, transposed).  Eight products are in flight, and are
// summed in pairs (a remainder in two runs): in one chain, of products of 128 keys in one chain each, the state was up to 1.4 times as far from fp64 as the
// hand-over's own sums (1 x 1300 tokens after 9000, 2 heads, W = 300: 8.5e-8 | 1.20e-7 of the norm, so 6.1e-8).  The other blocks
// copy the chunk's last rows to their ring slots, which nothing reads any more.
__global__ __launch_bounds__(256) void chunk_scan_kernel(const float* __restrict__ U, uint16_t* __restrict__ states, float* state,
                                                         int carried, ChunkPlan pl, int nst, int nscan, RingCopy rc) {
  constexpr int D = 128, NT = (D / 32) * (D / 32);
  __shared__ float tr[32][33];
  if ((int)blockIdx.x >= nscan) {
    copy_rings(rc, blockIdx.x - nscan, gridDim.x - nscan);
    return;
  }
  const int tile = blockIdx.x % NT, bg = blockIdx.x / NT, d0 = 32 * (tile / (D / 32)), f0 = 32 * (tile % (D / 32));
  const int row = threadIdx.x >> 3, c4 = 4 * (threadIdx.x & 7);
  float4* sp = reinterpret_cast<float4*>(state + (size_t)bg * (D * D) + (size_t)(f0 + row) * D + d0 + c4);
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  if (carried) {
    const float4 s = *sp;
    tr[c4][row] = s.x; tr[c4 + 1][row] = s.y; tr[c4 + 2][row] = s.z; tr[c4 + 3][row] = s.w;
    __syncthreads();
    acc = f32x4_t{tr[row][c4], tr[row][c4 + 1], tr[row][c4 + 2], tr[row][c4 + 3]};
    __syncthreads();
  }
  const size_t at = (size_t)(d0 + row) * D + f0 + c4;
  const float* u0 = U + (size_t)bg * pl.nprod * (D * D) + at;
  uint16_t* s0 = states + (size_t)bg * nst * (D * D) + at;
  const int shift = pl.ckeys == 64 ? 1 : 0;   // products per state: 2 or 1
  auto put = [&](int c, f32x4_t f) {   // the state in front of product c, if there is one
    const int n = c - pl.head, i = n >> shift;
    if (n >= 0 && (i << shift) == n && i < nst) *reinterpret_cast<bf16x4_t*>(s0 + (size_t)i * (D * D)) = __builtin_convertvector(f, bf16x4_t);
  };
  auto product = [&](int c) { return *reinterpret_cast<const f32x4_t*>(u0 + (size_t)c * (D * D)); };
  int c0 = 0;
  for (; c0 + 8 <= pl.nprod; c0 += 8) {
    f32x4_t u[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) u[j] = product(c0 + j);
    const f32x4_t u01 = u[0] + u[1], u03 = u01 + (u[2] + u[3]), u45 = u[4] + u[5];
    const f32x4_t f[8] = {acc, acc + u[0], acc + u01, acc + (u01 + u[2]), acc + u03, acc + (u03 + u[4]), acc + (u03 + u45),
                          acc + (u03 + (u45 + u[6]))};
#pragma unroll
    for (int j = 0; j < 8; ++j) put(c0 + j, f[j]);
    acc += u03 + (u45 + (u[6] + u[7]));
  }
  if (c0 < pl.nprod) {   // up to seven more, in two runs (with few products the instructions of eight are what takes the time)
    f32x4_t u[7], a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (c0 + j < pl.nprod) u[j] = product(c0 + j);
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      if (c0 + j >= pl.nprod) break;
      put(c0 + j, j == 0 ? acc : j <= 4 ? acc + a : acc + (a + b));
      if (j < 4) a += u[j]; else b += u[j];
    }
    acc += a + b;
  }
  tr[c4][row] = acc[0]; tr[c4 + 1][row] = acc[1]; tr[c4 + 2][row] = acc[2]; tr[c4 + 3][row] = acc[3];
  __syncthreads();
  *sp = make_float4(tr[row][c4], tr[row][c4 + 1], tr[row][c4 + 2], tr[row][c4 + 3]);
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
  const RingGather ga = {(const uint4*)k_ring, (const uint4*)v_ring, (uint4*)k_front, (uint4*)v_front, dmc.B, P, R, dmc.Hkv, dmc.W,
                         (pos0 - R) % dmc.W, dmc.D * 2 / 16};
  ProfScope ps("chunk_ring_kernel", st);
  chunk_ring_kernel<<<ga.blocks(), 256, 0, st>>>(ga);
}

void chunk_states(const LayerDims& dm, const SeqTensors& t, float* U, void* states, hipStream_t st) {
  const ChunkHandover& h = *t.handover;
  const ChunkPlan& pl = h.plan;
  const int slot0 = (h.pos0 - h.R) % dm.W, nst = fast_fwd_plan(dm).nstf, row_vecs = 128 * 2 / 16;
  {
    const RingGather ga = {(const uint4*)h.k_ring, (const uint4*)h.v_ring, (uint4*)t.k_front, (uint4*)t.v_front, dm.B, t.P, h.R,
                           dm.Hkv, dm.W, slot0, row_vecs};
    RingRows<128> k = {(const uint16_t*)h.k_ring, (const uint16_t*)t.k, 0, 0, dm.Hkv, dm.W, slot0, t.kmin, t.P, t.Tb}, v = k;
    v.ring = (const uint16_t*)h.v_ring;
    v.back = (const uint16_t*)t.v;
    const int nstate = pl.nprod * dm.Hkv * dm.B;
    ProfScope ps("chunk_products_kernel", st);
#define RATTN_PRODUCTS(PHI_)                                                                                              \
  do {                                                                                                                   \
    if (pl.piece < pl.ckeys) chunk_products_kernel<PHI_, true><<<nstate + ga.blocks(), 256, 0, st>>>(k, v, U, pl, nstate, ga); \
    else chunk_products_kernel<PHI_, false><<<nstate + ga.blocks(), 256, 0, st>>>(k, v, U, pl, nstate, ga);               \
  } while (0)
    if (dm.phi == PHI_RELU) RATTN_PRODUCTS(PHI_RELU); else RATTN_PRODUCTS(PHI_SOFTMAX);
#undef RATTN_PRODUCTS
  }
  const RingCopy rc = {(const uint4*)t.k, (const uint4*)t.v, (uint4*)h.k_ring, (uint4*)h.v_ring, dm.B, t.Tb, dm.Hkv, dm.W,
                       row_vecs, h.pos0};
  const long long total = (long long)dm.B * (t.Tb < dm.W ? t.Tb : dm.W) * dm.Hkv * row_vecs;
  const int copy_blocks = (int)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048), nscan = 16 * dm.Hkv * dm.B;
  ProfScope ps("chunk_scan_kernel", st);
  chunk_scan_kernel<<<nscan + copy_blocks, 256, 0, st>>>(U, (uint16_t*)states, h.state, h.carried, pl, nst, nscan, rc);
}

}  // namespace rattn
