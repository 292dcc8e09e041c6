// Prefill -> decode hand-over: from the keys and values of a prompt of T tokens, the rings and the lagged
// linear-attention state a decode step at pos = T reads (Sec. 2.1: the last W keys/values; Sec. 2.2 / Eq. 4: the
// state sum_{s < T-W} phi(k_s)^T v_s).  Keys are split into segments whose partial states are summed in a fixed order;
// the states keep fp32 precision throughout.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "segment_state.hpp"

namespace rattn {

namespace {

// Blocks behind the first ncopy clear the state (nzero 16-byte pieces): no key has left the window.
__global__ __launch_bounds__(256) void export_ring_kernel(RingCopy a, int ncopy, float4* state, long long nzero) {
  if ((int)blockIdx.x < ncopy) {
    copy_rings(a, blockIdx.x, ncopy);
    return;
  }
  for (long long i = (long long)(blockIdx.x - ncopy) * 256 + threadIdx.x; i < nzero; i += (long long)(gridDim.x - ncopy) * 256)
    state[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Partial states of key segments for bf16 (segment_state).
// One-dimensional grid: block i < nseg * B * Hkv is segment i % nseg of (b, kv head) i / nseg; the others copy the rings.  Key s is row
// key0 + s of the two-part sequence (SeqRows).
// Bound: HBM on long prompts (12 matrix instructions per 16 keys and wave are about 1.6 times as fast as the keys
// arrive), the launch on short ones.
// PIECES: the only segment, whose keys are summed `piece` at a time.
template <int D, int PHI, bool PIECES>
__global__ __launch_bounds__(256, 2) void export_state_mfma_kernel(SeqRows k, SeqRows v, float* __restrict__ partial, int Hkv,
                                                                   int key0, int Tp, int nseg, int seg_len, int nstate,
                                                                   RingCopy rc, int piece) {
  __shared__ __align__(16) unsigned char smem[5 * TileGeom<D>::KT];  // phi hi, mid, lo; V x 2
  if ((int)blockIdx.x >= nstate) {
    copy_rings(rc, blockIdx.x - nstate, gridDim.x - nstate);
    return;
  }
  const int seg = blockIdx.x % nseg, bg = blockIdx.x / nseg, g = bg % Hkv, b = bg / Hkv;
  const int lo = seg * seg_len, hi = min(lo + seg_len, Tp);
  const TwoPartRows<D> krow = {k, b, key0, Hkv, g}, vrow = {v, b, key0, Hkv, g};
  segment_state<D, PHI, false, PIECES>(smem, lo, 0, hi, krow, vrow, partial + ((size_t)bg * nseg + seg) * (D * D), piece);
}

// state[b,g] = (accumulate ? state[b,g] : 0) + sum over segments: four runs of segments, each in order, then the four sums
// in order.  grid (vecs / 64, B * Hkv); thread = (run, one float4), eight partials in flight.
__global__ __launch_bounds__(256) void export_state_reduce_kernel(const float4* __restrict__ partial, float4* state,
                                                                  int nseg, int vecs, int accumulate) {
  __shared__ float4 sum[3][64];
  const int run = threadIdx.x >> 6, e = blockIdx.x * 64 + (threadIdx.x & 63);
  const size_t bg = blockIdx.y;
  const int per = (nseg + 3) / 4, c0 = run * per, c1 = min(c0 + per, nseg);
  float4 s = run == 0 && accumulate ? state[bg * vecs + e] : make_float4(0.f, 0.f, 0.f, 0.f);
  const float4* p = partial + bg * nseg * vecs + e;
  for (int c = c0; c < c1; c += 8) {
    float4 u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (c + i < c1) u[i] = p[(size_t)(c + i) * vecs];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (c + i < c1) { s.x += u[i].x; s.y += u[i].y; s.z += u[i].z; s.w += u[i].w; }
  }
  if (run > 0) sum[run - 1][threadIdx.x & 63] = s;
  __syncthreads();
  if (run == 0) {
#pragma unroll
    for (int r = 0; r < 3; ++r) { const float4 t = sum[r][threadIdx.x]; s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w; }
    state[bg * vecs + e] = s;
  }
}

}  // namespace

void prefill_export(const LayerDims& dm, int dtype, const SeqTensors& t, void* k_ring, void* v_ring, float* state,
                    float* partial, hipStream_t st, int tok0, bool accumulate) {
  ExportPlan pl = export_plan(dm);
  const int esize = dtype == 0 ? 4 : 2, tiles = (pl.Tp + 63) / 64;
  const RingCopy rc = {(const uint4*)t.k, (const uint4*)t.v, (uint4*)k_ring, (uint4*)v_ring, dm.B, t.Tb, dm.Hkv, dm.W,
                       dm.D * esize / 16, tok0};
  const long long total = (long long)dm.B * (t.Tb < dm.W ? t.Tb : dm.W) * dm.Hkv * rc.row_vecs;
  const int copy_blocks = (int)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
  if (pl.nseg == 0 && !accumulate) {
    const long long nzero = (long long)dm.B * dm.Hkv * dm.D * dm.D / 4;
    ProfScope ps("export_ring_kernel", st);
    export_ring_kernel<<<copy_blocks + (int)((nzero + 255) / 256 < 2048 ? (nzero + 255) / 256 : 2048), 256, 0, st>>>(
        rc, copy_blocks, (float4*)state, nzero);
    return;
  }
  // Few keys: one segment, straight into the state, saves the launch that sums the segments; the keys of what would be a segment
  // stay a sum of their own, added in the order in which export_state_reduce_kernel adds up to four: the state is the same bits
  // either way.  (One chain over all keys, without those sums: 128 keys at D = 128 1.08e-7 -> 1.34e-7 of the norm off, 320 at
  // D = 64 1.11e-7 -> 1.94e-7.)  Export alone in us, segments and sum | one segment, captured and eager (where the host
  // takes 10 for the two launches one behind the other); pairs of batch and head, keys beyond the window:
  //   bf16, D = 128   4, 64: 7.8 | 6.3, 10.3 | 6.9;  4, 128: 7.9 | 9.4, 10.1 | 9.7;  16, 128: 8.9 | 9.7, 10.5 | 10.0
  //                   64, 128: 13.6 | 10.6, 13.7 | 10.9;  128, 192: 22.6 | 15.1;  128, 320: 23.6 | 20.3;  256, 320: 39 | 25
  //   bf16, D = 64    4, 128: 5.4 | 5.0, 10.4 | 6.9;  4, 192: 5.5 | 6.5, 10.5 | 7.5;  4, 256: 5.5 | 7.9, 10.5 | 9.3
  //                   64, 192: 7.6 | 7.1;  64, 256: 8.1 | 8.6;  128, 320: 11.8 | 10.3
  //   fp32            D = 64: 4, 64: 10.2 | 8.2;  4, 128: 10.3 | 12.7;  128, 128: 17.8 | 19.0;  D = 128: 4, 64: 15.2 | 13.1
  // (With a carried state the sum adds it.)
  const long long pairs = dm.B * (long long)dm.Hkv;
  const int one = dtype == 0 ? 1 : pairs >= 128 ? 5 : dm.D == 64 ? 3 : pairs >= 64 ? 2 : 1;
  const bool direct = !accumulate && tiles <= one;
  const int piece = pl.seg_len;
  if (direct) {
    pl.nseg = 1;
    pl.seg_len = 64 * tiles;
    partial = state;
  }
  if (pl.nseg > 0 && dtype == 1) {
    ProfScope ps("export_state_mfma_kernel", st);
    const int nstate = pl.nseg * dm.Hkv * dm.B;
    const SeqRows ks = {(const uint16_t*)t.k_front, (const uint16_t*)t.k, t.P, t.Tb};
    const SeqRows vs = {(const uint16_t*)t.v_front, (const uint16_t*)t.v, t.P, t.Tb};
#define RATTN_EXPORT_AS(D_, PHI_, PIECES_)                                                                                 \
  export_state_mfma_kernel<D_, PHI_, PIECES_><<<nstate + copy_blocks, 256, 0, st>>>(ks, vs, partial, dm.Hkv, t.kmin, pl.Tp, \
                                                                                    pl.nseg, pl.seg_len, nstate, rc, piece)
#define RATTN_EXPORT(D_, PHI_) \
  do { if (piece < pl.seg_len) RATTN_EXPORT_AS(D_, PHI_, true); else RATTN_EXPORT_AS(D_, PHI_, false); } while (0)
#define RATTN_EXPORT_MAP(D_)                                    \
  if (dm.phi == PHI_SOFTMAX) RATTN_EXPORT(D_, PHI_SOFTMAX);     \
  else if (dm.phi == PHI_RELU) RATTN_EXPORT(D_, PHI_RELU);      \
  else RATTN_EXPORT(D_, PHI_IDENTITY);
    if (dm.D == 64) { RATTN_EXPORT_MAP(64) } else { RATTN_EXPORT_MAP(128) }
#undef RATTN_EXPORT_MAP
#undef RATTN_EXPORT
#undef RATTN_EXPORT_AS
  } else {
    {
      ProfScope ps("export_ring_kernel", st);
      export_ring_kernel<<<copy_blocks, 256, 0, st>>>(rc, copy_blocks, nullptr, 0);
    }
    if (pl.nseg > 0) generic_chunk_products(dm, t.Tb, t.k, t.v, partial, pl.Tp, pl.nseg, pl.seg_len, st);
  }
  if (direct) return;
  const int vecs = dm.D * dm.D / 4;
  ProfScope ps("export_state_reduce_kernel", st);
  export_state_reduce_kernel<<<dim3(vecs / 64, dm.B * dm.Hkv), 256, 0, st>>>((const float4*)partial, (float4*)state,
                                                                             pl.nseg, vecs, accumulate ? 1 : 0);
}

}  // namespace rattn
