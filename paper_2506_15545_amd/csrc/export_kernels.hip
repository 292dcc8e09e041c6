// Prefill -> decode hand-over: from the keys and values of a prompt of T tokens, the rings and the lagged
// linear-attention state a decode step at pos = T reads (Sec. 2.1: the last W keys/values; Sec. 2.2 / Eq. 4: the
// state sum_{s < T-W} phi(k_s)^T v_s).  Keys are split into segments whose partial states are summed in a fixed order;
// the states keep fp32 precision throughout.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace rattn {

namespace {

// ring slot (tok0 + s) % W <- row s of k / v for the last min(T, W) rows (row s is token tok0 + s of its sequence).
// One thread per 16 bytes.
struct RingCopy {
  const uint4 *k, *v;
  uint4 *k_ring, *v_ring;
  int B, T, Hkv, W, row_vecs, tok0;
};
__device__ __forceinline__ void copy_rings(const RingCopy& a, int block, int nblocks) {
  const int first = max(0, a.T - a.W), ntok = a.T - first;
  const long long total = (long long)a.B * ntok * a.Hkv * a.row_vecs;
  for (long long i = (long long)block * 256 + threadIdx.x; i < total; i += (long long)nblocks * 256) {
    const int c = (int)(i % a.row_vecs);
    long long r = i / a.row_vecs;
    const int g = (int)(r % a.Hkv); r /= a.Hkv;
    const int s = first + (int)(r % ntok);
    const int b = (int)(r / ntok);
    const size_t src = ((size_t)(b * a.T + s) * a.Hkv + g) * a.row_vecs + c;
    const size_t dst = (((size_t)b * a.Hkv + g) * a.W + (a.tok0 + s) % a.W) * a.row_vecs + c;
    a.k_ring[dst] = a.k[src];
    a.v_ring[dst] = a.v[src];
  }
}
__global__ __launch_bounds__(256) void export_ring_kernel(RingCopy a) { copy_rings(a, blockIdx.x, gridDim.x); }

// exp(x) for x <= 0, to about one ulp: the rounding of x * log2(e) is carried as a second term (a relative error of
// |x| 2^-24 otherwise)
__device__ __forceinline__ float exp_neg(float x) {
  const float hi = x * LOG2E;
  const float lo = __builtin_fmaf(x, LOG2E, -hi) + x * 1.925963033500e-8f;   // log2(e) - (float)log2(e)
  return fast_exp2(hi) * __builtin_fmaf(lo, LN2, 1.f);
}

// Partial states of key segments for bf16, D = 128, on the bf16 matrix cores without losing the fp32 features: phi(k) is
// split into three bf16 terms (8 + 8 + 8 bits), v is bf16 already, and the three products share one fp32 accumulator.
// One-dimensional grid: block i < nseg * B * Hkv is segment i % nseg of (b, kv head) i / nseg; the others copy the rings.
// Tiles of 64 keys: four threads map a key row (held in registers, requested one tile ahead) into the three LDS tiles of
// phi; V arrives by direct-to-LDS loads, also one tile ahead; wave w then owns features 32w .. of the partial.
// Bound: HBM on long prompts (12 matrix instructions per 16 keys and wave are about 1.6 times as fast as the keys
// arrive), the launch on short ones.
template <int PHI>
__global__ __launch_bounds__(256, 2) void export_state_mfma_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                                   float* __restrict__ partial, int T, int Hkv, int Tp,
                                                                   int nseg, int seg_len, int nstate, RingCopy rc) {
  __shared__ __align__(16) unsigned char smem[5 * 16384];  // phi hi, mid, lo; V x 2
  if ((int)blockIdx.x >= nstate) {
    copy_rings(rc, blockIdx.x - nstate, gridDim.x - nstate);
    return;
  }
  const int seg = blockIdx.x % nseg, bg = blockIdx.x / nseg, g = bg % Hkv, b = bg / Hkv;
  const int lane = lane_id(), w = wave_id(), r32 = lane & 31, h = lane >> 5;
  const int lo = seg * seg_len, hi = min(lo + seg_len, Tp);
  const size_t rstride = (size_t)Hkv * 128;
  const uint16_t* kb = k + ((size_t)b * T * Hkv + g) * 128;
  const uint16_t* vb = v + ((size_t)b * T * Hkv + g) * 128;
  const int row = threadIdx.x >> 2, quarter = threadIdx.x & 3;  // key row and its features 32 * quarter ..
  bf16x8_t kreg[4];
  auto request = [&](int s0, int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // rows 16w + 4i + lane / 16 of the V tile
      const int r = 16 * w + 4 * i + (lane >> 4);
      dma16(vb + (size_t)min(s0 + r, hi - 1) * rstride + (((lane & 15) ^ swz(r)) << 3),
            (unsigned)(size_t)RATTN_LDS(smem + (3 + buf) * 16384 + (4 * w + i) * 1024));
    }
    const uint16_t* kp = kb + (size_t)min(s0 + row, hi - 1) * rstride + 32 * quarter;
#pragma unroll
    for (int c = 0; c < 4; ++c) kreg[c] = *reinterpret_cast<const bf16x8_t*>(kp + 8 * c);
  };
  f32x16_t acc[4] = {{0}, {0}, {0}, {0}};
  request(lo, 0);
  int buf = 0;
  for (int s0 = lo; s0 < hi; s0 += 64, buf ^= 1) {
    float x[32];
#pragma unroll
    for (int c = 0; c < 4; ++c) unpack_bf16x8(kreg[c], &x[8 * c]);
    float inv = 1.f;
    if (PHI == PHI_SOFTMAX) {
      float m = x[0];
#pragma unroll
      for (int i = 1; i < 32; ++i) m = fmaxf(m, x[i]);
      m = fmaxf(m, dpp_get<0xB1>(m));
      m = fmaxf(m, dpp_get<0x4E>(m));
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 32; ++i) { x[i] = exp_neg(x[i] - m); s += x[i]; }
      s += dpp_get<0xB1>(s);
      s += dpp_get<0x4E>(s);
      inv = 1.f / s;
    } else if (PHI == PHI_RELU) {
#pragma unroll
      for (int i = 0; i < 32; ++i) x[i] = fmaxf(x[i], 0.f);
    }
    if (s0 + row >= hi) inv = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float r[8], t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = x[8 * c + e] * inv;
#pragma unroll
      for (int part = 0; part < 3; ++part) {
        const bf16x8_t pk = pack_bf16x8(r);
        *reinterpret_cast<bf16x8_t*>(smem + part * 16384 + row * ROW_BYTES + (((4 * quarter + c) ^ swz(row)) << 4)) = pk;
        unpack_bf16x8(pk, t);
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] -= t[e];  // exact
      }
    }
    wait_vmem();  // this tile's V
    __syncthreads();
    if (s0 + 64 < hi) request(s0 + 64, buf ^ 1);
    const unsigned char* vt = smem + (3 + buf) * 16384;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int k0 = 16 * ks + 8 * h;
      bf16x8_t vop[4];
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) vop[dt] = lds_tr_pair(vt, k0, k0 + 4, 32 * dt, lane);
#pragma unroll
      for (int part = 2; part >= 0; --part) {
        const bf16x8_t a = lds_tr_pair(smem + part * 16384, k0, k0 + 4, 32 * w, lane);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) acc[dt] = mfma32(a, vop[dt], acc[dt]);
      }
    }
    __syncthreads();
  }
  float* out = partial + ((size_t)bg * nseg + seg) * 16384;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) out[(size_t)(32 * w + 8 * (i >> 2) + 4 * h + (i & 3)) * 128 + 32 * dt + r32] = acc[dt][i];
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

void prefill_export(const LayerDims& dm, int dtype, const void* k, const void* v, void* k_ring, void* v_ring,
                    float* state, float* partial, hipStream_t st, int tok0, bool accumulate) {
  const ExportPlan pl = export_plan(dm);
  const int esize = dtype == 0 ? 4 : 2;
  const RingCopy rc = {(const uint4*)k, (const uint4*)v, (uint4*)k_ring, (uint4*)v_ring, dm.B, dm.T, dm.Hkv, dm.W,
                       dm.D * esize / 16, tok0};
  const long long total = (long long)dm.B * (dm.T < dm.W ? dm.T : dm.W) * dm.Hkv * rc.row_vecs;
  const int copy_blocks = (int)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
  if (pl.nseg > 0 && dtype == 1 && dm.D == 128) {
    ProfScope ps("export_state_mfma_kernel", st);
    const int nstate = pl.nseg * dm.Hkv * dm.B;
#define RATTN_EXPORT(PHI_)                                                                                              \
  export_state_mfma_kernel<PHI_><<<nstate + copy_blocks, 256, 0, st>>>((const uint16_t*)k, (const uint16_t*)v, partial, dm.T, \
                                                                       dm.Hkv, pl.Tp, pl.nseg, pl.seg_len, nstate, rc)
    if (dm.phi == PHI_SOFTMAX) RATTN_EXPORT(PHI_SOFTMAX);
    else if (dm.phi == PHI_RELU) RATTN_EXPORT(PHI_RELU);
    else RATTN_EXPORT(PHI_IDENTITY);
#undef RATTN_EXPORT
  } else {
    {
      ProfScope ps("export_ring_kernel", st);
      export_ring_kernel<<<copy_blocks, 256, 0, st>>>(rc);
    }
    if (pl.nseg > 0) generic_chunk_products(dm, dtype, k, v, partial, pl.Tp, pl.nseg, pl.seg_len, st);
  }
  const int vecs = dm.D * dm.D / 4;
  ProfScope ps("export_state_reduce_kernel", st);
  export_state_reduce_kernel<<<dim3(vecs / 64, dm.B * dm.Hkv), 256, 0, st>>>((const float4*)partial, (float4*)state,
                                                                             pl.nseg, vecs, accumulate ? 1 : 0);
}

}  // namespace rattn
