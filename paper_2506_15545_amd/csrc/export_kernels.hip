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
// |x| 2^-24 otherwise).  Below -104 the result is zero in fp32 anyway, and is set: the second term of an x whose product
// overflows (-inf, features at the type's lowest value) is no number.  (NaN stays NaN.)
__device__ __forceinline__ float exp_neg(float x) {
  const float hi = x * LOG2E;
  const float lo = __builtin_fmaf(x, LOG2E, -hi) + x * 1.925963033500e-8f;   // log2(e) - (float)log2(e)
  const float y = fast_exp2(hi) * __builtin_fmaf(lo, LN2, 1.f);
  return x < -104.f ? 0.f : y;
}

// Partial states of key segments for bf16 on the bf16 matrix cores without losing the fp32 features: phi(k) is
// split into three bf16 terms (8 + 8 + 8 bits), v is bf16 already, and the three products share one fp32 accumulator.  The
// other two maps return bf16 values, which one term holds (and an infinite key stays one: inf - inf would not).
// One-dimensional grid: block i < nseg * B * Hkv is segment i % nseg of (b, kv head) i / nseg; the others copy the rings.  Key s is row
// key0 + s of the two-part sequence (SeqRows).
// Tiles of 64 keys: four threads map a key row (held in registers, requested one tile ahead) into the three LDS tiles of
// phi; V arrives by direct-to-LDS loads, also one tile ahead; wave w then owns features 32w .. of the partial (D = 64: one
// of its four 32 x 32 tiles).
// Bound: HBM on long prompts (12 matrix instructions per 16 keys and wave are about 1.6 times as fast as the keys
// arrive), the launch on short ones.
template <int D, int PHI>
__global__ __launch_bounds__(256, 2) void export_state_mfma_kernel(SeqRows k, SeqRows v, float* __restrict__ partial, int Hkv,
                                                                   int key0, int Tp, int nseg, int seg_len, int nstate,
                                                                   RingCopy rc) {
  typedef TileGeom<D> TG;
  constexpr int KT = TG::KT, NB = TG::NB / 4, NX = D / 4, NV = D == 128 ? 4 : 1, NPART = PHI == PHI_SOFTMAX ? 3 : 1;
  __shared__ __align__(16) unsigned char smem[5 * KT];  // phi hi, mid, lo; V x 2
  if ((int)blockIdx.x >= nstate) {
    copy_rings(rc, blockIdx.x - nstate, gridDim.x - nstate);
    return;
  }
  const int seg = blockIdx.x % nseg, bg = blockIdx.x / nseg, g = bg % Hkv, b = bg / Hkv;
  const int lane = lane_id(), w = wave_id(), r32 = lane & 31, h = lane >> 5;
  const int lo = seg * seg_len, hi = min(lo + seg_len, Tp);
  const int row = threadIdx.x >> 2, quarter = threadIdx.x & 3;  // key row and its features D/4 * quarter ..
  const int ft = D == 128 ? w : w & 1, dt0 = D == 128 ? 0 : w >> 1;
  // per-lane offsets of the transposed operand reads (natural contraction order, see lds_trn)
  int aoff[2], voff[NV][2];
#pragma unroll
  for (int ab = 0; ab < 2; ++ab) {
    aoff[ab] = tr_lane_off<D>(8 * h + 4 * ab, ft, lane);
#pragma unroll
    for (int d = 0; d < NV; ++d) voff[d][ab] = tr_lane_off<D>(8 * h + 4 * ab, dt0 + d, lane);
  }
  bf16x8_t kreg[NX / 8];
  auto request = [&](int s0, int buf) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {  // this wave's rows of the V tile
      const int r = (NB * w + i) * TG::RPB + lane / TG::CH;
      dma16(split_rows(v, b, key0 + min(s0 + r, hi - 1), Hkv, g, D).p + (((lane % TG::CH) ^ swz<D>(r)) << 3),
            (unsigned)(size_t)RATTN_LDS(smem + (3 + buf) * KT + (NB * w + i) * 1024));
    }
    const uint16_t* kp = split_rows(k, b, key0 + min(s0 + row, hi - 1), Hkv, g, D).p + NX * quarter;
#pragma unroll
    for (int c = 0; c < NX / 8; ++c) kreg[c] = *reinterpret_cast<const bf16x8_t*>(kp + 8 * c);
  };
  f32x16_t acc[NV];
#pragma unroll
  for (int d = 0; d < NV; ++d) acc[d] = f32x16_t{0};
  request(lo, 0);
  int buf = 0;
  for (int s0 = lo; s0 < hi; s0 += 64, buf ^= 1) {
    float x[NX];
#pragma unroll
    for (int c = 0; c < NX / 8; ++c) unpack_bf16x8(kreg[c], &x[8 * c]);
    float inv = 1.f;
    if (PHI == PHI_SOFTMAX) {
      float m = x[0];
#pragma unroll
      for (int i = 1; i < NX; ++i) m = fmaxf(m, x[i]);
      m = fmaxf(m, dpp_get<0xB1>(m));
      m = fmaxf(m, dpp_get<0x4E>(m));
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NX; ++i) { x[i] = exp_neg(x[i] - m); s += x[i]; }
      s += dpp_get<0xB1>(s);
      s += dpp_get<0x4E>(s);
      inv = 1.f / s;
    } else if (PHI == PHI_RELU) {
#pragma unroll
      for (int i = 0; i < NX; ++i) x[i] = fmaxf(x[i], 0.f);
    }
    const bool none = s0 + row >= hi;  // no key: zero features, whatever the row read in its place holds
#pragma unroll
    for (int c = 0; c < NX / 8; ++c) {
      float r[8], t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = none ? 0.f : x[8 * c + e] * inv;
#pragma unroll
      for (int part = 0; part < NPART; ++part) {
        const bf16x8_t pk = pack_bf16x8(r);
        *reinterpret_cast<bf16x8_t*>(smem + part * KT + row * TG::ROWB + (((NX / 8 * quarter + c) ^ swz<D>(row)) << 4)) = pk;
        unpack_bf16x8(pk, t);
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] -= t[e];  // exact
      }
    }
    wait_vmem();  // this tile's V
    __syncthreads();
    if (s0 + 64 < hi) request(s0 + 64, buf ^ 1);
    const unsigned char* vt = smem + (3 + buf) * KT;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int k0 = 16 * ks * TG::ROWB;
      bf16x8_t vop[NV];
#pragma unroll
      for (int d = 0; d < NV; ++d) vop[d] = lds_tr2(vt + voff[d][0] + k0, vt + voff[d][1] + k0);
#pragma unroll
      for (int part = NPART - 1; part >= 0; --part) {
        const unsigned char* pt = smem + part * KT + k0;
        const bf16x8_t a = lds_tr2(pt + aoff[0], pt + aoff[1]);
#pragma unroll
        for (int d = 0; d < NV; ++d) acc[d] = mfma32(a, vop[d], acc[d]);
      }
    }
    __syncthreads();
  }
  // A sum that is no number may come from a zero feature of the padding, or from terms of phi of different signs, times an
  // infinite or NaN value: such a tile is formed again, key by key in fp32, which has neither.
  float z = 0.f;
#pragma unroll
  for (int d = 0; d < NV; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) z = __builtin_fmaf(acc[d][i], 0.f, z);
  if (__any(z != 0.f)) {  // wave-uniform
#pragma unroll
    for (int d = 0; d < NV; ++d) acc[d] = f32x16_t{0};
    for (int s = lo; s < hi; ++s) {
      const uint16_t* kp = split_rows(k, b, key0 + s, Hkv, g, D).p;
      const uint16_t* vp = split_rows(v, b, key0 + s, Hkv, g, D).p;
      float x[D / 64], f[D / 64], val[NV];
#pragma unroll
      for (int e = 0; e < D / 64; ++e) x[e] = __uint_as_float((uint32_t)kp[lane + 64 * e] << 16);
      feature_row<D / 64>(x, f, PHI);
#pragma unroll
      for (int d = 0; d < NV; ++d) val[d] = __uint_as_float((uint32_t)vp[32 * (dt0 + d) + r32] << 16);
      const float mine = ft < 2 ? f[0] : f[D / 64 - 1];  // this wave's 32 features
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float fi = __shfl(mine, (32 * ft + 8 * (i >> 2) + 4 * h + (i & 3)) & 63);
#pragma unroll
        for (int d = 0; d < NV; ++d) acc[d][i] = __builtin_fmaf(fi, val[d], acc[d][i]);
      }
    }
  }
  float* out = partial + ((size_t)bg * nseg + seg) * (D * D);
#pragma unroll
  for (int d = 0; d < NV; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) out[(size_t)(32 * ft + 8 * (i >> 2) + 4 * h + (i & 3)) * D + 32 * (dt0 + d) + r32] = acc[d][i];
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
  const ExportPlan pl = export_plan(dm);
  const int esize = dtype == 0 ? 4 : 2;
  const RingCopy rc = {(const uint4*)t.k, (const uint4*)t.v, (uint4*)k_ring, (uint4*)v_ring, dm.B, t.Tb, dm.Hkv, dm.W,
                       dm.D * esize / 16, tok0};
  const long long total = (long long)dm.B * (t.Tb < dm.W ? t.Tb : dm.W) * dm.Hkv * rc.row_vecs;
  const int copy_blocks = (int)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
  if (pl.nseg > 0 && dtype == 1) {
    ProfScope ps("export_state_mfma_kernel", st);
    const int nstate = pl.nseg * dm.Hkv * dm.B;
    const SeqRows ks = {(const uint16_t*)t.k_front, (const uint16_t*)t.k, t.P, t.Tb};
    const SeqRows vs = {(const uint16_t*)t.v_front, (const uint16_t*)t.v, t.P, t.Tb};
#define RATTN_EXPORT(D_, PHI_)                                                                                             \
  export_state_mfma_kernel<D_, PHI_><<<nstate + copy_blocks, 256, 0, st>>>(ks, vs, partial, dm.Hkv, t.kmin, pl.Tp, pl.nseg, \
                                                                           pl.seg_len, nstate, rc)
#define RATTN_EXPORT_MAP(D_)                                    \
  if (dm.phi == PHI_SOFTMAX) RATTN_EXPORT(D_, PHI_SOFTMAX);     \
  else if (dm.phi == PHI_RELU) RATTN_EXPORT(D_, PHI_RELU);      \
  else RATTN_EXPORT(D_, PHI_IDENTITY);
    if (dm.D == 64) { RATTN_EXPORT_MAP(64) } else { RATTN_EXPORT_MAP(128) }
#undef RATTN_EXPORT_MAP
#undef RATTN_EXPORT
  } else {
    {
      ProfScope ps("export_ring_kernel", st);
      export_ring_kernel<<<copy_blocks, 256, 0, st>>>(rc);
    }
    if (pl.nseg > 0) generic_chunk_products(dm, t.Tb, t.k, t.v, partial, pl.Tp, pl.nseg, pl.seg_len, st);
  }
  const int vecs = dm.D * dm.D / 4;
  ProfScope ps("export_state_reduce_kernel", st);
  export_state_reduce_kernel<<<dim3(vecs / 64, dm.B * dm.Hkv), 256, 0, st>>>((const float4*)partial, (float4*)state,
                                                                             pl.nseg, vecs, accumulate ? 1 : 0);
}

}  // namespace rattn
