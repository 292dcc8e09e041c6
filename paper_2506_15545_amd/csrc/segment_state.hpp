// Partial linear-branch states of a segment of keys in fp32 precision (bf16 tensors), and the copy of rows into ring slots:
// what the prefill export and chunked prefill have in common.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace rattn {

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
// exp(x) for x <= 0, to about one ulp: the rounding of x * log2(e) is carried as a second term (a relative error of
// |x| 2^-24 otherwise).  Below -104 the result is zero in fp32 anyway, and is set: the second term of an x whose product
// overflows (-inf, features at the type's lowest value) is no number.  (NaN stays NaN.)
__device__ __forceinline__ float exp_neg(float x) {
  const float hi = x * LOG2E;
  const float lo = __builtin_fmaf(x, LOG2E, -hi) + x * 1.925963033500e-8f;   // log2(e) - (float)log2(e)
  const float y = fast_exp2(hi) * __builtin_fmaf(lo, LN2, 1.f);
  return x < -104.f ? 0.f : y;
}

// Rows of one head, as segment_state takes them: from row key0 of a two-part sequence on ...
template <int D> struct TwoPartRows {
  SeqRows s;
  int b, key0, H, g;
  __device__ __forceinline__ const uint16_t* operator()(int r) const { return split_rows(s, b, key0 + r, H, g, D).p; }
};
// ... or of a ring in time order (row kmin sits in slot slot0; rows in front of it are read as that one) followed from row P
// on by a chunk of Tb rows
template <int D> struct RingRows {
  const uint16_t *ring, *back;
  int b, g, H, W, slot0, kmin, P, Tb;
  __device__ __forceinline__ const uint16_t* operator()(int r) const {
    if (r >= P) return back + ((size_t)((size_t)b * Tb + (r - P)) * H + g) * D;
    const int slot = slot0 + max(r - kmin, 0);
    return ring + ((size_t)((size_t)b * H + g) * W + (slot < W ? slot : slot - W)) * D;
  }
};

// One work-group (256 threads): the partial state of keys lo .. hi-1, of which those below `first` do not exist (they add
// nothing, whatever is read in their place).  krow(s), vrow(s): row s of one head, called with lo <= s < hi.
// phi(k) of the softmax map is split into three bf16 terms (8 + 8 + 8 bits), v is bf16 already, and the three products share
// one fp32 accumulator.  The other two maps give bf16 values, which one term holds (and an infinite key stays one: inf - inf
// would not).
// Tiles of 64 keys: four threads map a key row (held in registers, requested one tile ahead) into the three LDS tiles of
// phi; V arrives by direct-to-LDS loads, also one tile ahead; wave w then owns features 32w .. of the partial (D = 64: one
// of its four 32 x 32 tiles).  smem: 5 tiles of 64 rows.  out: [f][d], or [d][f] when TRANSPOSED.
// PIECES: every `piece` keys (a multiple of 64) are a sum of their own, and those are added in order: rounding grows with the
// length of an accumulator's chain.
template <int D, int PHI, bool TRANSPOSED, bool PIECES, typename KR, typename VR>
__device__ __forceinline__ void segment_state(unsigned char* smem, int lo, int first, int hi, KR krow, VR vrow, float* out,
                                              int piece = 0) {
  typedef TileGeom<D> TG;
  constexpr int KT = TG::KT, NB = TG::NB / 4, NX = D / 4, NV = D == 128 ? 4 : 1, NPART = PHI == PHI_SOFTMAX ? 3 : 1;
  const int lane = lane_id(), w = wave_id(), r32 = lane & 31, h = lane >> 5;
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
      dma16(vrow(min(s0 + r, hi - 1)) + (((lane % TG::CH) ^ swz<D>(r)) << 3),
            (unsigned)(size_t)RATTN_LDS(smem + (3 + buf) * KT + (NB * w + i) * 1024));
    }
    const uint16_t* kp = krow(min(s0 + row, hi - 1)) + NX * quarter;
#pragma unroll
    for (int c = 0; c < NX / 8; ++c) kreg[c] = *reinterpret_cast<const bf16x8_t*>(kp + 8 * c);
  };
  f32x16_t acc[NV], sum[NV];
#pragma unroll
  for (int d = 0; d < NV; ++d) acc[d] = sum[d] = f32x16_t{0};
  // A sum (of keys a .. b-1) that is no number may come from a zero feature of the padding, or from terms of phi of different
  // signs, times an infinite or NaN value: such a tile is formed again, key by key in fp32, which has neither.
  auto settle = [&](int a, int b) {
    float z = 0.f;
#pragma unroll
    for (int d = 0; d < NV; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) z = __builtin_fmaf(acc[d][i], 0.f, z);
    if (!__any(z != 0.f)) return;  // wave-uniform
#pragma unroll
    for (int d = 0; d < NV; ++d) acc[d] = f32x16_t{0};
    for (int s = max(a, first); s < b; ++s) {
      const uint16_t *kp = krow(s), *vp = vrow(s);
      float x[D / 64], f[D / 64];
#pragma unroll
      for (int e = 0; e < D / 64; ++e) x[e] = __uint_as_float((uint32_t)kp[lane + 64 * e] << 16);
      feature_row<D / 64>(x, f, PHI);
      const float mine = ft < 2 ? f[0] : f[D / 64 - 1];  // this wave's 32 features
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = 8 * (i >> 2) + 4 * h + (i & 3);
        const float fi = __shfl(mine, (32 * ft + (TRANSPOSED ? r32 : r)) & 63);
#pragma unroll
        for (int d = 0; d < NV; ++d)
          acc[d][i] = __builtin_fmaf(fi, __uint_as_float((uint32_t)vp[32 * (dt0 + d) + (TRANSPOSED ? r : r32)] << 16), acc[d][i]);
      }
    }
  };
  request(lo, 0);
  int buf = 0, piece_lo = lo;
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
    const bool none = s0 + row >= hi || s0 + row < first;  // no key: zero features, whatever the row read in its place holds
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
        for (int d = 0; d < NV; ++d) acc[d] = TRANSPOSED ? mfma32(vop[d], a, acc[d]) : mfma32(a, vop[d], acc[d]);
      }
    }
    __syncthreads();
    if (PIECES && (s0 + 64 >= hi || s0 + 64 - piece_lo == piece)) {
      settle(piece_lo, min(s0 + 64, hi));
      piece_lo = s0 + 64;
#pragma unroll
      for (int d = 0; d < NV; ++d) { sum[d] += acc[d]; acc[d] = f32x16_t{0}; }
    }
  }
  if (!PIECES) settle(lo, hi);
#pragma unroll
  for (int d = 0; d < NV; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = 8 * (i >> 2) + 4 * h + (i & 3);
      out[TRANSPOSED ? (size_t)(32 * (dt0 + d) + r) * D + 32 * ft + r32 : (size_t)(32 * ft + r) * D + 32 * (dt0 + d) + r32] = PIECES ? sum[d][i] : acc[d][i];
    }
}

}  // namespace rattn
