// General-shape kernels of librattn: any T, any window W >= 1, D in {64,128}, fp32 or bf16 tensors, fp32 arithmetic
// throughout.  They serve fp32 tensors and every shape the bf16 matrix-core kernels do not cover, by the same
// decomposition:
//   softmax branch  : Sec. 2.1 (windowed softmax, online normalisation)
//   linear branch   : Eqs. 2-4 (chunk states S_[j], inter-chunk product + intra-chunk masked product, read at lag W),
//                     phi (row softmax, or the ablation's ReLU / identity of Sec. 4.5) computed in-kernel, never stored
//   combination     : Sec. 3.2 (two RMS norms with per-head gains)
//
// All contractions run on v_mfma_f32_16x16x4_f32 (exact fp32 products, fp32 sums).  A work-group of four waves owns 16
// query rows (forward, dq) or 16 key rows (dk/dv); the waves share the rows of the other side between them, 16 at a
// time, and add up their partial results in LDS at the end.  Inside a wave everything is transposed, as in the bf16
// kernels: the owned rows are the columns of the tiles (lane = 16*q4 + r16 holds column r16, register i row 4*q4 + i).
// The order of a contraction is free as long as both operands follow it, which lets every operand be loaded from global
// memory (L1/L2: neighbouring waves share the rows) as 16-byte pieces in one of two forms, without LDS:
//   row form     x[j][e]     = row r16,      feature 16j + 4*q4 + e        (contraction over features)
//   column form  x[i][hf][e] = row 4*q4 + i, feature 64hf + 4*r16 + e      (contraction over rows)
// A column-form product leaves feature 64hf + 4*(4*q4 + i) + e of column r16 in acc[4*hf + e][i].
//
// Bound: launch latency and the dependent chain of a wave on small tensors, the fp32 matrix rate (157 TFLOP/s; a tile
// takes 32 cycles, so operands out of L1 keep up) on large ones.  Measured, fp32, one sequence of T = 256, 2 heads,
// D = 64, W = 32, forward + backward: 42 us in three launches of eight waves per work-group; with states of 64 keys
// and four waves 51 us in seven launches, with one wave per row and vector arithmetic 427 us.
//
// The other side's 16-row tiles are dealt out to the waves; a wave requests its next tile behind the products of this one
// (D = 64; at D = 128 the backward kernels have no registers for that), and where both forms of the same rows are needed
// the column form comes out of the row form through LDS instead of a second trip to memory: backward of 2 x 512 tokens, 2 x 2
// heads, W = 128 61.0 -> 49.4 us at D = 64, 110.2 -> 91.0 at D = 128 (with eight waves, the same states).
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace rattn {

namespace {

constexpr int GWC = 4;  // waves per work-group of the chunk products

__device__ __forceinline__ f32x4_t mm4(float a, float b, f32x4_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ f32x4_t load4(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }
__device__ __forceinline__ f32x4_t load4(const bf16_t* p) {
  const uint2 r = *reinterpret_cast<const uint2*>(p);
  return f32x4_t{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float* p, f32x4_t v) { *reinterpret_cast<f32x4_t*>(p) = v; }
__device__ __forceinline__ void store4(bf16_t* p, f32x4_t v) {
  *reinterpret_cast<uint2*>(p) = make_uint2(f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                                            f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16));
}

// 16 rows in row form; `row` points to feature 0 of this lane's row
template <int D> struct RowForm {
  f32x4_t x[D / 16];
  template <typename IO> __device__ __forceinline__ void load(const IO* row, int q4) {
#pragma unroll
    for (int j = 0; j < D / 16; ++j) x[j] = load4(row + 16 * j + 4 * q4);
  }
  template <typename F> __device__ __forceinline__ float fold(float init, F f) const {  // over this lane's features
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) init = f(init, x[j][e]);
    return init;
  }
  __device__ __forceinline__ float dot(const RowForm& o) const {  // of the whole rows
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += x[j][e] * o.x[j][e];
    return rows_sum(s);
  }
  __device__ __forceinline__ void feature(int phi) {  // feature map, in place
    float m = 0.f;
    if (phi == PHI_SOFTMAX) m = rows_max(fold(-INFINITY, [](float a, float b) { return fmaxf(a, b); }));
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[j][e] = feat(x[j][e], m, phi);
    if (phi == PHI_SOFTMAX) {
      const float inv = 1.f / rows_sum(fold(0.f, [](float a, float b) { return a + b; }));
#pragma unroll
      for (int j = 0; j < D / 16; ++j) x[j] *= inv;
    }
  }
};

// 16 rows in column form; row(i) points to feature 0 of row 4*q4 + i
template <int D> struct ColForm {
  static constexpr int NH = D / 64;
  f32x4_t x[4][NH];
  template <typename R> __device__ __forceinline__ void load(R row, int r16) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hf = 0; hf < NH; ++hf) x[i][hf] = load4(row(i) + 64 * hf + 4 * r16);
  }
  __device__ __forceinline__ void feature(int phi) {  // feature map, in place
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float m = 0.f;
      if (phi == PHI_SOFTMAX) {
        m = x[i][0][0];
#pragma unroll
        for (int hf = 0; hf < NH; ++hf)
#pragma unroll
          for (int e = 0; e < 4; ++e) m = fmaxf(m, x[i][hf][e]);
        m = row16_reduce(m, [](float a, float b) { return fmaxf(a, b); });
      }
      float z = 0.f;
#pragma unroll
      for (int hf = 0; hf < NH; ++hf)
#pragma unroll
        for (int e = 0; e < 4; ++e) { x[i][hf][e] = feat(x[i][hf][e], m, phi); z += x[i][hf][e]; }
      if (phi == PHI_SOFTMAX) {
        const float inv = 1.f / sum16(z);
#pragma unroll
        for (int hf = 0; hf < NH; ++hf) x[i][hf] *= inv;
      }
    }
  }
};

// The column form of 16 rows held in row form, through the wave's own plane of LDS (a wave's LDS accesses are done in the
// order they are issued, so no barrier is needed)
template <int D> __device__ __forceinline__ void to_columns(const RowForm<D>& a, ColForm<D>& c, float* plane, int r16, int q4) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) *reinterpret_cast<f32x4_t*>(plane + r16 * (D + 4) + 16 * j + 4 * q4) = a.x[j];
  __builtin_amdgcn_wave_barrier();
  c.load([&](int i) { return plane + (4 * q4 + i) * (D + 4); }, r16);
  __builtin_amdgcn_wave_barrier();
}

// <rows of a, columns b> over the features: element i = row 4*q4 + i of a against column r16
// Four chains of products and a tree of sums: the rounding grows with the length of a chain.  Forward + backward in us, two
// chains | four: 8 x 512 tokens, 16/8 heads, W = 128 343 | 344 at D = 64, 787 | 753 at D = 128; small grids alike.
template <int D> __device__ __forceinline__ f32x4_t row_product(const RowForm<D>& a, const RowForm<D>& b) {
  f32x4_t t[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < D / 16; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = mm4(a.x[j][e], b.x[j][e], t[e]);
  return (t[0] + t[1]) + (t[2] + t[3]);
}
// acc += sum over the 16 rows of row^T (x) p,  p[i] = coefficient of row 4*q4 + i for column r16
template <int D> __device__ __forceinline__ void col_product(const ColForm<D>& a, f32x4_t p, f32x4_t (&acc)[D / 16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[4 * hf + e] = mm4(a.x[i][hf][e], p[i], acc[4 * hf + e]);
}
// The same with the 16 rows as a sum of their own, for chunks of any length: a chain over all of a chunk's keys rounds more than
// states of 64 keys do (one chunk, 4 x 256 tokens, 8/4 heads, W = 32, D = 64: o 1.35e-7 -> 1.50e-7 of the norm off, dv 2.06e-7 ->
// 2.16e-7; with these sums and four chains in row_product 1.28e-7 and 1.92e-7).
template <int D> __device__ __forceinline__ void col_product_apart(const ColForm<D>& a, f32x4_t p, f32x4_t (&acc)[D / 16]) {
#pragma unroll
  for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f32x4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) t = mm4(a.x[i][hf][e], p[i], t);
      acc[4 * hf + e] += t;
    }
}
// Ahead of a col_product whose tile has columns that do not see every row: `see[i]` says whether column r16 sees row
// 4*q4 + i, and p[i] = 0 where it does not.  0 times an infinite or NaN feature is not 0, so such features are taken out of
// the product and added here to the columns that see their row: a column keeps its bits whatever the rows hold that it
// does not see.
template <int D>
__device__ __forceinline__ void hide_unseen(ColForm<D>& a, f32x4_t p, const bool (&see)[4], int r16, int q4, f32x4_t (&acc)[D / 16]) {
  f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = fmaf(a.x[i][hf][e], 0.f, z[e]);
  if (!__any((z[0] + z[1]) + (z[2] + z[3]) != 0.f)) return;  // wave-uniform
#pragma unroll
  for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
#pragma unroll 1
        for (int r4 = 0; r4 < 4; ++r4) {  // row 4*r4 + k
          const float pk = __shfl(p[k], 16 * r4 + r16);
          const bool seen = __shfl((int)see[k], 16 * r4 + r16) != 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x = __shfl(a.x[k][hf][e], 16 * r4 + 4 * q4 + i);
            if (seen && x * 0.f != 0.f) acc[4 * hf + e][i] += pk * x;
          }
        }
        a.x[k][hf][e] = a.x[k][hf][e] * 0.f == 0.f ? a.x[k][hf][e] : 0.f;
      }
    }
}
// acc[d] += sum over the features f of slice j of  M[f][d] b[f],  M row-major [D][D] fp32
template <int D> __device__ __forceinline__ void state_product(const float* M, int j, f32x4_t b, int r16, int q4, f32x4_t (&acc)[D / 16]) {
  ColForm<D> a;
  a.load([&](int e) { return M + (size_t)(16 * j + 4 * q4 + e) * D; }, r16);
  col_product<D>(a, b, acc);
}
// acc[f] += sum over the values d of slice j of  M[f][d] b[d]
template <int D> __device__ __forceinline__ void state_product_t(const float* M, int j, f32x4_t b, int r16, int q4, f32x4_t (&acc)[D / 16]) {
#pragma unroll
  for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x4_t m = load4(M + (size_t)(64 * hf + 4 * r16 + e) * D + 16 * j + 4 * q4);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[4 * hf + e] = mm4(m[s], b[s], acc[4 * hf + e]);
    }
}

// Probability of a pair from its logit as the forward formed it: with the product rounded before the difference, a query
// that sees one key gets exactly 1
__device__ __forceinline__ float prob(float s, float scale, float lse) {
#pragma clang fp contract(off)
  const float a = s * scale;
  return expf(a - lse);
}

template <int D> __device__ __forceinline__ void zero(f32x4_t (&acc)[D / 16]) {
#pragma unroll
  for (int e = 0; e < D / 16; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// A wave's accumulators into its [16 columns][D + 4] plane of LDS
template <int D> __device__ __forceinline__ void put_partial(float* plane, const f32x4_t (&acc)[D / 16], int r16, int q4) {
#pragma unroll
  for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4_t*>(plane + r16 * (D + 4) + 64 * hf + 4 * (4 * q4 + i)) =
          f32x4_t{acc[4 * hf][i], acc[4 * hf + 1][i], acc[4 * hf + 2][i], acc[4 * hf + 3][i]};
}
template <int D> constexpr int plane_floats() { return 16 * (D + 4); }

// Jacobian of phi for a gradient df of phi(x), both in accumulator layout (x is re-read there): df <- J^T df.
// Linear in df, so every wave applies it to its own partial sum.
template <int D, typename IO>
__device__ __forceinline__ void feature_backward(const IO* row, f32x4_t (&df)[D / 16], int q4, int phi) {
  constexpr int NH = D / 64;
  f32x4_t x[NH][4];  // [hf][i]: features 64hf + 4*(4*q4 + i) ..
#pragma unroll
  for (int hf = 0; hf < NH; ++hf)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[hf][i] = load4(row + 64 * hf + 4 * (4 * q4 + i));
  float m = 0.f, inv = 1.f, inner = 0.f;
  if (phi == PHI_SOFTMAX) {
    m = -INFINITY;
#pragma unroll
    for (int hf = 0; hf < NH; ++hf)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = fmaxf(m, x[hf][i][e]);
    m = rows_max(m);
    float z = 0.f;
#pragma unroll
    for (int hf = 0; hf < NH; ++hf)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[hf][i][e] = expf(x[hf][i][e] - m);
          z += x[hf][i][e];
          inner += x[hf][i][e] * df[4 * hf + e][i];
        }
    inv = 1.f / rows_sum(z);
    inner = rows_sum(inner) * inv;
#pragma unroll
    for (int hf = 0; hf < NH; ++hf)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) df[4 * hf + e][i] = x[hf][i][e] * inv * (df[4 * hf + e][i] - inner);
  } else if (phi == PHI_RELU) {
#pragma unroll
    for (int hf = 0; hf < NH; ++hf)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) df[4 * hf + e][i] = x[hf][i][e] > 0.f ? df[4 * hf + e][i] : 0.f;
  }
}

// ------------------------------------------------------------------------------------------------
// Chunk-local products of the linear branch (Eq. 2): U_c[f][d] = sum over the tokens t' in [cC, (c+1)C) below Tp, and
// over the GA heads g*GA .. of tensors with H heads, of phi(a)[f] b[d]; token index t' + off.  grid (n, Hkv, B), block x
// forms product first + x into out[(b*Hkv + g)*nst + first + x].  Steps of 64 tokens: every wave maps 16 of them into LDS
// (the map is most of the step's latency), then each wave forms the products of its D/4 features with all 64.
template <typename AT, typename BT, int D>
__global__ __launch_bounds__(256, 2) void gen_chunk_kernel(const AT* __restrict__ a, const BT* __restrict__ bsrc,
                                                           float* __restrict__ out, int T, int H, int GA, int off, int Tp,
                                                           int C, int nst, int first, int phi) {
  constexpr int NH = D / 64, PS = D + 4;
  __shared__ __align__(16) float pf[64 * PS];
  const int c = first + blockIdx.x, g = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int lane = lane_id(), w = wave_id(), r16 = lane & 15, q4 = lane >> 4;
  const int lo = c * C, hi = min(lo + C, Tp);
  f32x4_t acc[NH][4 * NH];  // [feature tile GWC*ft + w][value 4*hd + e]
#pragma unroll
  for (int ft = 0; ft < NH; ++ft) zero<D>(acc[ft]);
  const int nt = (hi - lo + 63) / 64, nstep = GA * nt;
  auto row = [&](int u, int k) {  // token k of step u (heads outermost)
    return ((size_t)(b * T + min(lo + 64 * (u % nt) + k, hi - 1) + off) * H + g * GA + u / nt) * D;
  };
  // b of token k of step u; tokens past the end are zero, not what the row read in their place holds
  auto load_b = [&](int u, int k, f32x4_t (&x)[NH]) {
    const bool live = lo + 64 * (u % nt) + k < hi;
#pragma unroll
    for (int hd = 0; hd < NH; ++hd) {
      x[hd] = load4(bsrc + row(u, k) + 64 * hd + 4 * r16);
      if (!live) x[hd] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  };
  ColForm<D> fa;
  fa.load([&](int i) { return a + row(0, 16 * w + 4 * q4 + i); }, r16);
  for (int u = 0; u < nstep; ++u) {
    f32x4_t fb[8][NH];  // the first 32 tokens' b rows, requested ahead of the map
#pragma unroll
    for (int tg = 0; tg < 8; ++tg) load_b(u, 4 * tg + q4, fb[tg]);
    fa.feature(phi);
    if (u) __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool live = lo + 64 * (u % nt) + 16 * w + 4 * q4 + i < hi;
#pragma unroll
      for (int hf = 0; hf < NH; ++hf)
        *reinterpret_cast<f32x4_t*>(pf + (16 * w + 4 * q4 + i) * PS + 64 * hf + 4 * r16) = live ? fa.x[i][hf] : f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    if (u + 1 < nstep) fa.load([&](int i) { return a + row(u + 1, 16 * w + 4 * q4 + i); }, r16);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half) {
#pragma unroll
        for (int tg = 0; tg < 8; ++tg) load_b(u, 32 + 4 * tg + q4, fb[tg]);
      }
#pragma unroll
      for (int tg = 0; tg < 8; ++tg)
#pragma unroll
        for (int ft = 0; ft < NH; ++ft) {
          const float av = pf[(32 * half + 4 * tg + q4) * PS + 16 * (GWC * ft + w) + r16];
#pragma unroll
          for (int hd = 0; hd < NH; ++hd)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[ft][4 * hd + e] = mm4(av, fb[tg][hd][e], acc[ft][4 * hd + e]);
        }
    }
  }
  float* U = out + ((size_t)(b * Hkv + g) * nst + c) * D * D;
#pragma unroll
  for (int ft = 0; ft < NH; ++ft)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hd = 0; hd < NH; ++hd)
        store4(U + (size_t)(16 * (GWC * ft + w) + 4 * q4 + i) * D + 64 * hd + 4 * r16,
               f32x4_t{acc[ft][4 * hd][i], acc[ft][4 * hd + 1][i], acc[ft][4 * hd + 2][i], acc[ft][4 * hd + 3][i]});
}

// Products -> states, in place: exclusive prefix (REV = false; state 0 = `init` or zero) or suffix (REV = true) sums over
// the nst chunks of every (b, kv head), in order.  One thread per four elements; the products of eight chunks are
// requested together.  (The product of the last / first chunk is never read.)
template <bool REV>
__global__ __launch_bounds__(64) void gen_scan_kernel(float* __restrict__ U, const float* __restrict__ init, int nst, int vecs) {
  const int v = blockIdx.x * 64 + threadIdx.x;
  if (v >= vecs) return;
  f32x4_t* p = reinterpret_cast<f32x4_t*>(U) + (size_t)blockIdx.y * nst * vecs + v;
  f32x4_t acc = init ? reinterpret_cast<const f32x4_t*>(init)[(size_t)blockIdx.y * vecs + v] : f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto at = [&](int k) -> f32x4_t& { return p[(size_t)(REV ? nst - 1 - k : k) * vecs]; };
  constexpr int GRP = 8;
  for (int k0 = 0; k0 < nst; k0 += GRP) {
    f32x4_t u[GRP];
#pragma unroll
    for (int k = 0; k < GRP; ++k)
      if (k0 + k < nst - 1) u[k] = at(k0 + k);
#pragma unroll
    for (int k = 0; k < GRP; ++k)
      if (k0 + k < nst) {
        at(k0 + k) = acc;
        if (k0 + k < nst - 1) acc += u[k];
      }
  }
}

// ------------------------------------------------------------------------------------------------
// Forward.  grid (ceil((T - q0) / 16), Hq, B), GW waves: 16 query rows of one head.  Only rows q0 .. T-1 have queries; q, o and the
// saved tensors hold just those Tq = T - q0 rows per sequence.  states NULL: there are none (all keys in the first chunk).
template <typename IO, int D, int GW>
__global__ __launch_bounds__(64 * GW, 2) void gen_fwd_kernel(const IO* __restrict__ q, const IO* __restrict__ k,
                                                         const IO* __restrict__ v, const float* __restrict__ gs,
                                                         const float* __restrict__ gr, const float* __restrict__ states,
                                                         IO* __restrict__ o, float* __restrict__ xs_out,
                                                         float* __restrict__ xr_out, float* __restrict__ lse_out,
                                                         float* __restrict__ rs_out, float* __restrict__ rr_out,
                                                         LayerDims dm, int q0) {
  constexpr int PL = plane_floats<D>();
  __shared__ __align__(16) float part[GW * PL];  // partial x_s, then partial x_r
  __shared__ float ml[GW][16][2];
  const int h = blockIdx.y, b = blockIdx.z, g = h / dm.G;
  const int lane = lane_id(), w = wave_id(), r16 = lane & 15, q4 = lane >> 4;
  const int T = dm.T, W = dm.W, C = dm.C, Hq = dm.Hq, Hkv = dm.Hkv, Tq = T - q0;
  const int t0 = q0 + 16 * blockIdx.x, t_hi = min(t0 + 15, T - 1), t = min(t0 + r16, t_hi);
  auto krow = [&](int s) { return k + ((size_t)(b * T + min(s, t_hi)) * Hkv + g) * D; };
  auto vrow = [&](int s) { return v + ((size_t)(b * T + min(s, t_hi)) * Hkv + g) * D; };
  RowForm<D> qv;
  qv.load(q + ((size_t)(b * Tq + t - q0) * Hq + h) * D, q4);
  // ---- softmax branch over keys max(0,t-W+1)..t; key tile n is wave n % 4's
  {
    const int lo = max(0, t0 - W + 1), nt = (t_hi - lo) / 16 + 1;
    f32x4_t acc[D / 16];
    zero<D>(acc);
    float m = -1.0e30f, l = 0.f;
    RowForm<D> kf;
    ColForm<D> vf;
    if (w < nt) {
      kf.load(krow(lo + 16 * w + r16), q4);
      vf.load([&](int i) { return vrow(lo + 16 * w + 4 * q4 + i); }, r16);
    }
    for (int n = w; n < nt; n += GW) {
      const int s0 = lo + 16 * n, next = s0 + 16 * GW;
      f32x4_t s = row_product<D>(kf, qv);
      if (n + GW < nt) kf.load(krow(next + r16), q4);
      float mx = -INFINITY;
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        see[i] = (unsigned)(t - (s0 + 4 * q4 + i)) < (unsigned)W;  // in the window <=> 0 <= query - key < W
        s[i] = see[i] ? s[i] * dm.scale : -INFINITY;
        mx = fmaxf(mx, s[i]);
      }
      const float m_new = fmaxf(m, rows_max(mx)), alpha = expf(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) { s[i] = expf(s[i] - m); l += s[i]; }
#pragma unroll
      for (int e = 0; e < D / 16; ++e) acc[e] *= alpha;
      if (s0 + 15 > t0 || t_hi - s0 >= W) hide_unseen<D>(vf, s, see, r16, q4, acc);
      col_product<D>(vf, s, acc);
      if (n + GW < nt) vf.load([&](int i) { return vrow(next + 4 * q4 + i); }, r16);
    }
    l = rows_sum(l);
    if (q4 == 0) { ml[w][r16][0] = m; ml[w][r16][1] = l; }
    put_partial<D>(part + w * PL, acc, r16, q4);
  }
  // ---- linear branch: phi(q) S_[j] + intra-chunk part over keys jC..t-W, with the chunk j of the tile's first query
  const bool has_lin = t_hi >= W;
  f32x4_t acc[D / 16];
  zero<D>(acc);
  if (has_lin) {
    const int j = max(0, t0 - W) / C;
    const int lo = j * C, nt = (t_hi - W - lo) / 16 + 1;
    RowForm<D> kf;
    ColForm<D> vf;
    auto request = [&](int n) {
      kf.load(krow(lo + 16 * n + r16), q4);
      vf.load([&](int i) { return vrow(lo + 16 * n + 4 * q4 + i); }, r16);
    };
    if (w < nt) request(w);
    qv.feature(dm.phi);
    if (states) {
      const float* S = states + ((size_t)(b * Hkv + g) * dm.nst + j) * D * D;
#pragma unroll
      for (int jj = 0; jj < D / 16; ++jj)
        if (jj % GW == w) state_product<D>(S, jj, qv.x[jj], r16, q4, acc);
    }
    for (int n = w; n < nt; n += GW) {
      const int s0 = lo + 16 * n;
      kf.feature(dm.phi);
      f32x4_t c = row_product<D>(kf, qv);
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { see[i] = s0 + 4 * q4 + i <= t - W; c[i] = see[i] ? c[i] : 0.f; }
      if (s0 + 15 > t0 - W) hide_unseen<D>(vf, c, see, r16, q4, acc);
      if (n + GW < nt) kf.load(krow(s0 + 16 * GW + r16), q4);
      col_product_apart<D>(vf, c, acc);
      if (n + GW < nt) vf.load([&](int i) { return vrow(s0 + 16 * GW + 4 * q4 + i); }, r16);
    }
  }
  __syncthreads();
  // ---- the waves' partial results and the combination: 16 threads per query row, features 64hf + 4c .. (further waves
  // repeat a row and store nothing)
  {
    const int row = (threadIdx.x >> 4) & 15, c = threadIdx.x & 15;
    float M = ml[0][row][0];
#pragma unroll
    for (int r = 1; r < GW; ++r) M = fmaxf(M, ml[r][row][0]);
    float l = 0.f, sw[GW];
#pragma unroll
    for (int r = 0; r < GW; ++r) { sw[r] = expf(ml[r][row][0] - M); l += sw[r] * ml[r][row][1]; }
    f32x4_t xs[D / 64], xr[D / 64];
    float ss = 0.f, sr = 0.f;
    auto partial = [&](int r, int hf) { return *reinterpret_cast<const f32x4_t*>(part + r * PL + row * (D + 4) + 64 * hf + 4 * c); };
#pragma unroll
    for (int hf = 0; hf < D / 64; ++hf) {
      xs[hf] = xr[hf] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < GW; ++r) xs[hf] += sw[r] * partial(r, hf);
      xs[hf] *= 1.f / l;
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += xs[hf][e] * xs[hf][e];
    }
    if (has_lin) {
      __syncthreads();
      put_partial<D>(part + w * PL, acc, r16, q4);
      __syncthreads();
#pragma unroll
      for (int hf = 0; hf < D / 64; ++hf) {
#pragma unroll
        for (int r = 0; r < GW; ++r) xr[hf] += partial(r, hf);
#pragma unroll
        for (int e = 0; e < 4; ++e) sr += xr[hf][e] * xr[hf][e];
      }
    }
    const float r_s = rsqrtf(sum16(ss) / D + dm.eps), r_r = rsqrtf(sum16(sr) / D + dm.eps);
    const int tq = 16 * blockIdx.x + row;
    if (tq < Tq && threadIdx.x < 256) {
      const size_t off = ((size_t)(b * Tq + tq) * Hq + h) * D;
#pragma unroll
      for (int hf = 0; hf < D / 64; ++hf) {
        const int d = 64 * hf + 4 * c;
        f32x4_t y1 = xs[hf] * r_s, y2 = xr[hf] * r_r;
        if (gs) y1 *= load4(gs + h * D + d);
        if (gr) y2 *= load4(gr + h * D + d);
        store4(o + off + d, y1 + y2);
        if (xs_out) { store4(xs_out + off + d, xs[hf]); store4(xr_out + off + d, xr[hf]); }
      }
      if (xs_out && c == 0) {
        const size_t so = (size_t)(b * Hq + h) * Tq + tq;
        lse_out[so] = M + logf(l);
        rs_out[so] = r_s;
        rr_out[so] = r_r;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Backward, dq.  grid (ceil(T / 16), Hq, B): 16 query rows of one head.
//   RMS norms (Sec. 3.2): for y = g*x*r, r = (mean x^2+eps)^-1/2:  dx = r*(g*dy) - x*r^3*mean(g*dy*x),
//                   dgamma += dy*x*r,  delta = <dx_s, x_s>;  dx_s, dx_r, delta are stored for the dk/dv kernel, the sums
//                   over the 16 rows of the gain gradients go to dgpart[2][RB][Hq][D] (NULL: not wanted)
//   softmax branch: p = exp(scale q.k - lse), dp = <dx_s, v_s>, da = p(dp - delta), dq += scale*da*k_s.
//                   Windows of up to 64 keys take delta = sum p dp over the very p and dp that form da: their rows are often
//                   close to one-hot, where p (dp - delta) cancels (to exactly 0 for a single key) and the rounding of
//                   <dx_s, x_s> would be what is left (W = 1: error of dq 2.4e-7 -> 2e-6 .. 8e-5, growing with the logits).
//                   Such a range is at most five tiles, so each wave keeps the p and dp of its one or two.
//   linear branch : dphi(q) = S_[j] dx_r + sum_{intra} <dx_r, v_s> phi(k_s);  dq += phi(q)*(dphi - <dphi,phi(q)>)
//                   (softmax map; ReLU passes dphi where q > 0, identity passes it unchanged)
template <typename IO, int D, int GW>
__global__ __launch_bounds__(64 * GW, 2) void gen_bwd_dq_kernel(const IO* __restrict__ q, const IO* __restrict__ k,
                                                            const IO* __restrict__ v, const IO* __restrict__ dO,
                                                            const float* __restrict__ gs, const float* __restrict__ gr,
                                                            SavedPtrs sv, const float* __restrict__ states,
                                                            IO* __restrict__ dq, float* __restrict__ dxs_out,
                                                            float* __restrict__ dxr_out, float* __restrict__ delta_out,
                                                            float* __restrict__ dgpart, LayerDims dm) {
  constexpr int PL = plane_floats<D>();
  constexpr int SHORT_W = 64;
  __shared__ __align__(16) float part[GW * PL];
  __shared__ float dsum[GW][16];
  const int h = blockIdx.y, b = blockIdx.z, g = h / dm.G;
  const int lane = lane_id(), w = wave_id(), r16 = lane & 15, q4 = lane >> 4;
  const int T = dm.T, W = dm.W, C = dm.C, Hq = dm.Hq, Hkv = dm.Hkv;
  const int t0 = 16 * blockIdx.x, t_hi = min(t0 + 15, T - 1), t = min(t0 + r16, t_hi);
  const bool live = t0 + r16 <= t_hi;
  auto krow = [&](int s) { return k + ((size_t)(b * T + min(s, t_hi)) * Hkv + g) * D; };
  auto vrow = [&](int s) { return v + ((size_t)(b * T + min(s, t_hi)) * Hkv + g) * D; };
  const size_t qoff = ((size_t)(b * T + t) * Hq + h) * D, so = (size_t)(b * Hq + h) * T + t;
  // ---- RMS norms; every wave forms the gradients of the 16 rows for itself
  RowForm<D> dxs, dxr;
  float delta;
  {
    RowForm<D> dy, x, xr;   // requested together: the stores below could alias any of them
    dy.load(dO + qoff, q4);
    xr.load((const float*)sv.xr + qoff, q4);
    x.load((const float*)sv.xs + qoff, q4);
    const float r_s = sv.rs[so], r_r = sv.rr[so];
    float* dg = dgpart && w == 0 ? dgpart + ((size_t)(b * gridDim.x + blockIdx.x) * Hq + h) * D : nullptr;
    const size_t dg_which = (size_t)gridDim.x * gridDim.z * Hq * D;
    auto branch = [&](const RowForm<D>& x, const float* gain, float r, RowForm<D>& dx, float* dgp) {
      float mean = 0.f;
#pragma unroll
      for (int j = 0; j < D / 16; ++j) {
        const f32x4_t gj = gain ? load4(gain + h * D + 16 * j + 4 * q4) : f32x4_t{1.f, 1.f, 1.f, 1.f};
        dx.x[j] = gj * dy.x[j];
#pragma unroll
        for (int e = 0; e < 4; ++e) mean += dx.x[j][e] * x.x[j][e];
        if (dgp) {
          f32x4_t s = dy.x[j] * x.x[j] * (live ? r : 0.f);
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] = sum16(s[e]);
          if (r16 == 0) store4(dgp + 16 * j + 4 * q4, s);
        }
      }
      mean = rows_sum(mean) / D;
#pragma unroll
      for (int j = 0; j < D / 16; ++j) dx.x[j] = r * dx.x[j] - x.x[j] * (r * r * r * mean);
    };
    branch(xr, gr, r_r, dxr, dg ? dg + dg_which : nullptr);
    branch(x, gs, r_s, dxs, dg);
    delta = dxs.dot(x);
    if (w == GW - 1 && live) {
#pragma unroll
      for (int j = 0; j < D / 16; ++j) {
        store4(dxs_out + qoff + 16 * j + 4 * q4, dxs.x[j]);
        store4(dxr_out + qoff + 16 * j + 4 * q4, dxr.x[j]);
      }
      if (q4 == 0 && W > SHORT_W) delta_out[so] = delta;
    }
  }
  f32x4_t acc[D / 16];
  zero<D>(acc);
  // ---- linear branch
  if (t_hi >= W) {
    const int j = max(0, t0 - W) / C;
    const int lo = j * C, nt = (t_hi - W - lo) / 16 + 1;
    RowForm<D> vf;
    ColForm<D> kf;
    auto request_v = [&](int n) { vf.load(vrow(lo + 16 * n + r16), q4); };
    auto request_k = [&](int n) { kf.load([&](int i) { return krow(lo + 16 * n + 4 * q4 + i); }, r16); };
    if (w < nt) { request_v(w); request_k(w); }
    if (states) {
      const float* S = states + ((size_t)(b * Hkv + g) * dm.nst + j) * D * D;
#pragma unroll
      for (int jj = 0; jj < D / 16; ++jj)
        if (jj % GW == w) state_product_t<D>(S, jj, dxr.x[jj], r16, q4, acc);
    }
    for (int n = w; n < nt; n += GW) {
      const int s0 = lo + 16 * n;
      f32x4_t c = row_product<D>(vf, dxr);
      if (n + GW < nt) request_v(n + GW);
      kf.feature(dm.phi);
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { see[i] = s0 + 4 * q4 + i <= t - W; c[i] = see[i] ? c[i] : 0.f; }
      if (s0 + 15 > t0 - W) hide_unseen<D>(kf, c, see, r16, q4, acc);
      col_product<D>(kf, c, acc);
      if (n + GW < nt) request_k(n + GW);
    }
    feature_backward<D>(q + qoff, acc, q4, dm.phi);
  }
  // ---- softmax branch
  {
    RowForm<D> qv;
    qv.load(q + qoff, q4);
    const float lse = sv.lse[so];
    const int lo = max(0, t0 - W + 1), nt = (t_hi - lo) / 16 + 1;
    auto sees = [&](int s) { return (unsigned)(t - s) < (unsigned)W; };
    float* plane = part + w * PL;
    RowForm<D> kf, vf;
    auto request = [&](int n) {
      kf.load(krow(lo + 16 * n + r16), q4);
      vf.load(vrow(lo + 16 * n + r16), q4);
    };
    // p and dp of the 16 keys from s0 on (in kf, vf), 0 where the query does not see the key
    auto scores = [&](int s0, f32x4_t& p, f32x4_t& dp) {
      p = row_product<D>(kf, qv);
      dp = row_product<D>(vf, dxs);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool see = sees(s0 + 4 * q4 + i);
        p[i] = see ? prob(p[i], dm.scale, lse) : 0.f;
        dp[i] = see ? dp[i] : 0.f;
      }
    };
    auto add = [&](int s0, ColForm<D>& kc, f32x4_t p, f32x4_t dp) {
      f32x4_t da;
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        see[i] = sees(s0 + 4 * q4 + i);
        da[i] = see[i] ? p[i] * (dp[i] - delta) * dm.scale : 0.f;
      }
      if (s0 + 15 > t0 || t_hi - s0 >= W) hide_unseen<D>(kc, da, see, r16, q4, acc);
      col_product<D>(kc, da, acc);
    };
    constexpr bool AHEAD = D == 64;  // the next tile's rows requested behind this one's products (D = 128: no registers left)
    if (AHEAD && w < nt) request(w);
    if (W <= SHORT_W) {
      constexpr int NU = (5 + GW - 1) / GW;
      f32x4_t p[NU], dp[NU];
      float dl = 0.f;
#pragma unroll
      for (int u = 0; u < NU; ++u)
        if (w + GW * u < nt) {
          if (!AHEAD || u) request(w + GW * u);
          scores(lo + 16 * (w + GW * u), p[u], dp[u]);
#pragma unroll
          for (int i = 0; i < 4; ++i) dl += p[u][i] * dp[u][i];
        }
      dl = rows_sum(dl);
      if (q4 == 0) dsum[w][r16] = dl;
      __syncthreads();
      delta = (dsum[0][r16] + dsum[1][r16]) + (dsum[2][r16] + dsum[3][r16]);
      if (GW == 8) delta += dsum[4][r16];  // (the fifth tile; the other waves have none)
      if (w == GW - 1 && live && q4 == 0) delta_out[so] = delta;
#pragma unroll
      for (int u = NU - 1; u >= 0; --u)
        if (w + GW * u < nt) {
          if (u < NU - 1) kf.load(krow(lo + 16 * (w + GW * u) + r16), q4);  // (the last one's rows are still there)
          ColForm<D> kc;
          to_columns<D>(kf, kc, plane, r16, q4);
          add(lo + 16 * (w + GW * u), kc, p[u], dp[u]);
        }
    } else {
      for (int n = w; n < nt; n += GW) {
        f32x4_t p, dp;
        ColForm<D> kc;
        if (!AHEAD) request(n);
        scores(lo + 16 * n, p, dp);
        to_columns<D>(kf, kc, plane, r16, q4);
        if (AHEAD && n + GW < nt) request(n + GW);
        add(lo + 16 * n, kc, p, dp);
      }
    }
  }
  put_partial<D>(part + w * PL, acc, r16, q4);
  __syncthreads();
  const int row = threadIdx.x >> 4, c = threadIdx.x & 15;
  if (row < 16 && t0 + row < T) {
#pragma unroll
    for (int hf = 0; hf < D / 64; ++hf) {
      f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < GW; ++r) s += *reinterpret_cast<const f32x4_t*>(part + r * PL + row * (D + 4) + 64 * hf + 4 * c);
      store4(dq + ((size_t)(b * T + t0 + row) * Hq + h) * D + 64 * hf + 4 * c, s);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Backward, dk and dv.  grid (ceil(T / 16), Hkv, B): 16 key rows of one KV head; the G query heads of the group are
// visited in turn, so no atomics are needed.  `rstates` are the reverse-time chunk states R_[j] = sum over query chunks
// after j of phi(q)^T dx_r (summed over the group's heads); j is the chunk of the tile's last key.
template <typename IO, int D, int GW>
__global__ __launch_bounds__(64 * GW, 2) void gen_bwd_dkv_kernel(const IO* __restrict__ q, const IO* __restrict__ k,
                                                             const IO* __restrict__ v, const float* __restrict__ dxs,
                                                             const float* __restrict__ dxr, const float* __restrict__ delta,
                                                             const float* __restrict__ lse, const float* __restrict__ rstates,
                                                             IO* __restrict__ dk, IO* __restrict__ dv, LayerDims dm) {
  constexpr int PL = plane_floats<D>();
  __shared__ __align__(16) float part[GW * PL];
  const int g = blockIdx.y, b = blockIdx.z;
  const int lane = lane_id(), w = wave_id(), r16 = lane & 15, q4 = lane >> 4;
  const int T = dm.T, W = dm.W, C = dm.C, Hq = dm.Hq, Hkv = dm.Hkv, G = dm.G;
  const int Tp = max(T - W, 0);
  const int s0 = 16 * blockIdx.x, s_hi = min(s0 + 15, T - 1), s = min(s0 + r16, s_hi);
  const size_t koff = ((size_t)(b * T + s) * Hkv + g) * D;
  RowForm<D> kv, vv;
  vv.load(v + koff, q4);
  kv.load(k + koff, q4);
  f32x4_t dka[D / 16], dva[D / 16];
  zero<D>(dka);
  zero<D>(dva);
  constexpr bool AHEAD = D == 64;  // (D = 128: no registers for the next tile's rows)
  float* plane = part + w * PL;
  RowForm<D> qf, dr;  // the rows of a query tile: q and d x_r or d x_s; their column forms go through the wave's plane
  // ---- linear branch: queries t = t' + W, t' >= s
  if (s0 < Tp) {
    const int j = min(s_hi, Tp - 1) / C;
    const int hi = min((j + 1) * C, Tp) - 1, nt = (hi - s0) / 16 + 1;
    auto off = [&](int u) {  // of this lane's row of step u (heads outermost)
      return ((size_t)(b * T + min(s0 + 16 * (u % nt) + r16, hi) + W) * Hq + g * G + u / nt) * D;
    };
    auto request_q = [&](int u) { qf.load(q + off(u), q4); };
    auto request_d = [&](int u) { dr.load(dxr + off(u), q4); };
    if (AHEAD && w < G * nt) { request_d(w); request_q(w); }
    kv.feature(dm.phi);
    if (rstates) {
      const float* R = rstates + ((size_t)(b * Hkv + g) * dm.nst + j) * D * D;
#pragma unroll
      for (int jj = 0; jj < D / 16; ++jj)
        if (jj % GW == w) {
          state_product<D>(R, jj, kv.x[jj], r16, q4, dva);
          state_product_t<D>(R, jj, vv.x[jj], r16, q4, dka);
        }
    }
    for (int u = w; u < G * nt; u += GW) {
      const int tp0 = s0 + 16 * (u % nt);
      const bool all = tp0 >= s_hi && tp0 + 15 <= hi;  // every query of the tile sees every key
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { const int tp = tp0 + 4 * q4 + i; see[i] = tp >= s && tp <= hi; }
      auto add = [&](ColForm<D>& a, f32x4_t c, f32x4_t (&acc)[D / 16]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = see[i] ? c[i] : 0.f;
        if (!all) hide_unseen<D>(a, c, see, r16, q4, acc);
        col_product_apart<D>(a, c, acc);
      };
      ColForm<D> col;
      if (!AHEAD) { request_d(u); request_q(u); }
      const f32x4_t e = row_product<D>(dr, vv);
      to_columns<D>(dr, col, plane, r16, q4);
      if (AHEAD && u + GW < G * nt) request_d(u + GW);
      qf.feature(dm.phi);
      add(col, row_product<D>(qf, kv), dva);
      to_columns<D>(qf, col, plane, r16, q4);
      if (AHEAD && u + GW < G * nt) request_q(u + GW);
      add(col, e, dka);
    }
    kv.load(k + koff, q4);  // (as it is again, for the softmax branch)
    feature_backward<D>(k + koff, dka, q4, dm.phi);
    if (s >= Tp) {  // (a key without residual queries in a tile that has some: its column is zero up to here)
#pragma unroll
      for (int e = 0; e < D / 16; ++e) dka[e] = dva[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  }
  // ---- softmax branch: queries s .. s + W - 1
  {
    const int hi = s_hi < T - W ? s_hi + W - 1 : T - 1, nt = (hi - s0) / 16 + 1;  // (any W up to INT_MAX: no sum beyond T)
    float lse_t[4], delta_t[4];
    auto off = [&](int u) { return ((size_t)(b * T + min(s0 + 16 * (u % nt) + r16, hi)) * Hq + g * G + u / nt) * D; };
    auto request_q = [&](int u) { qf.load(q + off(u), q4); };
    auto request_d = [&](int u) {
      dr.load(dxs + off(u), q4);
      const int q0 = s0 + 16 * (u % nt);
      const size_t sbase = (size_t)(b * Hq + g * G + u / nt) * T;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = min(q0 + 4 * q4 + i, hi);
        lse_t[i] = lse[sbase + t];
        delta_t[i] = delta[sbase + t];
      }
    };
    if (AHEAD && w < G * nt) { request_q(w); request_d(w); }
    for (int u = w; u < G * nt; u += GW) {
      const int q0 = s0 + 16 * (u % nt);
      if (!AHEAD) { request_q(u); request_d(u); }
      f32x4_t p = row_product<D>(qf, kv), da = row_product<D>(dr, vv);
      bool see[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = q0 + 4 * q4 + i;
        see[i] = (unsigned)(t - s) < (unsigned)W && t <= hi;
        p[i] = see[i] ? prob(p[i], dm.scale, lse_t[i]) : 0.f;
        da[i] = see[i] ? p[i] * (da[i] - delta_t[i]) * dm.scale : 0.f;
      }
      const bool all = q0 >= s_hi && q0 + 15 <= hi && q0 + 15 - s0 < W;  // every query of the tile sees every key
      auto add = [&](ColForm<D>& a, f32x4_t x, f32x4_t (&acc)[D / 16]) {
        if (!all) hide_unseen<D>(a, x, see, r16, q4, acc);
        col_product<D>(a, x, acc);
      };
      ColForm<D> col;
      to_columns<D>(dr, col, plane, r16, q4);
      if (AHEAD && u + GW < G * nt) request_d(u + GW);
      add(col, p, dva);
      to_columns<D>(qf, col, plane, r16, q4);
      if (AHEAD && u + GW < G * nt) request_q(u + GW);
      add(col, da, dka);
    }
  }
  const int row = threadIdx.x >> 4, c = threadIdx.x & 15;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if (which) __syncthreads();
    put_partial<D>(part + w * PL, which ? dva : dka, r16, q4);
    __syncthreads();
    IO* dst = which ? dv : dk;
    if (row < 16 && s0 + row < T) {
#pragma unroll
      for (int hf = 0; hf < D / 64; ++hf) {
        f32x4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < GW; ++r) x += *reinterpret_cast<const f32x4_t*>(part + r * PL + row * (D + 4) + 64 * hf + 4 * c);
        store4(dst + ((size_t)(b * T + s0 + row) * Hkv + g) * D + 64 * hf + 4 * c, x);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// host launchers
// The states that the consumers read: none of their own where all keys lie in the first chunk, whose state is `init`
template <typename AT, typename BT, int D, bool REV>
const float* build_states(const LayerDims& dm, const void* a, const void* bsrc, float* states, int H, int GA, int off,
                          const float* init, hipStream_t st) {
  if (dm.nst <= 1) return init;
  {
    ProfScope ps(REV ? "gen_chunk_kernel(rev)" : "gen_chunk_kernel", st);
    gen_chunk_kernel<AT, BT, D><<<dim3(dm.nst - 1, dm.Hkv, dm.B), 256, 0, st>>>(
        (const AT*)a, (const BT*)bsrc, states, dm.T, H, GA, off, dm.T - dm.W, dm.C, dm.nst, REV ? 1 : 0, dm.phi);
  }
  ProfScope ps(REV ? "gen_scan_kernel(rev)" : "gen_scan_kernel", st);
  gen_scan_kernel<REV><<<dim3(D * D / 256, dm.B * dm.Hkv), 64, 0, st>>>(states, init, dm.nst, D * D / 4);
  return states;
}

// Eight waves share the other side's tiles where every work-group has a CU to itself.  Forward + backward in us, four | eight
// waves: T = 256, 2 heads, W = 32, one chunk 49.0 | 42.0 at D = 64, 85.6 | 72.6 at D = 128; T = 512, 2 x 2 x 2 heads, W = 128,
// chunks of 64 69.3 | 69.3, 134.0 | 125.2 (256 work-groups; with few tiles up to 2 us of it are lost: T = 128, W = 16 46.8 |
// 49.4).
bool wide_groups(const LayerDims& dm, int rows, int heads) { return (long long)((rows + 15) / 16) * heads * dm.B <= 256; }

template <typename IO, int D>
void launch_fwd(const LayerDims& dm, const void* q, const void* k, const void* v, const float* gs, const float* gr, void* o,
                const SavedPtrs& sv, float* states, hipStream_t st, int q0, const float* state0) {
  const float* s = build_states<IO, IO, D, false>(dm, k, v, states, dm.Hkv, 1, 0, state0, st);
  ProfScope ps("gen_fwd_kernel", st);
  const dim3 grid((dm.T - q0 + 15) / 16, dm.Hq, dm.B);
#define RATTN_GEN_FWD(GW_)                                                                                              \
  gen_fwd_kernel<IO, D, GW_><<<grid, 64 * GW_, 0, st>>>((const IO*)q, (const IO*)k, (const IO*)v, gs, gr, s, (IO*)o,    \
                                                        (float*)sv.xs, (float*)sv.xr, sv.lse, sv.rs, sv.rr, dm, q0)
  if (wide_groups(dm, dm.T - q0, dm.Hq)) RATTN_GEN_FWD(8); else RATTN_GEN_FWD(4);
#undef RATTN_GEN_FWD
}

template <typename IO, int D>
void launch_bwd(const LayerDims& dm, const void* q, const void* k, const void* v, const float* gs, const float* gr,
                const SavedPtrs& sv, const void* dO, void* dq, void* dk, void* dv, float* dgs, float* dgr,
                const GenericBwdWs& ws, hipStream_t st) {
  const int tiles = (dm.T + 15) / 16;
  // not kept by the forward: built again, where the reverse states go once dq has read them
  const float* states = sv.states && dm.nst > 1 ? (const float*)sv.states
                                                : build_states<IO, IO, D, false>(dm, k, v, ws.rstates, dm.Hkv, 1, 0, nullptr, st);
  {
    ProfScope ps("gen_bwd_dq_kernel", st);
#define RATTN_GEN_DQ(GW_)                                                                                                 \
  gen_bwd_dq_kernel<IO, D, GW_><<<dim3(tiles, dm.Hq, dm.B), 64 * GW_, 0, st>>>(                                           \
      (const IO*)q, (const IO*)k, (const IO*)v, (const IO*)dO, gs, gr, sv, states, (IO*)dq, ws.dxs, ws.dxr, ws.delta,     \
      dgs || dgr ? ws.dgpart : nullptr, dm)
    if (wide_groups(dm, dm.T, dm.Hq)) RATTN_GEN_DQ(8); else RATTN_GEN_DQ(4);
#undef RATTN_GEN_DQ
  }
  if (dgs || dgr) dgamma_reduce(DgammaSum{ws.dgpart, dgs, dgr, tiles * dm.B, dm.Hq * D}, st);
  const float* rstates = build_states<IO, float, D, true>(dm, q, ws.dxr, ws.rstates, dm.Hq, dm.G, dm.W, nullptr, st);
  ProfScope ps("gen_bwd_dkv_kernel", st);
#define RATTN_GEN_DKV(GW_)                                                                                               \
  gen_bwd_dkv_kernel<IO, D, GW_><<<dim3(tiles, dm.Hkv, dm.B), 64 * GW_, 0, st>>>(                                        \
      (const IO*)q, (const IO*)k, (const IO*)v, ws.dxs, ws.dxr, ws.delta, sv.lse, rstates, (IO*)dk, (IO*)dv, dm)
  if (wide_groups(dm, dm.T, dm.Hkv)) RATTN_GEN_DKV(8); else RATTN_GEN_DKV(4);
#undef RATTN_GEN_DKV
}

}  // namespace

void generic_fwd(const LayerDims& dm, int dtype, const void* q, const void* k, const void* v, const float* gs,
                 const float* gr, void* o, const SavedPtrs& sv, float* states, hipStream_t st, int q0, const float* state0) {
  if (dtype == 0) {
    if (dm.D == 64) launch_fwd<float, 64>(dm, q, k, v, gs, gr, o, sv, states, st, q0, state0);
    else launch_fwd<float, 128>(dm, q, k, v, gs, gr, o, sv, states, st, q0, state0);
  } else {
    if (dm.D == 64) launch_fwd<bf16_t, 64>(dm, q, k, v, gs, gr, o, sv, states, st, q0, state0);
    else launch_fwd<bf16_t, 128>(dm, q, k, v, gs, gr, o, sv, states, st, q0, state0);
  }
}

void generic_chunk_products(const LayerDims& dm, int T, const void* k, const void* v, float* out, int Tp, int nseg,
                            int seg_len, hipStream_t st) {
  ProfScope ps("gen_chunk_kernel", st);
  const dim3 grid(nseg, dm.Hkv, dm.B);
  if (dm.D == 64)
    gen_chunk_kernel<float, float, 64><<<grid, 256, 0, st>>>((const float*)k, (const float*)v, out, T, dm.Hkv, 1, 0, Tp, seg_len, nseg, 0, dm.phi);
  else
    gen_chunk_kernel<float, float, 128><<<grid, 256, 0, st>>>((const float*)k, (const float*)v, out, T, dm.Hkv, 1, 0, Tp, seg_len, nseg, 0, dm.phi);
}

void generic_bwd(const LayerDims& dm, int dtype, const void* q, const void* k, const void* v, const float* gs,
                 const float* gr, const SavedPtrs& sv, const void* dO, void* dq, void* dk, void* dv, float* dgs,
                 float* dgr, const GenericBwdWs& ws, hipStream_t st) {
  if (dtype == 0) {
    if (dm.D == 64) launch_bwd<float, 64>(dm, q, k, v, gs, gr, sv, dO, dq, dk, dv, dgs, dgr, ws, st);
    else launch_bwd<float, 128>(dm, q, k, v, gs, gr, sv, dO, dq, dk, dv, dgs, dgr, ws, st);
  } else {
    if (dm.D == 64) launch_bwd<bf16_t, 64>(dm, q, k, v, gs, gr, sv, dO, dq, dk, dv, dgs, dgr, ws, st);
    else launch_bwd<bf16_t, 128>(dm, q, k, v, gs, gr, sv, dO, dq, dk, dv, dgs, dgr, ws, st);
  }
}

}  // namespace rattn
