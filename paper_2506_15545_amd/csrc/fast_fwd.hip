// MFMA forward of the RAttention layer for bf16, D = 128 or 64, any T >= 128 (tiles are laid out for T rounded up to whole
// 128-row tiles, see SeqRows), any window W >= 8.
// Tiles, chunk states and loop ranges are laid out for the window rounded up to a multiple of 64 (`W` in the
// kernel arguments); `gap` = that minus the true window (0..63) enters only the element masks and, in the linear
// branch, the reach of the intra-chunk part (queries see `gap` more keys than the aligned layout gives them).
//
// One work-group (4 waves) owns 128 consecutive queries of one head; wave w owns 32 of them.
// Everything is computed TRANSPOSED so that a lane always owns one query (column) of the MFMA
// results and all row statistics are lane-local (plus one exchange with lane^32):
//   softmax branch (Sec. 2.1):  S^T = K Q^T  ->  online softmax  ->  O^T += V^T P^T
//   linear branch (Eqs. 2-4) :  X^T = St Qf^T  +  V^T (M^T .* (Kf Qf^T)),  St = S_[j]^T (bf16, from the
//                               state pre-pass), Qf/Kf = phi(Q)/phi(K) computed on the operand registers
//   combination (Sec. 3.2)   :  o = gs * x_s * r_s + gr * x_r * r_r, transposed through LDS for
//                               coalesced stores
// K/V tiles (64 keys) stream through a double buffer in LDS with direct-to-LDS loads; the softmax branch
// walks its key tiles from the diagonal downwards (every row's running maximum is finite from the start),
// then the linear branch runs on the two lowest tiles, which are still resident; the normalised softmax-branch
// result stays in fp32 registers meanwhile, so the output is rounded to bf16 once.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include <type_traits>

namespace rattn {

namespace {

struct FastFwdArgs {
  SeqRows q, k, v;         // q: the rows of the computed query tiles only (front part empty)
  const float *gs, *gr;
  uint16_t *o, *xs_out, *xr_out;
  float *lse_out, *rs_out, *rr_out;
  const uint16_t* states;  // [B,Hkv,nstf,D (value d),D (feature f)] bf16: S^T at key position base+128*i
  int B, T, Hq, Hkv, G, W, gap, nstf, ntile;  // T: padded length; W: window rounded up to 64; true window = W - gap
  int qt0;   // first query tile that is computed; q, o and the saved tensors hold rows 128 qt0 .. only
  int kmin;  // keys in front of this row do not exist (chunked prefill: rows in front of a short ring)
  float scale_log2, eps;
};

// The sweep over the 32-key sub-tiles j (upper keys first) for this wave's 32 queries (lane = query) is software-pipelined.
// Step j is one instruction stream of
//   1. S^T(j+1) = K Q^T (matrix cores)   ||  row maximum of S^T(j);  row sum and bf16 packing of P^T(j-1)
//   2. O^T += V^T P^T(j-1)               ||  P^T(j) = 2^(c S^T(j) - m)
// `m` is the reference maximum in scaled log2 units.  It is only raised (and O, l rescaled) when some row's maximum exceeds
// it by more than RESCALE_TH, so P stays below 2^RESCALE_TH; the exponentials do not wait for that decision, they are
// formed again in the rare step that takes it.  Vector work is dealt out evenly between the matrix instructions and operand
// reads run FWD_AHEAD instructions in front of their use, across the border of 1 and 2; scheduling fences keep the order of
// the source.  Left to the scheduler, every V operand was read right in front of its use and the exponentials and sums stood
// apart from the matrix instructions.  The kernel on one box, by events, the scheduler's order -> this one with the tile loads
// dealt out: 32768 tokens, W = 4096 1.65 -> 1.54 ms, 3B-shaped layer 0.210 -> 0.201, a chunk of 4 x 2048 tokens behind rings
// of 512 0.114 -> 0.107.  By the counters (32768 tokens) the matrix pipe is busy for 61 % of the kernel (52 before) at 6.7
// vector and matrix instructions, 1.5 LDS reads and 2.5 scalar instructions (3.6) per matrix instruction: the two waves of a
// SIMD still leave two fifths of the pipe to their waits, and the clock falls as it fills (1.66 -> 1.57 GHz over the kernel).
constexpr float RESCALE_TH = 8.f;
constexpr float M_INIT = -1.0e30f;  // finite "minus infinity" for the running maximum
constexpr int FWD_AHEAD = 4;

struct SweepGeom {
  int kt_lo, ntiles, qa, W, kmin;
  // first key of sub-tile j (tile j/2 counted from the diagonal, upper half first)
  __device__ __forceinline__ int ka(int j) const { return kt_lo + 64 * (ntiles - 1 - (j >> 1)) + 32 * (1 - (j & 1)); }
  // every (query, key) pair of the wave's 32 queries and the sub-tile's 32 keys is inside the window
  __device__ __forceinline__ bool full(int j) const {
    const int k = ka(j);
    return k + 31 <= qa && k >= max(qa + 31 - W + 1, kmin);
  }
};

template <int D> struct SweepState {
  f32x16_t oacc[D / 32];   // O^T against the reference maximum m
  f32x16_t s;              // S^T of the next sub-tile to be worked on
  float p[16];             // P^T of the last one
  float m, l;
};

// operand i of S^T = K Q^T for sub-tile half KS of the K tile in buffer KB; of O^T += V^T P^T for the V tile in buffer VB
template <int D, int KB, int KS>
__device__ __forceinline__ bf16x8_t k_operand(const unsigned char* smem, const LaneOff<D>& lo, int i) {
  return lds_row<D>(smem + KB * TileGeom<D>::KT, lo, 32 * KS, i);
}
template <int D, int VB, int KS>
__device__ __forceinline__ bf16x8_t v_operand(const unsigned char* smem, const LaneOff<D>& lo, int i) {
  return lds_trp<D>(smem + (2 + VB) * TileGeom<D>::KT, lo, 32 * KS + 16 * (i / (D / 32)), i % (D / 32));
}
template <int D, int KB, int KS>
__device__ __forceinline__ void qk_chain(const unsigned char* smem, const LaneOff<D>& lo, const bf16x8_t (&qop)[D / 16],
                                         f32x16_t& s) {
  s = f32x16_t{0};
#pragma unroll
  for (int i = 0; i < D / 16; ++i) s = mfma32(k_operand<D, KB, KS>(smem, lo, i), qop[i], s);
}
__device__ __forceinline__ void sum_and_pack(const float (&p)[16], float& l, bf16x8_t (&pop)[2]) {
  float ps = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) ps += p[i];
  l += ps;
  pop[0] = pack_bf16x8(&p[0]);
  pop[1] = pack_bf16x8(&p[8]);
}
template <int D, int VB, int KS>
__device__ __forceinline__ void pv_chain(const unsigned char* smem, const LaneOff<D>& lo, const bf16x8_t (&pop)[2],
                                         f32x16_t (&oacc)[D / 32]) {
#pragma unroll
  for (int i = 0; i < D / 16; ++i) oacc[i % (D / 32)] = mfma32(v_operand<D, VB, KS>(smem, lo, i), pop[i / (D / 32)], oacc[i % (D / 32)]);
}

// Step j with R = j % 4 (fixes which LDS buffers / halves sub-tiles j+1 and j-1 live in, so that every LDS address is a
// per-lane register plus an immediate).  Every wave runs every step of the work-group's key range: sub-tiles outside a
// wave's own window are fully masked (their probabilities are exactly 0), which costs a few percent of the matrix work and
// keeps one straight code path.  PREV: there is a sub-tile j-1.  request(i), i = 0 .. 2 D/16 - 1: tile loads to be dealt
// out between the matrix instructions.
template <int D, int R, bool PREV, typename F>
__device__ __forceinline__ void sweep_step(const unsigned char* smem, const LaneOff<D>& lo, const SweepGeom& gm, int j,
                                           int myq, float scale_log2, const bf16x8_t (&qop)[D / 16], SweepState<D>& st,
                                           int lane, F&& request) {
  constexpr int KS = R & 1;                           // sub-tile half of both j+1 and j-1
  constexpr int KB = (R == 1 || R == 2) ? 1 : 0;      // K buffer of sub-tile j+1
  constexpr int VB = (R == 0 || R == 3) ? 1 : 0;      // V buffer of sub-tile j-1
  constexpr int N = D / 16, PER = 16 / N;             // matrix instructions of each half of the step
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  if (!gm.full(j)) {  // wave-uniform: window edge, diagonal, or a sub-tile this wave does not see at all
    // in the window <=> 0 <= query - key < W: one unsigned compare per element against a per-lane base
    unsigned dist0 = (unsigned)(myq - gm.ka(j) - 4 * (lane >> 5)), width = (unsigned)min(gm.W, myq - gm.kmin + 1);
    asm volatile("" : "+v"(dist0));   // (nothing of this rare form is kept in registers across the steps)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      st.s[i] = (dist0 - (unsigned)(8 * (i >> 2) + (i & 3)) < width) ? st.s[i] : -INFINITY;
  }
  bf16x8_t op[FWD_AHEAD];
#pragma unroll
  for (int i = 0; i < FWD_AHEAD; ++i) op[i] = k_operand<D, KB, KS>(smem, lo, i);
  // ---- 1
  f32x16_t s_next;
  float mx = -INFINITY, ps = 0.f;
  bf16x8_t pop[2] = {};
  fence();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    s_next = mfma32(op[i % FWD_AHEAD], qop[i], i == 0 ? f32x16_t{0} : s_next);
    if (i + FWD_AHEAD < N) op[i % FWD_AHEAD] = k_operand<D, KB, KS>(smem, lo, i + FWD_AHEAD);
    else if (PREV) op[i % FWD_AHEAD] = v_operand<D, VB, KS>(smem, lo, i + FWD_AHEAD - N);
#pragma unroll
    for (int e = PER * i; e < PER * i + PER; e += 2) {
      if (PREV) { ps += st.p[e]; ps += st.p[e + 1]; }
      mx = max3(mx, st.s[e], st.s[e + 1]);
      asm volatile("" : "+v"(mx), "+v"(ps));   // stays between the matrix instructions
    }
    if (PREV && i == N / 2 - 1) pop[0] = pack_bf16x8(&st.p[0]);
    if (PREV && i == N - 1) pop[1] = pack_bf16x8(&st.p[8]);
    request(i);
    fence();
  }
  st.l += ps;
  // ---- 2
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (PREV) {
      st.oacc[i % (D / 32)] = mfma32(op[i % FWD_AHEAD], pop[i / (D / 32)], st.oacc[i % (D / 32)]);
      if (i + FWD_AHEAD < N) op[i % FWD_AHEAD] = v_operand<D, VB, KS>(smem, lo, i + FWD_AHEAD);
    }
#pragma unroll
    for (int e = PER * i; e < PER * i + PER; ++e) {
      st.p[e] = fast_exp2(__builtin_fmaf(st.s[e], scale_log2, -st.m));
      asm volatile("" : "+v"(st.p[e]));   // stays between the matrix instructions
    }
    if (i == N / 2 - 1) mx = half_max(mx) * scale_log2;
    request(N + i);
    fence();
  }
  if (__builtin_amdgcn_ballot_w64(mx - st.m > RESCALE_TH) != 0) {
    const float m_new = fmaxf(st.m, mx);
    const float alpha = fast_exp2(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;   // (l and O hold the sub-tiles up to j - 1)
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) st.oacc[dt] *= alpha;
#pragma unroll
    for (int i = 0; i < 16; ++i) st.p[i] = fast_exp2(__builtin_fmaf(st.s[i], scale_log2, -m_new));
  }
  st.s = s_next;
}

// keeps what is computed from x in a rare form of the code out of the registers of the code around it
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Waves per SIMD: the 32 x D accumulators of both branches and the q operand take most of 256 registers at D = 128, half
// of that at D = 64.
constexpr int fwd_occ(int D) { return D == 128 ? 2 : 3; }

// GAP: the window is not a multiple of 64 (a.gap > 0); the aligned case compiles without the extra key tile.
// FM: feature map of the linear branch (FM_* in mfma.hpp).
template <int D, bool GAP, int FM>
__global__ __launch_bounds__(256, fwd_occ(D)) void fwd_fused_kernel(FastFwdArgs a) {
  constexpr int KT = TileGeom<D>::KT, ND = D / 32, NB = TileGeom<D>::NB / 4;  // blocks of a 64-row tile per wave
  __shared__ __align__(16) unsigned char smem[4 * KT];
  const int lane = lane_id(), w = wave_id();
  const int r32 = lane & 31, h = lane >> 5;
  const LaneOff<D> lo = make_lane_off<D>(lane);
  const int W = a.W, Hq = a.Hq, Hkv = a.Hkv, G = a.G;

  // work id: consecutive ids share a KV head (its G query heads, then the next query tile); each XCD
  // (blockIdx % 8) gets one contiguous range of ids so K/V tiles are reused out of its own L2
  const int total = gridDim.x;
  const int bid = blockIdx.x;
  int wid = (total % 8 == 0) ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int hh = wid % G; wid /= G;
  const int ntq = a.ntile - a.qt0, Tq = 128 * ntq;  // query tiles and query rows per sequence
  const int qt = a.ntile - 1 - wid % ntq; wid /= ntq;  // late tiles first: they see the most keys (causal / start-up tiles)
  const int g = wid % Hkv;
  const int b = wid / Hkv;
  const int hq = g * G + hh;
  const int t0 = qt * 128;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  const size_t qtile_off = ((size_t)(b * Tq + t0 - 128 * a.qt0) * Hq + hq) * D;  // in the saved tensors
  const TileRows q_tile = split_rows(a.q, b, t0 - 128 * a.qt0, Hq, hq, D);
  const int qlive = min(q_tile.n, 128);  // rows of the tile that exist
  uint16_t* o_tile = a.o + (q_tile.p - a.q.back);
  // first row of a 64-key tile of this KV head
  auto k_rows = [&](int row) { return split_rows(a.k, b, row, Hkv, g, D); };
  auto v_rows = [&](int row) { return split_rows(a.v, b, row, Hkv, g, D); };
  const int myq = t0 + 32 * w + r32;
  const size_t stat_off = (size_t)(b * Hq + hq) * Tq + myq - 128 * a.qt0;

  // ------------------------------------------------------------------ softmax branch
  // key tiles of 64 from the diagonal (n = 0) down to kt_lo (n = ntiles-1); tile n uses LDS buffer n & 1.
  // K runs one tile ahead of V through the buffers (the S^T chain of a sub-tile is issued one step early).
  const int kt_lo = max(0, t0 - W);
  const int ntiles = (t0 + 128 - kt_lo) / 64;  // >= 2
  const DmaLane<D> dl = make_dma_lane<D>(lane, kstride);
  // (almost always every row of the sweep's tiles exists and lies in the back part: one base for all of them)
  const bool whole = kt_lo >= a.k.P && t0 + 128 <= a.k.P + a.k.Tb;
  const ptrdiff_t sweep_off = ((ptrdiff_t)((ptrdiff_t)b * a.k.Tb + kt_lo - a.k.P) * Hkv + g) * D;
  auto load_k = [&](int n) {
    const int it = ntiles - 1 - n;
    if (whole) tile_load_async_s<D, NB>(a.k.back + sweep_off + (size_t)(64 * it) * kstride, kstride, smem + (n & 1) * KT, w * NB, dl);
    else tile_load_async_s<D, NB>(k_rows(kt_lo + 64 * it), kstride, smem + (n & 1) * KT, w * NB, dl, opaque(lane));
  };
  auto load_v = [&](int n) {
    const int it = ntiles - 1 - n;
    if (whole) tile_load_async_s<D, NB>(a.v.back + sweep_off + (size_t)(64 * it) * kstride, kstride, smem + (2 + (n & 1)) * KT, w * NB, dl);
    else tile_load_async_s<D, NB>(v_rows(kt_lo + 64 * it), kstride, smem + (2 + (n & 1)) * KT, w * NB, dl, opaque(lane));
  };
  load_k(0);
  load_v(0);
  load_k(1);
  bf16x8_t qop[D / 16];
  {
    const uint16_t* qp = q_tile.p + (ptrdiff_t)min(32 * w + r32, qlive - 1) * (ptrdiff_t)qstride + 8 * h;
#pragma unroll
    for (int dk = 0; dk < D / 16; ++dk) qop[dk] = *reinterpret_cast<const bf16x8_t*>(qp + 16 * dk);
  }
  wait_vmem();
  __syncthreads();
  SweepState<D> sw;
  f32x16_t (&oacc)[ND] = sw.oacc;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) oacc[dt] = f32x16_t{0};
  sw.m = M_INIT; sw.l = 0.f;
  SweepGeom gm;
  gm.kt_lo = kt_lo; gm.ntiles = ntiles; gm.qa = t0 + 32 * w; gm.W = W - (GAP ? a.gap : 0);
  gm.kmin = a.kmin;
  qk_chain<D, 0, 1>(smem, lo, qop, sw.s);
  // step 0 has no earlier sub-tile to fold in; the step after the last one only folds
  const auto nothing = [](int) {};
  sweep_step<D, 0, false>(smem, lo, gm, 0, myq, a.scale_log2, qop, sw, lane, nothing);
  // Behind the barrier in front of step 2n + 1 the buffers of K tile n and V tile n - 1 are free: K tile n + 2 and V tile
  // n + 1 are requested load by load in the course of that step and have the next one to arrive.  (A wave that makes its
  // loads in one go stands still while the address unit works them off: 8 loads, 46 cycles each.)
  const ptrdiff_t tile_bytes = (ptrdiff_t)(128 * kstride), load_bytes = (ptrdiff_t)(2 * TileGeom<D>::RPB * kstride);
  const unsigned char* k_next = reinterpret_cast<const unsigned char*>(a.k.back + sweep_off) + (ntiles - 3) * tile_bytes + w * NB * load_bytes;
  const unsigned char* v_next = reinterpret_cast<const unsigned char*>(a.v.back + sweep_off) + (ntiles - 2) * tile_bytes + w * NB * load_bytes;
  const unsigned lds_wave = (unsigned)(size_t)RATTN_LDS(smem) + w * NB * 1024;
  auto odd_step = [&](int n, auto par) {   // step 2n + 1, par = n & 1
    constexpr int P = decltype(par)::value, EVERY = D / 16 / NB;
    const unsigned char *k_tile = k_next, *v_tile = v_next;
    bool go_k = n + 2 < ntiles, go_v = n + 1 < ntiles;
    // Otherwise each tile has a base of its own, in the tensor it lies in; requested in one go instead, a chunk of 4 x 2048
    // tokens behind rings of 512 takes 159.6 us against 156.5, one of 700 tokens 54.7 against 52.7.
    if (!whole) {
      const int row = kt_lo + 64 * (ntiles - 3 - n);
      if (go_k) k_tile = reinterpret_cast<const unsigned char*>(k_rows(row).p) + w * NB * load_bytes;  // (below the queries: whole)
      if (go_v) {
        const TileRows r = v_rows(row + 64);
        v_tile = reinterpret_cast<const unsigned char*>(r.p) + w * NB * load_bytes;
        if (r.n < 64) { load_v(n + 1); go_v = false; }
      }
    }
    sweep_step<D, 2 * P + 1, true>(smem, lo, gm, 2 * n + 1, myq, a.scale_log2, qop, sw, lane, [&](int i) {
      if (i % EVERY) return;
      const int part = i / EVERY % NB;
      if (i / EVERY < NB) {
        if (go_k) dma16s(k_tile + part * load_bytes, dl.off[part % TileGeom<D>::NV], lds_wave + P * KT + part * 1024);
      } else {
        if (go_v) dma16s(v_tile + part * load_bytes, dl.off[part % TileGeom<D>::NV], lds_wave + (3 - P) * KT + part * 1024);
      }
    });
    k_next -= tile_bytes;
    v_next -= tile_bytes;
  };
  for (int n = 0; n < ntiles; n += 2) {
    if (n > 0) sweep_step<D, 0, true>(smem, lo, gm, 2 * n, myq, a.scale_log2, qop, sw, lane, nothing);
    wait_vmem();
    __syncthreads();
    odd_step(n, std::integral_constant<int, 0>{});
    if (n + 1 < ntiles) {
      sweep_step<D, 2, true>(smem, lo, gm, 2 * n + 2, myq, a.scale_log2, qop, sw, lane, nothing);
      wait_vmem();
      __syncthreads();
      odd_step(n + 1, std::integral_constant<int, 1>{});
    }
  }
  {
    bf16x8_t pop[2];
    sum_and_pack(sw.p, sw.l, pop);
    if (ntiles & 1) pv_chain<D, 0, 0>(smem, lo, pop, oacc);
    else pv_chain<D, 1, 0>(smem, lo, pop, oacc);
  }
  const float m = sw.m;
  float l = sw.l;
  __syncthreads();
  // the two lowest key tiles are still resident: tile `it` sits in buffer (ntiles-1-it) & 1

  l = half_sum(l);
  const float inv_l = 1.f / l;
  float ss = 0.f;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) {
    oacc[dt] *= inv_l;
#pragma unroll
    for (int i = 0; i < 16; ++i) ss += oacc[dt][i] * oacc[dt][i];
  }
  ss = half_sum(ss);
  const float rs_val = rsqrtf(ss * (1.f / D) + a.eps);
  // key tile of the intra-chunk part starts at j0 = t0 - W; when W % 128 == 64 the first query tile that
  // reaches past the window has j0 = -64: no state yet (S = 0) and only its upper 64 keys exist
  // (with gap > 0 the tile at j0 = -128 reaches keys too: only through the extra 64 keys fetched below)
  const int j0 = t0 - W;
  const bool has_lin = j0 > -128 || (GAP && j0 == -128);
  if (a.xs_out) {
    if (!has_lin) {   // (with a linear branch LDS still holds the tiles that branch works on: x_s is stored after it)
      float vals[ND][16];
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) vals[dt][i] = oacc[dt][i];
      store_tile_transposed<D>(smem, vals, a.xs_out + qtile_off, qstride, w, lane);
    }
  }
  // x_s * r_s stays in fp32 across the linear branch: the output is rounded once, after the sum of the branches
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) oacc[dt] *= rs_val;
  const float lse_val = (m + log2f(l)) * LN2;

  // ------------------------------------------------------------------ linear branch
  // intra-chunk part on the resident tiles (phi applied to K in place), then the state product
  f32x16_t xr[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) xr[dt] = f32x16_t{0};
  float rr_val = rsqrtf(a.eps);
  if (has_lin) {
    const bool has_state = j0 >= 0;
    const int shift = has_state ? 0 : 1;                  // chunk tile ti is softmax tile ti - shift
    const int buf0 = (ntiles - 1 + shift) & 1;            // buffer of chunk tile 0 (tile 1 is the other one)
    bf16x8_t qfop[D / 16];
    {
      float x[D / 2];
#pragma unroll
      for (int dk = 0; dk < D / 16; ++dk) unpack_bf16x8(qop[dk], &x[8 * dk]);
      phi_rows<FM>(x, qfop);
    }
    const bool has_res = j0 > -128;  // the resident tiles hold keys of this chunk
    if (has_res) phi_tiles_inplace<FM, D>(has_state ? smem + buf0 * KT : nullptr, smem + (buf0 ^ 1) * KT);
    __syncthreads();
    // Key sub-tile u (keys j0 + 32u .. +31) meets query block w when 32u <= 32w + 31 + gap; a query sees
    // key_local <= q_local + gap.  Sub-tiles 0..3 are resident; with gap > 0 the top queries also reach
    // into the next 64 keys, fetched afterwards.
    const int gap = GAP ? a.gap : 0;
    const int u_hi = w + ((31 + gap) >> 5);
    auto intra_unit = [&](const unsigned char* kt, const unsigned char* vt, int ks, int u) {
      f32x16_t c = {0};
#pragma unroll
      for (int dk = 0; dk < D / 16; ++dk) c = mfma32(lds_row<D>(kt, lo, 32 * ks, dk), qfop[dk], c);
      float cv[16];
      if (32 * u + 31 > 32 * w + gap) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key_local = 32 * u + 8 * (i >> 2) + 4 * h + (i & 3);
          cv[i] = key_local > 32 * w + r32 + gap ? 0.f : c[i];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) cv[i] = c[i];
      }
      bf16x8_t cop[2] = {pack_bf16x8(&cv[0]), pack_bf16x8(&cv[8])};
#pragma unroll
      for (int mf = 0; mf < 2; ++mf) {
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) xr[dt] = mfma32(lds_trp<D>(vt, lo, 32 * ks + 16 * mf, dt), cop[mf], xr[dt]);
      }
    };
    for (int u = has_state ? 0 : (has_res ? 2 : 4); u <= min(3, u_hi); ++u) {
      const int bsel = buf0 ^ (u >> 1);
      intra_unit(smem + bsel * KT, smem + (2 + bsel) * KT, u & 1, u);
    }
    __syncthreads();
    if (GAP) {
      tile_load_async_s<D, NB>(k_rows(j0 + 128), kstride, smem, w * NB, dl, lane);
      tile_load_async_s<D, NB>(v_rows(j0 + 128), kstride, smem + 2 * KT, w * NB, dl, lane);
      wait_vmem();
      __syncthreads();
      phi_tiles_inplace<FM, D>(smem, nullptr);
      __syncthreads();
      for (int u = 4; u <= min(5, u_hi); ++u) intra_unit(smem, smem + 2 * KT, u & 1, u);
      __syncthreads();
    }
    if (has_state) {
      const uint16_t* sbase = a.states + ((size_t)(b * Hkv + g) * a.nstf + j0 / 128) * (D * D);
      constexpr int SB = D * TileGeom<D>::ROWB / 4096;  // blocks of the state tile per wave
      tile_load_async<D, SB>(sbase, D, smem, w * SB, lane);
      wait_vmem();
      __syncthreads();
#pragma unroll
      for (int kf = 0; kf < D / 16; ++kf)
#pragma unroll
        for (int dt = 0; dt < ND; ++dt) xr[dt] = mfma32(lds_row<D>(smem, lo, 32 * dt, kf), qfop[kf], xr[dt]);
      __syncthreads();
    }
    float sr = 0.f;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) sr += xr[dt][i] * xr[dt][i];
    sr = half_sum(sr);
    rr_val = rsqrtf(sr * (1.f / D) + a.eps);
  }
  if (a.xs_out) {
    float vals[ND][16];
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) vals[dt][i] = xr[dt][i];
    // (a tile without residual keys has x_r = 0, which backward knows from the tile's position: not stored)
    if (has_lin) {
      store_tile_transposed<D>(smem, vals, a.xr_out + qtile_off, qstride, w, lane);
      // x_s = (x_s r_s) / r_s: the accumulators hold the normalised rows by now
      const float inv_rs = 1.f / rs_val;
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) vals[dt][i] = oacc[dt][i] * inv_rs;
      store_tile_transposed<D>(smem, vals, a.xs_out + qtile_off, qstride, w, lane);
    }
    if (h == 0) {
      a.lse_out[stat_off] = lse_val;
      a.rs_out[stat_off] = rs_val;
      a.rr_out[stat_off] = rr_val;
    }
  }

  // ------------------------------------------------------------------ combination
  {
    float vals[ND][16];
    if (!a.gs && !a.gr) {  // no gains: one multiply-add per element, no loads
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) vals[dt][i] = __builtin_fmaf(rr_val, xr[dt][i], oacc[dt][i]);
    } else {
      // the head's two gain rows go through LDS (free since the last barrier; the store below uses the K tiles)
      float* gl = reinterpret_cast<float*>(smem + 2 * KT);
      if (threadIdx.x < D) {
        gl[threadIdx.x] = a.gs ? a.gs[hq * D + threadIdx.x] : 1.f;
        gl[D + threadIdx.x] = a.gr ? a.gr[hq * D + threadIdx.x] : 1.f;
      }
      __syncthreads();
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const int d0 = 32 * dt + 8 * i4 + 4 * h;
          const float4 g1 = *reinterpret_cast<const float4*>(gl + d0);
          const float4 g2 = *reinterpret_cast<const float4*>(gl + D + d0);
          const float ga[4] = {g1.x, g1.y, g1.z, g1.w}, gb[4] = {g2.x * rr_val, g2.y * rr_val, g2.z * rr_val, g2.w * rr_val};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * i4 + e;
            vals[dt][i] = ga[e] * oacc[dt][i] + gb[e] * xr[dt][i];
          }
        }
    }
    store_tile_transposed<D>(smem, vals, o_tile, qstride, w, lane, qlive);
  }
}

}  // namespace

void fast_fwd(const LayerDims& dm, const SeqTensors& t, const void* q, const float* gs, const float* gr, void* o,
              const SavedPtrs& sv, float* U, void* states, hipStream_t st) {
  const FastFwdPlan pl = fast_fwd_plan(dm);
  // `states` receives every chunk state; with a state stride the stored subset also goes to `saved`
  if (t.handover)
    chunk_states(dm, t, U, states, st);
  else if (pl.nstf > 0)
    rla_forward_states(dm, pl, t, U, states, st, sv.state_stride > 1 ? sv.states : nullptr, nullptr, sv.state_stride);
  FastFwdArgs a;
  a.q = {nullptr, (const uint16_t*)q, 0, t.Tb};
  a.k = {(const uint16_t*)t.k_front, (const uint16_t*)t.k, t.P, t.Tb};
  a.v = {(const uint16_t*)t.v_front, (const uint16_t*)t.v, t.P, t.Tb};
  a.gs = gs; a.gr = gr;
  a.o = (uint16_t*)o; a.xs_out = (uint16_t*)sv.xs; a.xr_out = (uint16_t*)sv.xr;
  a.lse_out = sv.lse; a.rs_out = sv.rs; a.rr_out = sv.rr;
  a.states = (const uint16_t*)states;
  a.B = dm.B; a.T = dm.T; a.Hq = dm.Hq; a.Hkv = dm.Hkv; a.G = dm.G; a.W = pl.W; a.gap = pl.gap; a.nstf = pl.nstf;
  a.ntile = dm.T / 128; a.qt0 = t.P / 128; a.kmin = t.kmin;
  a.scale_log2 = dm.scale * LOG2E; a.eps = dm.eps;
  ProfScope ps("fwd_fused_kernel", st);
  const dim3 grid((a.ntile - a.qt0) * dm.Hq * dm.B);
#define RATTN_FWD_LAUNCH(D_, FM_)                                             \
  do {                                                                        \
    if (a.gap > 0) fwd_fused_kernel<D_, true, FM_><<<grid, 256, 0, st>>>(a);  \
    else fwd_fused_kernel<D_, false, FM_><<<grid, 256, 0, st>>>(a);           \
  } while (0)
#define RATTN_FWD_MAP(D_)                                                     \
  switch (dm.phi) {                                                           \
    case PHI_RELU: RATTN_FWD_LAUNCH(D_, FM_RELU); break;                      \
    case PHI_IDENTITY: RATTN_FWD_LAUNCH(D_, FM_IDENTITY); break;              \
    default: RATTN_FWD_LAUNCH(D_, FM_SOFTMAX); break;                         \
  }
  if (dm.D == 64) { RATTN_FWD_MAP(64) } else { RATTN_FWD_MAP(128) }
#undef RATTN_FWD_MAP
#undef RATTN_FWD_LAUNCH
}

}  // namespace rattn
