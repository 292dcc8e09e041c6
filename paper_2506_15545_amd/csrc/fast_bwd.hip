// MFMA backward of the RAttention layer (same shape class as the MFMA forward: bf16, D = 128 or 64, T >= 128, any
// W >= 8; tiles and states are laid out for T rounded up to 128 and W rounded up to 64, see fast_fwd.hip).
// No floating-point atomics: dq is produced by a kernel that owns query tiles, dk/dv by a kernel that
// owns key tiles (and visits the G query heads of its KV head in turn); both recompute the attention
// probabilities from the saved log-sum-exp.
//
//   RMS  : through the two RMS norms (Sec. 3.2), as the prologue of the dq kernel: dx_s, dx_r (bf16 MFMA
//          operands, also written out for the kernels that follow), delta = <dx_s, x_s>, dgamma partials
//   states: S_[j] (Eq. 2, kept by the forward pass) and the reverse-time states R_[j] = sum_{later chunks} phi(q)^T dx_r
//   dq   : transposed, lane = query:  dQ^T = scale * K^T dS^T,  dS = P .* (dP - delta),  dP^T = V dXs^T
//          linear branch: dphi(Q)^T = S dXr^T + Kf^T (M^T .* (V dXr^T)), then the softmax Jacobian of phi
//   dkv  : transposed, lane = key:   dV^T = dXs^T P + dXr^T C + R^T Kf^T,
//          dK^T = scale * Q^T dS + J_phi(Qf^T dC + R V^T)
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include <type_traits>

namespace rattn {

namespace {

struct FastBwdArgs {
  SeqRows q, k, v;                  // the caller's tensors: Tc rows per sequence, rows past them read as the last one
  const uint16_t *dxs, *dxr;        // workspace and saved tensors are laid out for the padded length T
  const float* lse;                 // as the forward saved it
  // <dx_s, x_s> * scale and lse * log2(e), left by the dq kernel for the dk/dv kernels: fewer vector instructions per
  // (query, key) pair.  Scaled per pair there instead, everything else alike, in turn on one box: a step of the 3B-shaped
  // layer takes 895 us against 881 (runs of one side differ by 2 %), at head size 64 474 against 462, 12B-shaped 1210
  // against 1203.
  float *delta, *lse2;
  const uint16_t *states, *rstates;
  uint16_t *dq, *dk, *dv;
  float *dk_part, *dv_part;         // fp32 [nsplit][B,Tc,Hkv,D] when the query heads of a group are split (nsplit > 1)
  int nsplit, hps;                  // work-groups per key tile, query heads of each
  int B, T, Tc, Hq, Hkv, G, W, gap, nstf, nk, ntile;  // W: window rounded up to 64; true window = W - gap
  float scale, scale_log2;
  // inputs of the RMS-norm backward in the dq kernel's prologue, which fills dxs, dxr and delta above; rows of dO from
  // Tfull = 128 * (Tc / 128) on come from dO_tail [B,128,Hq,D], zero past row Tc (ragged lengths)
  const uint16_t *dO, *dO_tail, *xs, *xr;
  int Tfull;
  const float *rs, *rr, *gs, *gr;   // gains [Hq][D], NULL = ones
  float* dgpart;                    // gain-gradient partials [2][4 * ntile * B][Hq][D], NULL = not wanted
};

// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dgamma_reduce_kernel(DgammaSum dg) { dgamma_reduce_tile(dg, blockIdx.x); }

// the D/8 8-byte pieces of row `src` that a lane holds in accumulator layout (piece 4 ft + i4 = features
// 32ft + 8*i4 + 4h .. +3; the row's other half sits in lane ^ 32): fetched ahead of their use, unpacked by phi_row_clayout
template <int D>
__device__ __forceinline__ void load_row_clayout(const uint16_t* src, int h, bf16x4_t (&raw)[D / 8]) {
#pragma unroll
  for (int j = 0; j < D / 8; ++j) raw[j] = *reinterpret_cast<const bf16x4_t*>(src + 8 * j + 4 * h);
}

// phi of that row: x[4 j + e] = feature 8 j + 4 h + e
template <int D, int FM>
__device__ __forceinline__ void phi_row_clayout(const bf16x4_t (&raw)[D / 8], float (&x)[D / 2]) {
#pragma unroll
  for (int j = 0; j < D / 8; ++j) {
    f32x4_t f = __builtin_convertvector(raw[j], f32x4_t);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * j + e] = f[e];
  }
  if (FM == FM_RELU) {
#pragma unroll
    for (int i = 0; i < D / 2; ++i) x[i] = fmaxf(x[i], 0.f);
    return;
  }
  float m = x[0];
#pragma unroll
  for (int i = 1; i < D / 2; ++i) m = fmaxf(m, x[i]);
  m = half_max(m);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < D / 2; ++i) { x[i] = fast_exp2((x[i] - m) * LOG2E); s += x[i]; }
  s = half_sum(s);
  const float inv = 1.f / s;
#pragma unroll
  for (int i = 0; i < D / 2; ++i) x[i] *= inv;
}

// acc <- f .* (acc - <acc, f>)   (softmax Jacobian applied to a gradient held in accumulator layout);  ReLU map: acc <- acc where the input was positive, i.e. where f = max(x, 0) > 0
template <int D, int FM>
__device__ __forceinline__ void phi_jacobian(f32x16_t (&acc)[D / 32], const float (&f)[D / 2]) {
  if (FM == FM_RELU) {
#pragma unroll
    for (int ft = 0; ft < D / 32; ++ft)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[ft][i] = f[ft * 16 + i] > 0.f ? acc[ft][i] : 0.f;
    return;
  }
  float inner = 0.f;
#pragma unroll
  for (int ft = 0; ft < D / 32; ++ft)
#pragma unroll
    for (int i = 0; i < 16; ++i) inner += acc[ft][i] * f[ft * 16 + i];
  inner = half_sum(inner);
#pragma unroll
  for (int ft = 0; ft < D / 32; ++ft)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[ft][i] = f[ft * 16 + i] * (acc[ft][i] - inner);
}

template <int D>
__device__ __forceinline__ void load_bop(const uint16_t* rowp, int h, bf16x8_t (&op)[D / 16]) {
#pragma unroll
  for (int c = 0; c < D / 16; ++c) op[c] = *reinterpret_cast<const bf16x8_t*>(rowp + 16 * c + 8 * h);
}

// ------------------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void dq_subtile(const unsigned char* kt, const unsigned char* vt, int ks, int ka, int myq,
                                           int W, bool masked, float scale, float scale_log2, float lse2, float dl,
                                           const bf16x8_t (&qop)[D / 16], const bf16x8_t (&dxsop)[D / 16],
                                           f32x16_t (&acc)[D / 32], int lane, const LaneOff<D>& lo) {
  const int h = lane >> 5;
  f32x16_t s = {0}, dp = {0};
#pragma unroll
  for (int c = 0; c < D / 16; ++c) s = mfma32(lds_row<D>(kt, lo, 32 * ks, c), qop[c], s);
#pragma unroll
  for (int c = 0; c < D / 16; ++c) dp = mfma32(lds_row<D>(vt, lo, 32 * ks, c), dxsop[c], dp);
  // probabilities of the unmasked case; they depend on the first chain only, so they are scheduled into the
  // second chain (masked entries are zeroed afterwards, which equals masking the logits)
  float p[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) p[i] = fast_exp2(__builtin_fmaf(s[i], scale_log2, -lse2));
  // operand reads run four ahead of the matrix chains (the default schedule issues them one ahead, which
  // exposes the LDS latency once per MFMA); the exponentials go between the MFMAs of the dP chain
  __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
#pragma unroll
  for (int i = 0; i < D / 16 - 4; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
  }
  if (masked) {
    // in the window <=> 0 <= query - key < W: one unsigned compare per element against a per-lane base
    const unsigned dist0 = (unsigned)(myq - ka - 4 * h);
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = (dist0 - (unsigned)(8 * (i >> 2) + (i & 3)) < (unsigned)W) ? p[i] : 0.f;
  }
  float ds[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) ds[i] = p[i] * __builtin_fmaf(dp[i], scale, -dl);
  bf16x8_t dsop[2] = {pack_bf16x8(&ds[0]), pack_bf16x8(&ds[8])};
#pragma unroll
  for (int mf = 0; mf < 2; ++mf) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) acc[dt] = mfma32(lds_trp<D>(kt, lo, 32 * ks + 16 * mf, dt), dsop[mf], acc[dt]);
  }
}

// Backward of the two RMS norms (Sec. 3.2) for 32 consecutive query rows of one head, by one wave: D/8 lanes per row,
// 8 features each, four (D = 128) or eight rows per pass (row-contiguous 16-byte accesses).  With y = g * x * r, r = rsqrt(mean x^2 +
// eps):  dx = r g dy - x r^3 mean(g dy x),  dg += dy x r.  Stores d xs, d xr (bf16) and delta * scale, delta =
// rowsum(d xs * xs), to global memory for the later kernels and also into LDS: d xs in two 16-row pieces at `stage_s` and
// `stage_s` + one 64-row tile (rows 0..15 of each, swizzled row layout; the caller passes a 16-row-aligned address: these are
// exactly the LDS rows into which the same wave later loads its share of two 64-key tiles, so no other wave's
// tile load can land on rows that are still being read) and, if `stage_r` is given, d xr into rows 0..31 of that
// tile, delta * scale into dl_stage[0..31]; the wave
// takes them from there as MFMA operands / row statistics without waiting for (or re-reading) the global stores.
// dO, x_s, x_r are read once and d xs, d xr are not read again by this kernel: their accesses are marked
// non-temporal so that they do not push the K/V tiles, which neighbouring work-groups share, out of the L2.
// GAINS: gains other than one and/or gain gradients; the wave's gradient partials (sums over its 32 rows) go to
// dgp_s / dgp_r (D floats each) when those are given.
template <int D, bool GAINS>
__device__ __forceinline__ void rms_bwd_rows(const FastBwdArgs& a, int hq, size_t row0_off, const uint16_t* dO_row0,
                                             size_t qstride, size_t stat0, unsigned char* stage_s, unsigned char* stage_r, float* dl_stage,
                                             float* dgp_s, float* dgp_r, int lane) {
  typedef TileGeom<D> TG;
  constexpr int LPR = D / 8, RPP = 64 / LPR, NP = 32 / RPP;  // lanes per row, rows per pass, passes
  const int sub = lane / LPR, c = lane % LPR;
  auto row_sum = [](float x) { return D == 128 ? sum16(x) : sum8(x); };
  // A query tile none of whose rows has a key beyond its window (the first tiles of a sequence; every tile of a
  // causal layer, W >= T) has x_r = 0: the forward does not store it, no later kernel reads its d x_r, and neither
  // is touched here.  The caller passes `stage_r` exactly for the tiles that have a linear branch (wave-uniform).
  const bool with_r = stage_r != nullptr;
  uint16_t* dxs_w = const_cast<uint16_t*>(a.dxs);
  uint16_t* dxr_w = const_cast<uint16_t*>(a.dxr);
  float g1[8], g2[8], dg1[8], dg2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    g1[e] = (GAINS && a.gs) ? a.gs[hq * D + 8 * c + e] : 1.f;
    g2[e] = (GAINS && a.gr) ? a.gr[hq * D + 8 * c + e] : 1.f;
    dg1[e] = dg2[e] = 0.f;
  }
  // All rows are requested before the first is worked on: the loads below and the stores further down go through
  // pointers the compiler cannot tell apart, so inside one loop every iteration's loads would wait behind the
  // previous iteration's stores - eight memory round trips in a row instead of one.
  bf16x8_t dy_raw[NP], xs_raw[NP], xr_raw[NP];
  float rs_row[NP], rr_row[NP];
#pragma unroll
  for (int it = 0; it < NP; ++it) {
    const int r = RPP * it + sub;
    const size_t off = row0_off + (size_t)r * qstride + 8 * c;
    dy_raw[it] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t*>(dO_row0 + (size_t)r * qstride + 8 * c));
    xs_raw[it] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t*>(a.xs + off));
    rs_row[it] = a.rs[stat0 + r];
    rr_row[it] = a.rr[stat0 + r];
  }
  if (with_r) {
#pragma unroll
    for (int it = 0; it < NP; ++it)
      xr_raw[it] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t*>(
          a.xr + row0_off + (size_t)(RPP * it + sub) * qstride + 8 * c));
  } else {
#pragma unroll
    for (int it = 0; it < NP; ++it) xr_raw[it] = bf16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
  }
#pragma unroll
  for (int it = 0; it < NP; ++it) {
    const int r = RPP * it + sub;
    const size_t off = row0_off + (size_t)r * qstride + 8 * c;
    float dy[8], xs[8], xr[8];
    unpack_bf16x8(dy_raw[it], dy);
    unpack_bf16x8(xs_raw[it], xs);
    unpack_bf16x8(xr_raw[it], xr);
    const float r_s = rs_row[it], r_r = rr_row[it];
    float m1 = 0.f, m2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (GAINS) {
        dg1[e] = fmaf(dy[e] * xs[e], r_s, dg1[e]);
        dg2[e] = fmaf(dy[e] * xr[e], r_r, dg2[e]);
      }
      m1 = fmaf(g1[e] * dy[e], xs[e], m1);
      m2 = fmaf(g2[e] * dy[e], xr[e], m2);
    }
    m1 = row_sum(m1) * (1.f / D);
    m2 = row_sum(m2) * (1.f / D);
    const float b_s = r_s * r_s * r_s * m1, b_r = r_r * r_r * r_r * m2;
    float av[8], cv[8], dl = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      av[e] = r_s * g1[e] * dy[e] - xs[e] * b_s;
      cv[e] = r_r * g2[e] * dy[e] - xr[e] * b_r;
    }
    const bf16x8_t apk = pack_bf16x8(av);
    const bf16x8_t cpk = pack_bf16x8(cv);
    // delta from d xs as the matrix cores will see it (rounded to bf16): dS = P (dP - delta) is a near-cancellation
    // for peaked rows, and dP is formed from the rounded values
    unpack_bf16x8(apk, av);
#pragma unroll
    for (int e = 0; e < 8; ++e) dl = fmaf(av[e], xs[e], dl);
    __builtin_nontemporal_store(apk, reinterpret_cast<bf16x8_t*>(dxs_w + off));
    if (with_r) __builtin_nontemporal_store(cpk, reinterpret_cast<bf16x8_t*>(dxr_w + off));
    {  // staged in two 16-row pieces (see the function's header)
      const int R = r & 15;
      *reinterpret_cast<bf16x8_t*>(stage_s + (r >> 4) * TG::KT + R * TG::ROWB + ((c ^ swz<D>(R)) << 4)) = apk;
    }
    if (stage_r) *reinterpret_cast<bf16x8_t*>(stage_r + r * TG::ROWB + ((c ^ swz<D>(r)) << 4)) = cpk;
    dl = row_sum(dl);
    if (c == 0) { a.delta[stat0 + r] = dl * a.scale; dl_stage[r] = dl * a.scale; }
  }
  if (GAINS && dgp_s) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (D == 64) { dg1[e] += __shfl_xor(dg1[e], 8, 64); dg2[e] += __shfl_xor(dg2[e], 8, 64); }
      dg1[e] = rows_sum(dg1[e]);
      dg2[e] = rows_sum(dg2[e]);
    }
    if (sub == 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) { dgp_s[8 * c + e] = dg1[e]; dgp_r[8 * c + e] = dg2[e]; }
    }
  }
}

// GAINS: RMS gains other than one and/or gain gradients (see rms_bwd_rows); FM: feature map (FM_* in mfma.hpp)
// grid (ntile * Hq * B), 256 threads: 128 queries of one head, wave w owns 32.
// RAGGED: Tc is no multiple of 128, so the last tile has rows that do not exist (a whole-tile call compiles without the
// clamps and the second form of the tile loads: with them the kernel spills scalar registers, 0.264 against 0.256 ms).
template <int D, bool GAINS, int FM, bool RAGGED>
__global__ __launch_bounds__(256, D == 128 ? 2 : 3) void bwd_dq_kernel(FastBwdArgs a) {
  typedef TileGeom<D> TG;
  constexpr int KT = TG::KT, ND = D / 32, NB = TG::NB / 4;  // blocks of a 64-row tile per wave
  __shared__ __align__(16) unsigned char smem[4 * KT];
  __shared__ float dl_stage[128];
  const int lane = lane_id(), w = wave_id();
  const int r32 = lane & 31, h = lane >> 5;
  const LaneOff<D> lo = make_lane_off<D>(lane);
  const LaneOffN<D> lon = make_lane_off_n<D>(lane);
  const int T = a.T, W = a.W, Hq = a.Hq, Hkv = a.Hkv, G = a.G;
  const int total = gridDim.x, bid = blockIdx.x;
  int wid = (total % 8 == 0) ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int hh = wid % G; wid /= G;
  const int qt = a.ntile - 1 - wid % a.ntile; wid /= a.ntile;  // late tiles first: they see the most keys
  const int g = wid % Hkv;
  const int b = wid / Hkv;
  const int hq = g * G + hh;
  const int t0 = qt * 128;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  const size_t qtile_off = ((size_t)(b * T + t0) * Hq + hq) * D;   // in the saved / workspace tensors (padded length)
  // the caller's tensors: this query tile of q, dO, dq; 64-key tiles of k, v
  // (in one part each: the backward has no rows in front)
  const TileRows q_tile = {a.q.back + ((size_t)((size_t)b * a.Tc + t0) * Hq + hq) * D, RAGGED ? a.Tc - t0 : 128};
  const int qlive = RAGGED ? min(q_tile.n, 128) : 128;  // rows of the tile that exist
  const uint16_t* dO_tile = !RAGGED || t0 < a.Tfull ? a.dO + ((size_t)((size_t)b * a.Tc + t0) * Hq + hq) * D
                                         : a.dO_tail + ((size_t)b * 128 * Hq + hq) * D;
  uint16_t* dq_tile = a.dq + (q_tile.p - a.q.back);
  const ptrdiff_t kv_off = ((ptrdiff_t)((size_t)b * a.Tc) * Hkv + g) * D;
  auto k_rows = [&](int row) { return TileRows{a.k.back + kv_off + row * (ptrdiff_t)kstride, a.Tc - row}; };
  auto v_rows = [&](int row) { return TileRows{a.v.back + kv_off + row * (ptrdiff_t)kstride, a.Tc - row}; };
  auto load_tile = [&](const TileRows& src, unsigned char* tile) {
    tile_load_async<D, NB>(src.p, kstride, tile, w * NB, lane, RAGGED ? src.n : ALL_ROWS);
  };
  const int myq = t0 + 32 * w + r32;
  const size_t stat_off = (size_t)(b * Hq + hq) * T + myq;

  const int j0 = t0 - W, gap = a.gap;
  const bool has_lin = j0 > -128 || (gap > 0 && j0 == -128);
  {
    // RMS-norm backward of this wave's 32 rows first: everything below starts from d xs, d xr and delta
    float* dgp_s = nullptr;
    float* dgp_r = nullptr;
    if (GAINS && a.dgpart) {
      const int rb = ((b * a.ntile + qt) << 2) + w;  // one partial per wave: [2][4 * ntile * B][Hq][D]
      dgp_s = a.dgpart + ((size_t)rb * Hq + hq) * D;
      dgp_r = dgp_s + (size_t)4 * a.ntile * a.B * Hq * D;
    }
    rms_bwd_rows<D, GAINS>(a, hq, qtile_off + (size_t)(32 * w) * qstride, dO_tile + (size_t)(32 * w) * qstride, qstride,
                        stat_off - r32,
                        smem + 2 * KT + 16 * w * TG::ROWB, has_lin ? smem + 32 * w * TG::ROWB : nullptr,
                        dl_stage + 32 * w, dgp_s, dgp_r, lane);
  }
  // own rows, staged by this wave in the prologue: LDS executes a wave's accesses in order, and the reads below are
  // complete (lgkmcnt wait) before this wave's tile loads may overwrite the rows.  Every later tile load of wave w
  // covers rows 16w..16w+15 of a 64-key tile (or, at D = 128, rows 32w..32w+31 of the 128-row state tile): the staged
  // d xs rows sit in rows 16w..16w+15 of the two V tiles, the staged d xr rows in rows 32w..32w+31 of the tile at 0, so a
  // wave only ever overwrites its own staging rows.  (At D = 64 the state tile has 64 rows: a barrier instead, below.)
  bf16x8_t dxsop[D / 16];
  {
    const int R = 16 * w + (r32 & 15);  // query row r32 of this wave sits in row R of piece r32 / 16
    const unsigned char* rowp = smem + 2 * KT + (r32 >> 4) * KT + R * TG::ROWB;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) dxsop[c] = *reinterpret_cast<const bf16x8_t*>(rowp + (((2 * c + h) ^ swz<D>(R)) << 4));
  }
  const float dl = dl_stage[32 * w + r32];
  f32x16_t acc[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) acc[dt] = f32x16_t{0};

  // ---- linear branch: d phi(q)
  // Tiles and states are laid out for the window rounded up to 64 (W); with gap = W - true window > 0 a query
  // sees key_local <= q_local + gap of the chunk that starts at j0 = t0 - W, i.e. up to 64 keys past the two
  // 64-key tiles of the aligned layout (a third tile, handled after them), and the query tile at j0 = -128
  // reaches keys only through that third tile.
  if (has_lin) {
    const bool has_state = j0 >= 0, has_res = j0 > -128;
    const int u_hi = w + ((31 + gap) >> 5);
    bf16x8_t dxrop[D / 16];
#pragma unroll
    for (int c = 0; c < D / 16; ++c) dxrop[c] = lds_row<D>(smem, lo, 32 * w, c);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the staged rows are in registers
    if (D == 64) __syncthreads();
    // key sub-tile u (keys j0 + 32u .. +31): dC = V dXr^T, masked, then d phi(q)^T += phi(K)^T dC
    auto intra_unit = [&](const unsigned char* kt, const unsigned char* vt, int ks, int u) {
      f32x16_t c = {0};
#pragma unroll
      for (int kd = 0; kd < D / 16; ++kd) c = mfma32(lds_row<D>(vt, lo, 32 * ks, kd), dxrop[kd], c);
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
        for (int ft = 0; ft < ND; ++ft) acc[ft] = mfma32(lds_trp<D>(kt, lo, 32 * ks + 16 * mf, ft), cop[mf], acc[ft]);
      }
    };
    if (has_res) {
      if (has_state) {
        const uint16_t* sbase = a.states + ((size_t)(b * Hkv + g) * a.nstf + j0 / 128) * (D * D);
        constexpr int SB = D * TG::ROWB / 4096;  // blocks of the state tile per wave
        tile_load_async<D, SB>(sbase, D, smem, w * SB, lane);
        load_tile(v_rows(j0), smem + 2 * KT);
      }
      load_tile(v_rows(j0 + 64), smem + 3 * KT);
      wait_vmem();
      __syncthreads();
      if (has_state) {
#pragma unroll
        for (int kd = 0; kd < D / 16; ++kd) {
#pragma unroll
          for (int ft = 0; ft < ND; ++ft) acc[ft] = mfma32(lds_trn<D>(smem, lon, 16 * kd, ft), dxrop[kd], acc[ft]);
        }
      }
      __syncthreads();
      if (has_state) load_tile(k_rows(j0), smem);
      load_tile(k_rows(j0 + 64), smem + KT);
      wait_vmem();
      __syncthreads();
      if (has_state) phi_tile_inplace<FM, D>(smem, 128);
      else phi_tile_inplace<FM, D>(smem + KT, 64);
      __syncthreads();
      for (int u = has_state ? 0 : 2; u <= min(3, u_hi); ++u)
        intra_unit(smem + (u >> 1) * KT, smem + (2 + (u >> 1)) * KT, u & 1, u);
    }
    __syncthreads();
    if (gap > 0) {
      load_tile(k_rows(j0 + 128), smem);
      load_tile(v_rows(j0 + 128), smem + 2 * KT);
      wait_vmem();
      __syncthreads();
      phi_tile_inplace<FM, D>(smem, 64);
      __syncthreads();
      for (int u = 4; u <= min(5, u_hi); ++u) intra_unit(smem, smem + 2 * KT, u & 1, u);
      __syncthreads();
    }
  }

  // ---- softmax branch
  // The first key tile and the work-group's q tile are requested together: q goes into the two tile buffers the
  // key sweep does not need yet (rows 0..63 and 64..127), and every wave takes its own rows from there in both of the
  // layouts it needs, instead of two more round trips to global memory for row pieces.
  if (!has_lin) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the staged rows are in registers
  const float lse2 = a.lse[stat_off] * LOG2E;
  if (h == 0) a.lse2[stat_off] = lse2;
  const int kt_lo = max(0, t0 - W);
  const int ntiles = (t0 + 128 - kt_lo) / 64;
  {
    const int kt0 = kt_lo + 64 * (ntiles - 1);
    load_tile(k_rows(kt0), smem);
    load_tile(v_rows(kt0), smem + 2 * KT);
    tile_load_async<D, NB>(q_tile.p, qstride, smem + KT, w * NB, lane, RAGGED ? q_tile.n : ALL_ROWS);
    tile_load_async<D, NB>(q_tile.p + (size_t)64 * qstride, qstride, smem + 3 * KT, w * NB, lane, RAGGED ? q_tile.n - 64 : ALL_ROWS);
    wait_vmem();
    __syncthreads();
  }
  bf16x8_t qop[D / 16];
  {
    const unsigned char* qhalf = smem + ((w >> 1) ? 3 * KT : KT);
    const int R0 = 32 * (w & 1);
    if (has_lin) {  // phi(q) and its Jacobian close the linear branch
      const int row = R0 + r32;
      const unsigned char* rowp = qhalf + row * TG::ROWB + 8 * h;
      bf16x4_t qraw[D / 8];
#pragma unroll
      for (int j = 0; j < D / 8; ++j) qraw[j] = *reinterpret_cast<const bf16x4_t*>(rowp + ((j ^ swz<D>(row)) << 4));
      float qf[D / 2];
      phi_row_clayout<D, FM>(qraw, qf);
      phi_jacobian<D, FM>(acc, qf);
    }
#pragma unroll
    for (int c = 0; c < D / 16; ++c) qop[c] = lds_row<D>(qhalf, lo, R0, c);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __syncthreads();  // the sweep's second tile load reuses the q buffers
  }
  const int qa = t0 + 32 * w, qb = qa + 31;
  const DmaLane<D> dma_lane = make_dma_lane<D>(lane, kstride);
  // all key tiles of the sweep but the one in hand (the diagonal one, loaded above) lie below t0 + 64: every row of theirs
  // exists unless the query tile itself starts past the last whole 64-row tile
  const bool whole = !RAGGED || t0 + 64 <= a.Tc;
  const size_t sweep_off = ((size_t)((size_t)b * a.Tc + kt_lo) * Hkv + g) * D;
  const uint16_t *k_sweep = a.k.back + sweep_off, *v_sweep = a.v.back + sweep_off;
  const int Wm = W - gap;  // the true window: element masks and sub-tile skipping
  // one key tile; the buffer index is a compile-time constant so that every LDS address of the sub-tile code is a
  // per-lane register plus an immediate (the loop below is unrolled by two for that)
  auto tile_step = [&](int n, auto cur_c) {
    constexpr int cur = decltype(cur_c)::value;
    const int it = ntiles - 1 - n;
    if (n + 1 < ntiles) {
      const size_t off = (size_t)(64 * (it - 1)) * kstride;
      if (whole) {
        tile_load_async_s<D, NB>(k_sweep + off, kstride, smem + (cur ^ 1) * KT, w * NB, dma_lane);
        tile_load_async_s<D, NB>(v_sweep + off, kstride, smem + (2 + (cur ^ 1)) * KT, w * NB, dma_lane);
      } else {
        load_tile(k_rows(kt_lo + 64 * (it - 1)), smem + (cur ^ 1) * KT);
        load_tile(v_rows(kt_lo + 64 * (it - 1)), smem + (2 + (cur ^ 1)) * KT);
      }
    }
    const unsigned char* kt = smem + cur * KT;
    const unsigned char* vt = smem + (2 + cur) * KT;
    const int kt0 = kt_lo + 64 * it;
#pragma unroll
    for (int ks = 1; ks >= 0; --ks) {
      const int ka = kt0 + 32 * ks;
      const bool need = ka <= qb && ka + 31 >= qa - Wm + 1;
      if (need) {
        const bool full = ka + 31 <= qa && ka >= qb - Wm + 1;
        dq_subtile<D>(kt, vt, ks, ka, myq, Wm, !full, a.scale, a.scale_log2, lse2, dl, qop, dxsop, acc, lane, lo);
      }
    }
    wait_vmem();
    __syncthreads();
  };
  {
    int n = 0;
    for (; n + 1 < ntiles; n += 2) {
      tile_step(n, std::integral_constant<int, 0>{});
      tile_step(n + 1, std::integral_constant<int, 1>{});
    }
    if (n < ntiles) tile_step(n, std::integral_constant<int, 0>{});
  }
  float vals[ND][16];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) vals[dt][i] = acc[dt][i];
  store_tile_transposed<D>(smem, vals, dq_tile, qstride, w, lane, qlive);
}

// ------------------------------------------------------------------------------------------------
// LDS map of the dk/dv kernel at D = 128 (D = 64 has a kernel of its own below): three slots, each a 64-row q tile followed by a 64-row dx tile; 32 KB for the
// probabilities handed from the V-role to the K-role waves; per slot the 64 lse2 and 64 delta values (as the dq kernel leaves them) of
// its rows.  The linear branch uses the same space as two buffers of one 128-row q tile and one 128-row dx tile
// each: A = slots 0-1, B = slot 2 + the hand-over area (which first receives the reverse-state tile).
struct DkvLds {
  static constexpr int D = 128, SLOT = 2 * TileGeom<D>::KT, PEX = 3 * SLOT, STAT = PEX + 32768, BYTES = STAT + 3 * 2048;
  // dk, dv leave as two [128][D] tiles (fp32 rows padded by 16 bytes when they are partial sums)
  static constexpr int OUT = 128 * (4 * D + 16);
  static_assert(2 * OUT <= BYTES, "output staging");
};

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// grid (ntile * nsplit * Hkv * B), 512 threads: 128 keys of one KV head and `hps` of its query heads (all of them, unless
// there are too few key tiles to fill the chip: then every work-group leaves fp32 partial sums, see dkv_reduce_kernel).  Waves w and 7-w both work on key block w
// (lane = key) with complementary roles, so each keeps only one 128 x 32 accumulator and one set of operand
// rows and two waves (w and w+4, one of each role) fit on a SIMD:
//   V-role (waves 0-3): S^T = Q K^T -> P (also written to LDS, fp32),  dV^T += dXs^T P;
//                       linear branch: C = phi(Q) phi(K)^T (masked),   dV^T += dXr^T C + R-state rows * phi(K)
//   K-role (waves 4-7): dP = dXs V^T, then dS = P .* (dP - delta) * scale with the P of its partner,
//                       dK^T += Q^T dS;  linear branch: dC = dXr V^T (masked), dphi(K)^T += phi(Q)^T dC + R V^T,
//                       softmax Jacobian of phi before the softmax-branch terms are added.
// Per 32-query sub-tile one work-group barrier hands P over (LDS buffer alternates with the sub-tile parity).
// Query tiles run through three LDS buffers: tile s+2 is requested right after the first barrier of step s
// (every wave has then left tile s-1, whose buffer it takes) and each wave waits for its share of tile s+1
// before the second barrier of step s, so no further barrier is needed.  The loop has no other vector-memory
// operation (row statistics arrive with the tiles), which is what makes the explicit counter waits exact.
template <int FM>
__global__ __launch_bounds__(512) void bwd_dkv_kernel(FastBwdArgs a) {
  typedef DkvLds L;
  constexpr int D = L::D;
  typedef TileGeom<D> TG;
  constexpr int KT = TG::KT, ND = D / 32, NB = TG::NB / 8;  // blocks of a 64-row tile per wave
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* pex = smem + L::PEX;
  const int lane = lane_id(), w8 = wave_id();
  const bool krole = w8 >= 4;
  // key block of the wave: the K-role takes them in reverse, so that in the linear branch, where block j pairs with
  // 4 - j query sub-tiles, the two waves of every SIMD (w8 and w8 + 4) carry five sub-tiles between them
  const int w = krole ? 7 - w8 : w8;
  const int r32 = lane & 31, h = lane >> 5;
  const LaneOff<D> lo = make_lane_off<D>(lane);
  const int T = a.T, W = a.W, Hq = a.Hq, Hkv = a.Hkv;
  const int total = gridDim.x, bid = blockIdx.x;
  int wid = (total % 8 == 0) ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int kti = wid % a.ntile; wid /= a.ntile;
  const int hs = wid % a.nsplit; wid /= a.nsplit;
  const int g = wid % Hkv;
  const int b = wid / Hkv;
  const int h0 = g * a.G + hs * a.hps, G = min(a.hps, a.G - hs * a.hps);  // this work-group's query heads
  const int s0 = kti * 128;
  const int Tp = T - W;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  // this key tile in the caller's k, v (dk and dv have the same layout)
  const TileRows k_tile = split_rows(a.k, b, s0, Hkv, g, D);
  const ptrdiff_t myrow = (k_tile.p - a.k.back) + (ptrdiff_t)min(32 * w + r32, k_tile.n - 1) * (ptrdiff_t)kstride;
  const uint16_t* k_myrow = a.k.back + myrow;
  const uint16_t* v_myrow = a.v.back + myrow;
  const int mykey = s0 + 32 * w + r32;

  bf16x8_t xop[D / 16];  // V-role: K rows (phi(K) rows during the linear branch); K-role: V rows
  load_bop<D>(krole ? v_myrow : k_myrow, h, xop);
  f32x16_t acc[ND];
#pragma unroll
  for (int t = 0; t < ND; ++t) acc[t] = f32x16_t{0};  // V-role: dV^T; K-role: dK^T
  // what each role needs of its K rows right after the linear branch, fetched now so that no global load sits on the
  // path between the two branches: the K-role the row in accumulator layout (softmax Jacobian), the V-role a copy of
  // the raw rows (xop holds phi(K) meanwhile)
  // (one register set for both roles)
  bf16x8_t kkeep[D / 16];

  // ---- request machinery of the softmax branch (query tiles of 64 rows from s0 up to the last row that still
  // sees these keys); defined first because the linear branch already requests the first tiles
  const int n_qt = (min(s0 + 128 + W, T) - s0) / 64;
  const int nsteps = G * n_qt;
  const int ka = s0 + 32 * w;
  // per-lane part of the tile addresses (swizzled 16-byte chunk of this wave's NB blocks of a tile), computed once
  int ir[NB];
  unsigned lane_g[NB];  // bytes
  const int ip = lane % TG::CH;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    ir[i] = (NB * w8 + i) * TG::RPB + lane / TG::CH;
    lane_g[i] = (unsigned)(((size_t)ir[i] * qstride + ((ip ^ swz<D>(ir[i])) << 3)) * 2);
  }
  const unsigned lds_q = (unsigned)(size_t)RATTN_LDS(smem) + w8 * (NB * 1024);
  const unsigned lds_st = (unsigned)(size_t)RATTN_LDS(smem + L::STAT) + (krole ? 1024 : 0);
  const float* stat_base = (krole ? a.delta : a.lse2) + (size_t)(b * Hq + h0) * T + s0;  // 64 rows, 16 bytes per lane
  const size_t tile_g = ((size_t)(b * T + s0) * Hq + h0) * D;     // workspace tensors (padded length)
  const uint16_t* q_base = a.q.back + ((ptrdiff_t)((size_t)b * a.Tc + s0) * Hq + h0) * D;
  int is_h = 0, is_n = 0, is_buf = 0;  // head, tile and slot of the next tile to request
  auto issue = [&]() {
    const size_t off = (size_t)is_n * 64 * qstride + (size_t)is_h * D;
    const int live = a.Tc - s0 - 64 * is_n;  // rows of q from this tile's first on
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const unsigned dst = lds_q + is_buf * L::SLOT + i * 1024;
      if (live >= 64) dma16s(q_base + off, lane_g[i], dst);
      else dma16(q_base + off + (ptrdiff_t)min(ir[i], live - 1) * (ptrdiff_t)qstride + ((ip ^ swz<D>(ir[i])) << 3), dst);
      dma16s(a.dxs + tile_g + off, lane_g[i], dst + KT);
    }
    if (w == 0)  // one wave of each role: the row statistics that role consumes (lanes 16.. fetch duplicates)
      dma16s(stat_base + (size_t)is_h * T + 64 * is_n, 16 * (lane & 15), lds_st + is_buf * 2048);
    if (++is_n == n_qt) { is_n = 0; ++is_h; }
    if (++is_buf == 3) is_buf = 0;
  };
  int buf = 0, issued = 0;  // slot of the first softmax-branch tile, tiles requested so far

  // ---- linear branch
  // Key s pairs with the queries t >= s + (true window).  In the aligned layout (W) those of this key tile are
  // the "head" rows t = s0 + W + [0, nq) of every query head, masked to q_local >= key_local, plus everything
  // later through the reverse state.  With gap = W - true window > 0 a key also pairs with up to `gap` earlier
  // queries, q_local >= key_local - gap: they lie in the 64 rows before the head rows, which are run as a
  // second (first) pass per head.  A pass = 64 or 128 query rows of one head, q_local of its first row = qb0.
  const int gap = a.gap;
  const bool has_main = s0 < Tp;
  const bool has_pre = gap > 0 && s0 <= Tp;
  if (has_main || has_pre) {
    const int nq = has_main ? min(128, Tp - s0) : 0;  // head rows
    const int np = (has_pre ? 1 : 0) + (has_main ? 1 : 0), NV = G * np;
    if (krole) {
      bf16x4_t kraw[D / 8];
      load_row_clayout<D>(k_myrow, h, kraw);
#pragma unroll
      for (int j = 0; j < D / 16; ++j) kkeep[j] = __builtin_shufflevector(kraw[2 * j], kraw[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
    unsigned char* const qA = smem;
    unsigned char* const dA = smem + 2 * KT;
    unsigned char* const qB = smem + 4 * KT;
    unsigned char* const dB = smem + L::PEX;
    auto pass_is_pre = [&](int vh) { return has_pre && (vh % np) == 0; };
    auto issue_pass = [&](int vh, unsigned char* qb, unsigned char* db) {
      const bool pre = pass_is_pre(vh);
      const int row0 = s0 + W - (pre ? 64 : 0), nrow = pre ? 64 : nq;
      const int hd = h0 + vh / np;
      const uint16_t* dx = a.dxr + ((size_t)(b * T + row0) * Hq + hd) * D;   // workspace tensor (padded length)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        if (64 * half < nrow) {
          const TileRows qs = split_rows(a.q, b, row0 + 64 * half, Hq, hd, D);
          tile_load_async<D, NB>(qs.p, qstride, qb + half * KT, w8 * NB, lane, qs.n);
          tile_load_async<D, NB>(dx + (size_t)(64 * half) * qstride, qstride, db + half * KT, w8 * NB, lane);
        }
    };
    if (has_main && hs == 0) {
      const uint16_t* rbase = a.rstates + ((size_t)(b * Hkv + g) * a.nk + kti) * (D * D);
      constexpr int SB = D * TG::ROWB / 8192;  // blocks of the state tile per wave
      tile_load_async<D, SB>(rbase, D, dB, w8 * SB, lane);
    }
    issue_pass(0, qA, dA);
    if (!krole) {  // phi of the own K rows while the first tiles are on their way
      float x[D / 2];
#pragma unroll
      for (int c = 0; c < D / 16; ++c) { kkeep[c] = xop[c]; unpack_bf16x8(xop[c], &x[8 * c]); }
      phi_rows<FM>(x, xop);
    }
    wait_vmem();
    __syncthreads();
    if (has_main && hs == 0) {  // (the reverse state sums over the whole group: one of the work-groups that share it adds it)
      if (!krole) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c)
#pragma unroll
          for (int t = 0; t < ND; ++t) acc[t] = mfma32(lds_row<D>(dB, lo, 32 * t, c), xop[c], acc[t]);
      } else {
        const LaneOffN<D> lon = make_lane_off_n<D>(lane);
#pragma unroll
        for (int c = 0; c < D / 16; ++c)
#pragma unroll
          for (int t = 0; t < ND; ++t) acc[t] = mfma32(lds_trn<D>(dB, lon, 16 * c, t), xop[c], acc[t]);
      }
    }
    __syncthreads();  // buffer B is free again
    for (int vh = 0; vh < NV; ++vh) {
      const bool in_a = !(vh & 1);
      unsigned char* const qb = in_a ? qA : qB;
      unsigned char* const db = in_a ? dA : dB;
      // while this pass is worked on, the other buffer receives the next one, or after the last pass the
      // first query tiles of the softmax branch (slot 2 if buffer B is the free one, else slots 0 and 1)
      if (vh + 1 < NV) {
        issue_pass(vh + 1, in_a ? qB : qA, in_a ? dB : dA);
      } else if (in_a) {
        is_buf = buf = 2;
        issue();
        issued = 1;
      } else {
        issue();
        issued = 1;
        if (nsteps > 1) { issue(); issued = 2; }
      }
      const bool pre = pass_is_pre(vh);
      const int nrow = pre ? 64 : nq, qb0 = pre ? -64 : 0;
      phi_row_inplace<FM, D, 4>((int)threadIdx.x < 4 * nrow ? qb : nullptr, threadIdx.x >> 2, threadIdx.x & 3);
      __syncthreads();
      const unsigned char* mine = krole ? db : qb;    // rows contracted with xop
      const unsigned char* other = krole ? qb : db;   // rows accumulated into acc
      for (int u = 0; u < nrow / 32; ++u) {
        const int ql0 = qb0 + 32 * u;                  // q_local of the sub-tile's first row
        if (32 * w > ql0 + 31 + gap) continue;         // no pair of this key block and sub-tile
        f32x16_t c = {0};
#pragma unroll
        for (int e = 0; e < D / 16; ++e) c = mfma32(lds_row<D>(mine, lo, 32 * u, e), xop[e], c);
        float cv[16];
        if (32 * w + 31 > ql0 + gap) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int q_local = ql0 + 8 * (i >> 2) + 4 * h + (i & 3);
            cv[i] = 32 * w + r32 > q_local + gap ? 0.f : c[i];
          }
        } else {
#pragma unroll
          for (int i = 0; i < 16; ++i) cv[i] = c[i];
        }
        const bf16x8_t cop[2] = {pack_bf16x8(&cv[0]), pack_bf16x8(&cv[8])};
#pragma unroll
        for (int mf = 0; mf < 2; ++mf)
#pragma unroll
          for (int t = 0; t < ND; ++t) acc[t] = mfma32(lds_trp<D>(other, lo, 32 * u + 16 * mf, t), cop[mf], acc[t]);
      }
      wait_vmem();
      __syncthreads();  // what was requested above has landed, and everyone is done with this buffer
    }
    if (krole) {
      float kf[D / 2];
      bf16x4_t kraw[D / 8];
#pragma unroll
      for (int j = 0; j < D / 16; ++j) {
        kraw[2 * j] = __builtin_shufflevector(kkeep[j], kkeep[j], 0, 1, 2, 3);
        kraw[2 * j + 1] = __builtin_shufflevector(kkeep[j], kkeep[j], 4, 5, 6, 7);
      }
      phi_row_clayout<D, FM>(kraw, kf);
      phi_jacobian<D, FM>(acc, kf);
    } else {
#pragma unroll
      for (int c = 0; c < D / 16; ++c) xop[c] = kkeep[c];
    }
  }

  // ---- softmax branch
  const int Wm = W - gap;  // the true window: element masks and sub-tile skipping
  if (issued == 0) {
    issue();
    if (nsteps > 1) issue();
    wait_vmem();
    __syncthreads();
  } else if (issued == 1 && nsteps > 1) {
    issue();  // tile 0 is already visible; tile 1 has all of step 0 to arrive
  }
  // The loop exists once per role (the role is fixed per wave): with the role a compile-time constant the code between
  // two barriers has no role branches in it, which the instruction scheduler needs to overlap a chain with its reads.
  auto tile_loop = [&](auto role) {
    constexpr bool KR = decltype(role)::value;
    int n = 0;
    for (int step = 0; step < nsteps; ++step, buf = buf == 2 ? 0 : buf + 1, n = n + 1 == n_qt ? 0 : n + 1) {
      const unsigned char* qtile = smem + buf * L::SLOT;
      const unsigned char* dxt = qtile + KT;
      const float* stat_lds = reinterpret_cast<const float*>(smem + L::STAT + buf * 2048 + (KR ? 1024 : 0));
#pragma unroll
      for (int qs = 0; qs < 2; ++qs) {
        const int qa = s0 + 64 * n + 32 * qs;
        const bool need = qa + 31 >= ka && qa <= ka + 31 + Wm - 1;
        const bool full = qa >= ka + 31 && qa + 31 <= ka + Wm - 1;
        f32x4_t* px = reinterpret_cast<f32x4_t*>(pex + (w * 2 + qs) * 4096 + lane * 16);  // [i4][lane] x 16 bytes
        f32x16_t s = {0};
        float stat[16];
        bf16x8_t early[ND] = {};
        if (need) {
          const unsigned char* rows = KR ? dxt : qtile;
#pragma unroll
          for (int c = 0; c < D / 16; ++c) s = mfma32(lds_row<D>(rows, lo, 32 * qs, c), xop[c], s);
          __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);  // operand reads run four ahead of the chain
#pragma unroll
          for (int i = 0; i < D / 16 - 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4_t f = *reinterpret_cast<const f32x4_t*>(stat_lds + 32 * qs + 8 * i4 + 4 * h);
            stat[4 * i4] = f[0]; stat[4 * i4 + 1] = f[1]; stat[4 * i4 + 2] = f[2]; stat[4 * i4 + 3] = f[3];
          }
          if (!KR) {
            if (!full) {
              const unsigned dist0 = (unsigned)(qa + 4 * h - mykey);  // 0 <= query - key < W, one compare per element
#pragma unroll
              for (int i = 0; i < 16; ++i)
                s[i] = (dist0 + (unsigned)(8 * (i >> 2) + (i & 3)) < (unsigned)Wm) ? s[i] : -INFINITY;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = fast_exp2(__builtin_fmaf(s[i], a.scale_log2, -stat[i]));
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) px[i4 * 64] = f32x4_t{s[4 * i4], s[4 * i4 + 1], s[4 * i4 + 2], s[4 * i4 + 3]};
          } else {
            // The K-role gets here first: what does not need P is done while it would wait for the V-role.  Behind the barrier
            // instead, in turn on two boxes, a step of the 3B-shaped layer takes 881.1 us against 881.8 and 884.1 against
            // 881.6, 12B-shaped 1204.8 against 1205.1 and 1214.0 against 1211.8: 0.3 % at most.
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = __builtin_fmaf(s[i], a.scale, -stat[i]);
#pragma unroll
            for (int dt = 0; dt < ND; ++dt) early[dt] = lds_trp<D>(qtile, lo, 32 * qs, dt);
          }
        }
        if (qs == 1) {  // this wave's share of tile step+1 has landed (tile step+2 may still be in flight)
          if (step + 2 < nsteps) {
            if (w == 0) wait_vmcnt<2 * NB + 1>();
            else wait_vmcnt<2 * NB>();
          } else {
            wait_vmcnt<0>();
          }
        }
        __syncthreads();  // P of this sub-tile is in LDS
        if (qs == 0 && step + 2 < nsteps) issue();
        if (need) {
          float x[16];
          if (!KR) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = s[i];
          } else {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
              const f32x4_t pv = px[i4 * 64];
#pragma unroll
              for (int e = 0; e < 4; ++e) x[4 * i4 + e] = pv[e] * s[4 * i4 + e];
            }
          }
          const bf16x8_t xo[2] = {pack_bf16x8(&x[0]), pack_bf16x8(&x[8])};
          const unsigned char* cols = KR ? qtile : dxt;
#pragma unroll
          for (int mf = 0; mf < 2; ++mf)
#pragma unroll
            for (int dt = 0; dt < ND; ++dt)
              acc[dt] = mfma32(KR && mf == 0 ? early[dt] : lds_trp<D>(cols, lo, 32 * qs + 16 * mf, dt), xo[mf], acc[dt]);
        }
      }
    }
  };
  if (krole) tile_loop(std::true_type{});
  else tile_loop(std::false_type{});
  __syncthreads();
  // ---- dV^T (V-role) and dK^T (K-role) leave through LDS as two row-major tiles
  const int row = 32 * w + r32, tid = threadIdx.x, nlive = min(k_tile.n, 128);
  const ptrdiff_t out_off = k_tile.p - a.k.back;
  if (a.nsplit == 1) {
    unsigned char* tile = smem + (krole ? 2 * KT : 0);
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f32x4_t f = {acc[dt][4 * i4], acc[dt][4 * i4 + 1], acc[dt][4 * i4 + 2], acc[dt][4 * i4 + 3]};
        const int c = 4 * dt + i4;
        *reinterpret_cast<bf16x4_t*>(tile + row * TG::ROWB + ((c ^ swz<D>(row)) << 4) + 8 * h) =
            __builtin_convertvector(f, bf16x4_t);
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2 * 128 * TG::CH / 512; ++i) {
      const int id = tid + 512 * i;
      const int which = id / (128 * TG::CH), r = (id / TG::CH) % 128, pch = id % TG::CH;
      const int c = pch ^ swz<D>(r);
      const u32x4_t val = *reinterpret_cast<const u32x4_t*>(smem + which * 2 * KT + r * TG::ROWB + (pch << 4));
      uint16_t* dst = (which ? a.dk : a.dv) + out_off;
      if (r < nlive) __builtin_nontemporal_store(val, reinterpret_cast<u32x4_t*>(dst + (size_t)r * kstride + c * 8));
    }
  } else {
    float* tile = reinterpret_cast<float*>(smem + (krole ? L::OUT : 0));
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *reinterpret_cast<f32x4_t*>(tile + row * (D + 4) + 32 * dt + 8 * i4 + 4 * h) =
            f32x4_t{acc[dt][4 * i4], acc[dt][4 * i4 + 1], acc[dt][4 * i4 + 2], acc[dt][4 * i4 + 3]};
    __syncthreads();
    const size_t part_off = (size_t)hs * a.B * a.Tc * kstride;
#pragma unroll
    for (int i = 0; i < 2 * 128 * (D / 4) / 512; ++i) {
      const int id = tid + 512 * i;
      const int which = id / (128 * (D / 4)), r = (id / (D / 4)) % 128, c = id % (D / 4);
      const f32x4_t val = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<float*>(smem + which * L::OUT) + r * (D + 4) + 4 * c);
      float* dst = (which ? a.dk_part : a.dv_part) + part_off + out_off;
      if (r < nlive) *reinterpret_cast<f32x4_t*>(dst + (size_t)r * kstride + 4 * c) = val;
    }
  }
}

// The same for a head size of 64.  Both accumulators and both sets of operand rows of 32 keys fit in one wave's registers
// there, so a wave does everything for its keys: no hand-over of P, one barrier per 64-row query tile instead of one per 32
// rows, four waves of 256 registers with 70 KB of LDS, two work-groups per CU.  (The two-role kernel above instantiated for
// 64 features keeps one work-group per CU: 3B-shaped layer at D = 64, 0.273 ms against 0.200 ms.)
// LDS: three slots of a 64-row q tile and a 64-row dx tile, in the linear branch two buffers of 128 rows of each.
struct Dkv64Lds {
  static constexpr int KT = TileGeom<64>::KT, SLOT = 2 * KT, STAT = 8 * KT, BYTES = STAT + 3 * 2048, OUT = 128 * (4 * 64 + 16);
};

template <int FM>
__global__ __launch_bounds__(256, 2) void bwd_dkv64_kernel(FastBwdArgs a) {
  constexpr int D = 64;
  typedef TileGeom<D> TG;
  typedef Dkv64Lds L;
  constexpr int KT = TG::KT, NB = TG::NB / 4;  // blocks of a 64-row tile per wave
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = lane_id(), w = wave_id();
  const int r32 = lane & 31, h = lane >> 5;
  const LaneOff<D> lo = make_lane_off<D>(lane);
  const int T = a.T, W = a.W, Hq = a.Hq, Hkv = a.Hkv;
  const int total = gridDim.x, bid = blockIdx.x;
  int wid = (total % 8 == 0) ? (bid % 8) * (total / 8) + bid / 8 : bid;
  const int kti = wid % a.ntile; wid /= a.ntile;
  const int hs = wid % a.nsplit; wid /= a.nsplit;
  const int g = wid % Hkv;
  const int b = wid / Hkv;
  const int h0 = g * a.G + hs * a.hps, G = min(a.hps, a.G - hs * a.hps);  // this work-group's query heads
  const int s0 = kti * 128;
  const int Tp = T - W;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  const TileRows k_tile = split_rows(a.k, b, s0, Hkv, g, D);
  const ptrdiff_t out_off = k_tile.p - a.k.back;
  const ptrdiff_t myrow = out_off + (ptrdiff_t)min(32 * w + r32, k_tile.n - 1) * (ptrdiff_t)kstride;
  const int mykey = s0 + 32 * w + r32;
  bf16x8_t kop[D / 16], vop[D / 16];
  load_bop<D>(a.k.back + myrow, h, kop);
  load_bop<D>(a.v.back + myrow, h, vop);
  f32x16_t dk[2] = {{0}, {0}}, dv[2] = {{0}, {0}};

  // ---- linear branch (see bwd_dkv_kernel for the passes)
  const int gap = a.gap;
  const bool has_main = s0 < Tp;
  const bool has_pre = gap > 0 && s0 <= Tp;
  if (has_main || has_pre) {
    const int nq = has_main ? min(128, Tp - s0) : 0;
    const int np = (has_pre ? 1 : 0) + (has_main ? 1 : 0), NV = G * np;
    auto pass_is_pre = [&](int vh) { return has_pre && (vh % np) == 0; };
    auto issue_pass = [&](int vh) {  // 128 rows of q, then 128 rows of dx_r, in buffer vh & 1
      const bool pre = pass_is_pre(vh);
      const int row0 = s0 + W - (pre ? 64 : 0), nrow = pre ? 64 : nq, hd = h0 + vh / np;
      unsigned char* buf = smem + (vh & 1) * 4 * KT;
      const uint16_t* dx = a.dxr + ((size_t)(b * T + row0) * Hq + hd) * D;
#pragma unroll
      for (int half = 0; half < 2; ++half)
        if (64 * half < nrow) {
          const TileRows qs = split_rows(a.q, b, row0 + 64 * half, Hq, hd, D);
          tile_load_async<D, NB>(qs.p, qstride, buf + half * KT, w * NB, lane, qs.n);
          tile_load_async<D, NB>(dx + (size_t)(64 * half) * qstride, qstride, buf + (2 + half) * KT, w * NB, lane);
        }
    };
    if (has_main && hs == 0)  // the reverse state, where the second pass will go
      tile_load_async<D, NB>(a.rstates + ((size_t)(b * Hkv + g) * a.nk + kti) * (D * D), D, smem + 4 * KT, w * NB, lane);
    issue_pass(0);
    bf16x8_t kfop[D / 16];
    {
      float x[D / 2];
#pragma unroll
      for (int c = 0; c < D / 16; ++c) unpack_bf16x8(kop[c], &x[8 * c]);
      phi_rows<FM>(x, kfop);
    }
    wait_vmem();
    __syncthreads();
    if (has_main && hs == 0) {
      const LaneOffN<D> lon = make_lane_off_n<D>(lane);
      const unsigned char* R = smem + 4 * KT;
#pragma unroll
      for (int c = 0; c < D / 16; ++c)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          dv[t] = mfma32(lds_row<D>(R, lo, 32 * t, c), kfop[c], dv[t]);
          dk[t] = mfma32(lds_trn<D>(R, lon, 16 * c, t), vop[c], dk[t]);
        }
      __syncthreads();  // the second pass may take its place
    }
    for (int vh = 0; vh < NV; ++vh) {
      unsigned char* const qb = smem + (vh & 1) * 4 * KT;
      const unsigned char* const db = qb + 2 * KT;
      if (vh + 1 < NV) issue_pass(vh + 1);
      const bool pre = pass_is_pre(vh);
      const int nrow = pre ? 64 : nq, qb0 = pre ? -64 : 0;
      phi_tile_inplace<FM, D>(qb, nrow);
      __syncthreads();
      for (int u = 0; u < nrow / 32; ++u) {
        const int ql0 = qb0 + 32 * u;                  // q_local of the sub-tile's first row
        if (32 * w > ql0 + 31 + gap) continue;         // no pair of this key block and sub-tile
        f32x16_t c = {0}, dc = {0};
#pragma unroll
        for (int e = 0; e < D / 16; ++e) {
          c = mfma32(lds_row<D>(qb, lo, 32 * u, e), kfop[e], c);
          dc = mfma32(lds_row<D>(db, lo, 32 * u, e), vop[e], dc);
        }
        if (32 * w + 31 > ql0 + gap) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const bool out = 32 * w + r32 > ql0 + 8 * (i >> 2) + 4 * h + (i & 3) + gap;
            c[i] = out ? 0.f : c[i];
            dc[i] = out ? 0.f : dc[i];
          }
        }
        float cv[16], dcv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) { cv[i] = c[i]; dcv[i] = dc[i]; }
#pragma unroll
        for (int mf = 0; mf < 2; ++mf) {
          const bf16x8_t co = pack_bf16x8(&cv[8 * mf]), dco = pack_bf16x8(&dcv[8 * mf]);
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            dv[t] = mfma32(lds_trp<D>(db, lo, 32 * u + 16 * mf, t), co, dv[t]);
            dk[t] = mfma32(lds_trp<D>(qb, lo, 32 * u + 16 * mf, t), dco, dk[t]);
          }
        }
      }
      wait_vmem();
      __syncthreads();  // the next pass has landed, and everyone is done with this buffer
    }
    {
      float kf[D / 2];
      bf16x4_t kraw[D / 8];
      load_row_clayout<D>(a.k.back + myrow, h, kraw);
      phi_row_clayout<D, FM>(kraw, kf);
      phi_jacobian<D, FM>(dk, kf);
    }
  }

  // ---- softmax branch: query tiles of 64 rows from s0 up to the last row that still sees these keys, head by head.
  // Tile s+2 is requested right after the barrier of step s (every wave has then left tile s-1, whose slot it takes); the
  // loop has no other vector-memory operation, which is what makes the counter waits exact.
  const int Wm = W - gap;  // the true window: element masks and sub-tile skipping
  const int n_qt = (min(s0 + 128 + W, T) - s0) / 64;
  const int nsteps = G * n_qt;
  const int ka = s0 + 32 * w;
  int ir[NB];
  unsigned lane_g[NB];  // bytes
  const int ip = lane % TG::CH;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    ir[i] = (NB * w + i) * TG::RPB + lane / TG::CH;
    lane_g[i] = (unsigned)(((size_t)ir[i] * qstride + ((ip ^ swz<D>(ir[i])) << 3)) * 2);
  }
  const unsigned lds_q = (unsigned)(size_t)RATTN_LDS(smem) + w * (NB * 1024);
  const unsigned lds_st = (unsigned)(size_t)RATTN_LDS(smem + L::STAT) + w * 1024;
  const float* stat_base = (w == 0 ? a.lse2 : a.delta) + (size_t)(b * Hq + h0) * T + s0;
  const size_t tile_g = ((size_t)(b * T + s0) * Hq + h0) * D;
  const uint16_t* q_base = a.q.back + ((ptrdiff_t)((size_t)b * a.Tc + s0) * Hq + h0) * D;
  int is_h = 0, is_n = 0, is_buf = 0;  // head, tile and slot of the next tile to request
  auto issue = [&]() {
    const size_t off = (size_t)is_n * 64 * qstride + (size_t)is_h * D;
    const int live = a.Tc - s0 - 64 * is_n;  // rows of q from this tile's first on
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const unsigned dst = lds_q + is_buf * L::SLOT + i * 1024;
      if (live >= 64) dma16s(q_base + off, lane_g[i], dst);
      else dma16(q_base + off + (ptrdiff_t)min(ir[i], live - 1) * (ptrdiff_t)qstride + ((ip ^ swz<D>(ir[i])) << 3), dst);
      dma16s(a.dxs + tile_g + off, lane_g[i], dst + KT);
    }
    if (w < 2)  // wave 0: the log-sum-exp values of the rows, wave 1: delta (lanes 16.. fetch duplicates)
      dma16s(stat_base + (size_t)is_h * T + 64 * is_n, 16 * (lane & 15), lds_st + is_buf * 2048);
    if (++is_n == n_qt) { is_n = 0; ++is_h; }
    if (++is_buf == 3) is_buf = 0;
  };
  issue();
  if (nsteps > 1) issue();
  int buf = 0, n = 0;
  for (int step = 0; step < nsteps; ++step, buf = buf == 2 ? 0 : buf + 1, n = n + 1 == n_qt ? 0 : n + 1) {
    if (step + 1 < nsteps) {  // this wave's share of tile `step` has landed (the next tile may still be in flight)
      if (w < 2) wait_vmcnt<2 * NB + 1>();
      else wait_vmcnt<2 * NB>();
    } else {
      wait_vmcnt<0>();
    }
    __syncthreads();
    if (step + 2 < nsteps) issue();
    const unsigned char* qtile = smem + buf * L::SLOT;
    const unsigned char* dxt = qtile + KT;
    const float* lse_l = reinterpret_cast<const float*>(smem + L::STAT + buf * 2048);
    const float* del_l = lse_l + 256;
#pragma unroll
    for (int qs = 0; qs < 2; ++qs) {
      const int qa = s0 + 64 * n + 32 * qs;
      if (qa + 31 < ka || qa > ka + 31 + Wm - 1) continue;
      const bool full = qa >= ka + 31 && qa + 31 <= ka + Wm - 1;
      f32x16_t s = {0}, dp = {0};
#pragma unroll
      for (int c = 0; c < D / 16; ++c) s = mfma32(lds_row<D>(qtile, lo, 32 * qs, c), kop[c], s);
#pragma unroll
      for (int c = 0; c < D / 16; ++c) dp = mfma32(lds_row<D>(dxt, lo, 32 * qs, c), vop[c], dp);
      float ls[16], dl[16];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4_t f = *reinterpret_cast<const f32x4_t*>(lse_l + 32 * qs + 8 * i4 + 4 * h);
        const f32x4_t d = *reinterpret_cast<const f32x4_t*>(del_l + 32 * qs + 8 * i4 + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) { ls[4 * i4 + e] = f[e]; dl[4 * i4 + e] = d[e]; }
      }
      if (!full) {
        const unsigned dist0 = (unsigned)(qa + 4 * h - mykey);  // 0 <= query - key < W, one compare per element
#pragma unroll
        for (int i = 0; i < 16; ++i)
          s[i] = (dist0 + (unsigned)(8 * (i >> 2) + (i & 3)) < (unsigned)Wm) ? s[i] : -INFINITY;
      }
      float p[16], ds[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        p[i] = fast_exp2(__builtin_fmaf(s[i], a.scale_log2, -ls[i]));
        ds[i] = p[i] * __builtin_fmaf(dp[i], a.scale, -dl[i]);
      }
#pragma unroll
      for (int mf = 0; mf < 2; ++mf) {
        const bf16x8_t po = pack_bf16x8(&p[8 * mf]), dso = pack_bf16x8(&ds[8 * mf]);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          dv[t] = mfma32(lds_trp<D>(dxt, lo, 32 * qs + 16 * mf, t), po, dv[t]);
          dk[t] = mfma32(lds_trp<D>(qtile, lo, 32 * qs + 16 * mf, t), dso, dk[t]);
        }
      }
    }
  }
  __syncthreads();
  // ---- dV^T and dK^T leave through LDS as two row-major tiles
  const int row = 32 * w + r32, tid = threadIdx.x, nlive = min(k_tile.n, 128);
  if (a.nsplit == 1) {
#pragma unroll
    for (int which = 0; which < 2; ++which)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x16_t& x = which ? dk[dt] : dv[dt];
          f32x4_t f = {x[4 * i4], x[4 * i4 + 1], x[4 * i4 + 2], x[4 * i4 + 3]};
          const int c = 4 * dt + i4;
          *reinterpret_cast<bf16x4_t*>(smem + which * 2 * KT + row * TG::ROWB + ((c ^ swz<D>(row)) << 4) + 8 * h) =
              __builtin_convertvector(f, bf16x4_t);
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2 * 128 * TG::CH / 256; ++i) {
      const int id = tid + 256 * i;
      const int which = id / (128 * TG::CH), r = (id / TG::CH) % 128, pch = id % TG::CH;
      const int c = pch ^ swz<D>(r);
      const u32x4_t val = *reinterpret_cast<const u32x4_t*>(smem + which * 2 * KT + r * TG::ROWB + (pch << 4));
      uint16_t* dst = (which ? a.dk : a.dv) + out_off;
      if (r < nlive) __builtin_nontemporal_store(val, reinterpret_cast<u32x4_t*>(dst + (size_t)r * kstride + c * 8));
    }
  } else {
#pragma unroll
    for (int which = 0; which < 2; ++which)
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x16_t& x = which ? dk[dt] : dv[dt];
          *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(smem + which * L::OUT) + row * (D + 4) + 32 * dt + 8 * i4 + 4 * h) =
              f32x4_t{x[4 * i4], x[4 * i4 + 1], x[4 * i4 + 2], x[4 * i4 + 3]};
        }
    __syncthreads();
    const size_t part_off = (size_t)hs * a.B * a.Tc * kstride;
#pragma unroll
    for (int i = 0; i < 2 * 128 * (D / 4) / 256; ++i) {
      const int id = tid + 256 * i;
      const int which = id / (128 * (D / 4)), r = (id / (D / 4)) % 128, c = id % (D / 4);
      const f32x4_t val = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<float*>(smem + which * L::OUT) + r * (D + 4) + 4 * c);
      float* dst = (which ? a.dk_part : a.dv_part) + part_off + out_off;
      if (r < nlive) *reinterpret_cast<f32x4_t*>(dst + (size_t)r * kstride + 4 * c) = val;
    }
  }
}

// dk, dv = sum of the nsplit partial sums, in order.  One thread per eight elements, blockIdx.y = which.
__global__ __launch_bounds__(256) void dkv_reduce_kernel(const float* __restrict__ dk_part, const float* __restrict__ dv_part,
                                                         uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, size_t n, int nsplit) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i >= n) return;
  const float* src = (blockIdx.y ? dk_part : dv_part) + i;
  f32x4_t s0 = *reinterpret_cast<const f32x4_t*>(src), s1 = *reinterpret_cast<const f32x4_t*>(src + 4);
  for (int k = 1; k < nsplit; ++k) {
    s0 += *reinterpret_cast<const f32x4_t*>(src + k * n);
    s1 += *reinterpret_cast<const f32x4_t*>(src + k * n + 4);
  }
  const float x[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
  *reinterpret_cast<bf16x8_t*>((blockIdx.y ? dk : dv) + i) = pack_bf16x8(x);
}

}  // namespace

void dgamma_reduce(const DgammaSum& dg, hipStream_t st) {
  ProfScope ps("dgamma_reduce_kernel", st);
  dgamma_reduce_kernel<<<dg.tiles(), 256, 0, st>>>(dg);
}

void fast_bwd(const LayerDims& dm, int Tc, const void* q, const void* k, const void* v, const float* gs, const float* gr,
              const SavedPtrs& sv, const void* dO, const void* dO_tail, void* dq, void* dk, void* dv, float* dgs,
              float* dgr, const FastBwdWs& ws, hipStream_t st) {
  const FastBwdPlan pl = fast_bwd_plan(dm);
  // The RMS-norm backward runs as the prologue of the dq kernel (each wave on its own rows); the variant with
  // gains also leaves per-wave partials of the gain gradients, summed afterwards in a fixed order.
  const bool gains = gs || gr || dgs || dgr;
  FastBwdArgs a;
  a.q = {nullptr, (const uint16_t*)q, 0, Tc};
  a.k = {nullptr, (const uint16_t*)k, 0, Tc};
  a.v = {nullptr, (const uint16_t*)v, 0, Tc};
  a.dxs = (const uint16_t*)ws.dxs; a.dxr = (const uint16_t*)ws.dxr;
  a.lse = sv.lse; a.delta = ws.delta; a.lse2 = ws.delta + (size_t)dm.B * dm.Hq * dm.T;
  // chunk states of the forward pass: kept in `saved`, or (state policy "rebuild") built again here from k and v
  // (or, with a state stride, every m-th kept and the ones in between built again from those)
  const bool all_kept = sv.states && sv.state_stride <= 1;
  if (!all_kept && pl.fwd.nstf > 0) {
    SeqTensors t;
    t.k = k; t.v = v; t.Tb = Tc;
    rla_forward_states(dm, pl.fwd, t, ws.U, ws.states, st, nullptr, sv.state_stride > 1 ? sv.states : nullptr, sv.state_stride);
  }
  a.states = (const uint16_t*)(all_kept ? sv.states : ws.states); a.rstates = (const uint16_t*)ws.rstates;
  a.dq = (uint16_t*)dq; a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv;
  a.dk_part = ws.dkv_part;
  a.dv_part = ws.dkv_part + (size_t)pl.nsplit * dm.B * Tc * dm.Hkv * dm.D;
  a.nsplit = pl.nsplit; a.hps = (dm.G + pl.nsplit - 1) / pl.nsplit;
  a.B = dm.B; a.T = dm.T; a.Tc = Tc; a.Tfull = Tc / 128 * 128;
  a.Hq = dm.Hq; a.Hkv = dm.Hkv; a.G = dm.G; a.W = pl.fwd.W; a.gap = pl.fwd.gap;
  a.nstf = pl.fwd.nstf; a.nk = pl.nk; a.ntile = dm.T / 128;
  a.scale = dm.scale; a.scale_log2 = dm.scale * LOG2E;
  a.dO = (const uint16_t*)dO; a.dO_tail = (const uint16_t*)dO_tail;
  a.xs = (const uint16_t*)sv.xs; a.xr = (const uint16_t*)sv.xr;
  a.rs = sv.rs; a.rr = sv.rr; a.gs = gs; a.gr = gr;
  a.dgpart = (dgs || dgr) ? ws.dgpart : nullptr;
  // (softmax and ReLU maps only: with the identity map the host layer sends every call that keeps `saved` to the
  // general kernels, see make_layout)
  const bool relu = dm.phi == PHI_RELU;
  {
    ProfScope ps("bwd_dq_kernel", st);
    const dim3 grid(a.ntile * dm.Hq * dm.B);
    const bool ragged = Tc != dm.T;
#define RATTN_DQ_LAUNCH(D_, FM_)                                                         \
  do {                                                                                   \
    if (gains && ragged) bwd_dq_kernel<D_, true, FM_, true><<<grid, 256, 0, st>>>(a);    \
    else if (gains) bwd_dq_kernel<D_, true, FM_, false><<<grid, 256, 0, st>>>(a);        \
    else if (ragged) bwd_dq_kernel<D_, false, FM_, true><<<grid, 256, 0, st>>>(a);       \
    else bwd_dq_kernel<D_, false, FM_, false><<<grid, 256, 0, st>>>(a);                  \
  } while (0)
    if (dm.D == 64) {
      if (relu) RATTN_DQ_LAUNCH(64, FM_RELU); else RATTN_DQ_LAUNCH(64, FM_SOFTMAX);
    } else {
      if (relu) RATTN_DQ_LAUNCH(128, FM_RELU); else RATTN_DQ_LAUNCH(128, FM_SOFTMAX);
    }
#undef RATTN_DQ_LAUNCH
  }
  rla_reverse_states(dm, pl, q, Tc, ws.dxr, ws.U, ws.rstates, st, DgammaSum{a.dgpart, dgs, dgr, pl.RB, dm.Hq * dm.D});
  // the dk/dv kernel needs more LDS than a launch gets by default: raised once per instantiation
  static const bool lds_attr = [] {
    auto raise = [](const void* f, int bytes) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess; };
    return raise(reinterpret_cast<const void*>(bwd_dkv_kernel<FM_SOFTMAX>), DkvLds::BYTES) &&
           raise(reinterpret_cast<const void*>(bwd_dkv_kernel<FM_RELU>), DkvLds::BYTES) &&
           raise(reinterpret_cast<const void*>(bwd_dkv64_kernel<FM_SOFTMAX>), Dkv64Lds::BYTES) &&
           raise(reinterpret_cast<const void*>(bwd_dkv64_kernel<FM_RELU>), Dkv64Lds::BYTES);
  }();
  (void)lds_attr;
  {
    ProfScope ps("bwd_dkv_kernel", st);
    const dim3 kgrid(a.ntile * a.nsplit * dm.Hkv * dm.B);
    if (dm.D == 64) {
      if (relu) bwd_dkv64_kernel<FM_RELU><<<kgrid, 256, Dkv64Lds::BYTES, st>>>(a);
      else bwd_dkv64_kernel<FM_SOFTMAX><<<kgrid, 256, Dkv64Lds::BYTES, st>>>(a);
    } else {
      if (relu) bwd_dkv_kernel<FM_RELU><<<kgrid, 512, DkvLds::BYTES, st>>>(a);
      else bwd_dkv_kernel<FM_SOFTMAX><<<kgrid, 512, DkvLds::BYTES, st>>>(a);
    }
  }
  if (a.nsplit > 1) {
    ProfScope ps("dkv_reduce_kernel", st);
    const size_t n = (size_t)dm.B * Tc * dm.Hkv * dm.D;
    dkv_reduce_kernel<<<dim3((unsigned)((n / 8 + 255) / 256), 2), 256, 0, st>>>(a.dk_part, a.dv_part, a.dk, a.dv, n, a.nsplit);
  }
}

}  // namespace rattn
