// Chunk states of the linear branch for the MFMA paths (Eq. 2): chunk-local outer-product sums on the
// matrix cores, then an element-wise scan over chunks in fp32, stored as bf16 MFMA operands.
// States are kept transposed, [value feature d][phi feature f], because that is the row-major operand
// the consumers need.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace rattn {

namespace {

struct ChunkArgs {
  SeqRows a;           // rows that go through phi  (k, or q for the reverse states)
  SeqRows b;           // rows multiplied in        (v, or dx_r)
  float* U;            // [B,Hkv,nchunks,D,D] fp32, U^T = B^T phi(A)
  int H, GA, GS;       // heads in a/b, heads summed per kv head, work-groups that share them: product c of work-group s is
                       // number c GS + s, a sum over heads s ceil(GA / GS) .. of the group
  int tok_off;         // token index = t' + tok_off
  int skip_m, skip_head, skip_per;  // skip_m > 1: product c leads from state i = (c - skip_head) / skip_per to i + 1 and is
                                    // left out when that state is a stored one ((i + 1) % skip_m == 0) or c < skip_head
  int first_lo, first_n, rest_lo, ckeys, tok_end;  // chunk 0 = [first_lo, +first_n); chunk c > 0 = ckeys tokens from
                                                   // rest_lo + ckeys (c-1); every chunk is clipped at tok_end
};

// grid (nchunks GS, Hkv, B), 256 threads.  D = 128: wave w owns rows d in [32w, 32w+32) of U^T; D = 64: one of its four
// 32 x 32 tiles.
template <int D, int FM>
__global__ __launch_bounds__(256, 2) void rla_chunk_kernel(ChunkArgs p) {
  constexpr int KT = TileGeom<D>::KT, NB = TileGeom<D>::NB / 4, NF = D == 128 ? 4 : 1;
  __shared__ __align__(16) unsigned char smem[4 * KT];
  unsigned char* At = smem;
  unsigned char* Bt = smem + 2 * KT;
  const int c = blockIdx.x / p.GS, g = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int per = (p.GA + p.GS - 1) / p.GS, ga0 = (int)(blockIdx.x % p.GS) * per, ga1 = min(ga0 + per, p.GA);
  if (p.skip_m > 1 && (c < p.skip_head || ((c - p.skip_head) / p.skip_per + 1) % p.skip_m == 0)) return;  // block-uniform
  const int lane = lane_id(), w = wave_id();
  const int r32 = lane & 31, h = lane >> 5;
  const int lo = c == 0 ? p.first_lo : p.rest_lo + p.ckeys * (c - 1);
  const int ntok = min(c == 0 ? p.first_n : p.ckeys, p.tok_end - lo);  // 64 or 128
  const size_t rstride = (size_t)p.H * D;
  const DmaLane<D> dl = make_dma_lane<D>(lane, rstride);
  const int dt = D == 128 ? w : w & 1, ft0 = D == 128 ? 0 : w >> 1;
  // per-lane offsets of the transposed operand reads (natural contraction order, see lds_trn)
  int boff[2], aoff[NF][2];
#pragma unroll
  for (int ab = 0; ab < 2; ++ab) {
    boff[ab] = tr_lane_off<D>(8 * h + 4 * ab, dt, lane);
#pragma unroll
    for (int f = 0; f < NF; ++f) aoff[f][ab] = tr_lane_off<D>(8 * h + 4 * ab, ft0 + f, lane);
  }
  f32x16_t acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x16_t{0};
  for (int ga = ga0; ga < ga1; ++ga) {
    const int row = lo + p.tok_off, hd = g * p.GA + ga;   // chunks start at multiples of 64 rows
    if (ga > ga0) __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half)
      if (64 * half < ntok) {
        tile_load_async_s<D, NB>(split_rows(p.a, b, row + 64 * half, p.H, hd, D), rstride, At + half * KT, w * NB, dl, lane);
        tile_load_async_s<D, NB>(split_rows(p.b, b, row + 64 * half, p.H, hd, D), rstride, Bt + half * KT, w * NB, dl, lane);
      }
    wait_vmem();
    __syncthreads();
    phi_tile_inplace<FM, D>(At, ntok);
    __syncthreads();
    // rolled on purpose: fully unrolled, the operand reads of all sub-blocks are hoisted and the kernel needs twice
    // the registers, which halves the work-groups per CU of a kernel that lives on memory-level parallelism
#pragma unroll 1
    for (int ks = 0; ks < ntok / 16; ++ks) {
      const int k0 = 16 * ks * TileGeom<D>::ROWB;
      const bf16x8_t aop = lds_tr2(Bt + boff[0] + k0, Bt + boff[1] + k0);
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f] = mfma32(aop, lds_tr2(At + aoff[f][0] + k0, At + aoff[f][1] + k0), acc[f]);
    }
  }
  float* out = p.U + ((size_t)(b * Hkv + g) * gridDim.x + blockIdx.x) * (D * D);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int d = 32 * dt + 8 * (i >> 2) + 4 * h + (i & 3);
      out[(size_t)d * D + 32 * (ft0 + f) + r32] = acc[f][i];
    }
}

// Exclusive scan over chunks, every state element independently, fp32 accumulation, bf16 output.  A state spans
// PER chunk products (1, or 2 when the products cover 64 keys each; reverse: times the work-groups that share the heads).
//   forward: state[0] = sum of the `head` products in front of it; state[i+1] = state[i] + the next `per` products
//   reverse: state[n-1] = 0; state[i] = state[i+1] + products per*i .. per*i + per - 1 (those that exist)
// grid (D*D/1024, Hkv, B), 256 threads, 4 elements per thread.  Blocks with z >= B (reverse scan, `dg.part` given) sum gain
// gradients instead: a launch of its own for those took 4.7 us between kernels that do not need them.
// Forward scan with m > 1: `subset` (may be NULL) also receives states 0, m, 2m, ... ([B,Hkv,ceil(nst/m),128,128]);
// `restart` (may be NULL) holds such a subset, and the running sum is replaced by the stored state at every multiple
// of m (the products that lead to a stored state are then never used and need not exist).
template <int D, bool REV, int PER>
__global__ __launch_bounds__(256) void rla_scan_kernel(const float* __restrict__ U, uint16_t* __restrict__ states,
                                                       int nchunks, int nst, int head,
                                                       uint16_t* __restrict__ subset, const uint16_t* __restrict__ restart,
                                                       int m, int B, DgammaSum dg) {
  const int g = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  if (REV && b >= B) {
    dgamma_reduce_tile(dg, ((b - B) * gridDim.y + g) * gridDim.x + blockIdx.x);
    return;
  }
  const int e4 = (blockIdx.x * 256 + threadIdx.x) * 4;
  constexpr int N = D * D;
  const float* Ub = U + (size_t)(b * Hkv + g) * nchunks * N + e4;
  uint16_t* Sb = states + (size_t)(b * Hkv + g) * nst * N + e4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  const int nsub = (!REV && m > 1) ? (nst + m - 1) / m : 0;
  const size_t sub0 = (size_t)(b * Hkv + g) * nsub * N + e4;
  auto put = [&](int i) {
    if (!REV && restart && i % m == 0) {  // continue from the state the forward pass stored
      const bf16x4_t s = *reinterpret_cast<const bf16x4_t*>(restart + sub0 + (size_t)(i / m) * N);
      acc = make_float4((float)s[0], (float)s[1], (float)s[2], (float)s[3]);
    }
    f32x4_t f = {acc.x, acc.y, acc.z, acc.w};
    const bf16x4_t o = __builtin_convertvector(f, bf16x4_t);
    *reinterpret_cast<bf16x4_t*>(Sb + (size_t)i * N) = o;
    if (!REV && subset && i % m == 0) *reinterpret_cast<bf16x4_t*>(subset + sub0 + (size_t)(i / m) * N) = o;
  };
  auto ld = [&](int c) {  // product c, or zero when it does not exist
    return (c >= 0 && c < nchunks) ? *reinterpret_cast<const float4*>(Ub + (size_t)c * N) : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto add = [&](const float4& u) { acc.x += u.x; acc.y += u.y; acc.z += u.z; acc.w += u.w; };
  // States are walked in groups of GRP: the group's products are all requested before the first is added, so the
  // loads of a group are in flight together (the additions keep their fixed order).  Groups of 4 | 8 | 16 products: 8 heads,
  // 224 states 67 | 54 | 47 us, 4 heads, 20 states 6.4 | 5.8 | 6.0 us, 32 heads, 28 states 15.0 | 14.9 | 15.5 us.
  constexpr int GRP = PER < 8 ? 8 / PER : 1;
  if (!REV) {
    if (!restart)
      for (int c = 0; c < head; ++c) add(ld(c));
    // state i is stored, then products head + PER*i .. + PER - 1 are added to reach state i + 1
    for (int i0 = 0; i0 < nst; i0 += GRP) {
      float4 u[GRP][PER];
#pragma unroll
      for (int j = 0; j < GRP; ++j)
#pragma unroll
        for (int r = 0; r < PER; ++r) u[j][r] = (i0 + j + 1 < nst && !(restart && (i0 + j + 1) % m == 0)) ? ld(head + PER * (i0 + j) + r) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int j = 0; j < GRP; ++j) {
        if (i0 + j < nst) put(i0 + j);
#pragma unroll
        for (int r = 0; r < PER; ++r) add(u[j][r]);
      }
    }
  } else {
    // state nst-1 = 0; state i = state i+1 + products PER*i .. PER*i + PER - 1 (descending order of addition)
    for (int i0 = nst - 1; i0 >= 0; i0 -= GRP) {
      float4 u[GRP][PER];
#pragma unroll
      for (int j = 0; j < GRP; ++j)
#pragma unroll
        for (int r = 0; r < PER; ++r) u[j][r] = (i0 - j > 0) ? ld(PER * (i0 - j - 1) + r) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int j = 0; j < GRP; ++j) {
        if (i0 - j >= 0) put(i0 - j);
#pragma unroll
        for (int r = PER - 1; r >= 0; --r) add(u[j][r]);
      }
    }
  }
}

// Few products: products and scan in one launch.  A work-group holds all chunks of one (b, kv head) in LDS, for 32 value
// features, and keeps the running sum in registers.  The map is formed once for every 32 value features, so that a launch is
// saved only where there are few chunks (MAX_WALK, see rla_forward_states).  Each product is a sum of its own, added in order:
// the states are the bits that rla_chunk_kernel and rla_scan_kernel leave.
struct WalkArgs {
  const uint16_t *a, *b;   // rows that go through phi, rows multiplied in: [B,T,H,D]
  uint16_t* states;
  int H, T, B, head, nchunks, nst;   // product 0 covers 64 rows if head is 1; state i is the sum of products 0 .. head + i - 1
};
constexpr int MAX_WALK = 3;
constexpr int walk_bytes(int D) { return 128 * (2 * D + 64); }   // LDS of a chunk: rows of a, 32 features of b
// 512 threads; D/32 work-groups per (b, kv head).  Rows of 32 features of b need no swizzle (4 rows of 64 bytes are all banks).
// Wave w < D/32 owns features 32w .. of phi.
template <int D, int FM>
__global__ __launch_bounds__(512) void rla_walk_kernel(WalkArgs p) {
  typedef TileGeom<D> TG;
  constexpr int NS = D / 32, AT = 128 * TG::ROWB, CB = walk_bytes(D), NBLK = AT / 1024 / 8;
  extern __shared__ __align__(16) unsigned char chunks[];
  const int pair = blockIdx.x / NS, slice = blockIdx.x % NS, g = pair % p.H, b = pair / p.H;
  const int lane = lane_id(), w = wave_id(), r32 = lane & 31, h = lane >> 5;
  const size_t rstride = (size_t)p.H * D;
  const uint16_t* arow = p.a + ((size_t)b * p.T * p.H + g) * D;
  const uint16_t* brow = p.b + ((size_t)b * p.T * p.H + g) * D + 32 * slice;
  auto rows = [&](int c) { return c < p.head ? 64 : 128; };
  for (int c = 0; c < p.nchunks; ++c) {
    unsigned char* at = chunks + c * CB;
    const int lo = c < p.head ? 0 : 64 * p.head + 128 * (c - p.head), n = rows(c);
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
      const int blk = NBLK * w + i, r = blk * TG::RPB + lane / TG::CH;
      if (blk * TG::RPB < n)
        dma16(arow + (size_t)(lo + r) * rstride + (((lane % TG::CH) ^ swz<D>(r)) << 3), (unsigned)(size_t)RATTN_LDS(at + blk * 1024));
    }
    if (16 * w < n) dma16(brow + (size_t)(lo + 16 * w + lane / 4) * rstride + 8 * (lane % 4), (unsigned)(size_t)RATTN_LDS(at + AT + w * 1024));
  }
  int aoff[2], boff[2];
#pragma unroll
  for (int ab = 0; ab < 2; ++ab) {
    aoff[ab] = tr_lane_off<D>(8 * h + 4 * ab, w % NS, lane);
    boff[ab] = AT + (8 * h + 4 * ab + ((lane & 15) >> 2)) * 64 + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
  }
  uint16_t* out = p.states + (size_t)pair * p.nst * (D * D) + (size_t)(32 * slice + 4 * h) * D + 32 * w + r32;
  f32x16_t run = {0};
  auto put = [&](int i) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      out[(size_t)i * (D * D) + (size_t)(8 * (e >> 2) + (e & 3)) * D] = __builtin_bit_cast(uint16_t, (__bf16)run[e]);
  };
  wait_vmem();
  __syncthreads();
  // two threads per row, as in rla_chunk_kernel: the features are the same bits (each half of the threads takes every other chunk)
  for (int c = threadIdx.x >> 8; c < p.nchunks; c += 2) {
    const int row = (threadIdx.x & 255) >> 1;
    phi_row_inplace<FM, D, 2>(row < rows(c) ? chunks + c * CB : nullptr, row, threadIdx.x & 1);
  }
  __syncthreads();
  if (w >= NS) return;
  if (p.head == 0) put(0);
  for (int c = 0; c < p.nchunks; ++c) {
    const unsigned char* at = chunks + c * CB;
    f32x16_t acc = {0};
    for (int ks = 0; ks < rows(c) / 16; ++ks)
      acc = mfma32(lds_tr2(at + boff[0] + 1024 * ks, at + boff[1] + 1024 * ks),
                   lds_tr2(at + aoff[0] + 16 * TG::ROWB * ks, at + aoff[1] + 16 * TG::ROWB * ks), acc);
    run += acc;
    if (c + 1 >= p.head) put(c + 1 - p.head);
  }
}

template <int D, int FM> void launch_walk_kernel(const WalkArgs& p, hipStream_t st) {
  static const bool attr = hipFuncSetAttribute(reinterpret_cast<const void*>(rla_walk_kernel<D, FM>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, MAX_WALK * walk_bytes(D)) == hipSuccess;
  (void)attr;
  rla_walk_kernel<D, FM><<<D / 32 * p.H * p.B, 512, p.nchunks * walk_bytes(D), st>>>(p);
}
template <int D> void launch_walk(int phi, const WalkArgs& p, hipStream_t st) {
  switch (phi) {
    case PHI_RELU: launch_walk_kernel<D, FM_RELU>(p, st); break;
    case PHI_IDENTITY: launch_walk_kernel<D, FM_IDENTITY>(p, st); break;
    default: launch_walk_kernel<D, FM_SOFTMAX>(p, st); break;
  }
}

template <int D> void launch_chunk_kernel(int phi, dim3 grid, const ChunkArgs& p, hipStream_t st) {
  switch (phi) {
    case PHI_RELU: rla_chunk_kernel<D, FM_RELU><<<grid, 256, 0, st>>>(p); break;
    case PHI_IDENTITY: rla_chunk_kernel<D, FM_IDENTITY><<<grid, 256, 0, st>>>(p); break;
    default: rla_chunk_kernel<D, FM_SOFTMAX><<<grid, 256, 0, st>>>(p); break;
  }
}

// layers (in z) of the reverse scan's grid that sum gain gradients
int dgamma_layers(const LayerDims& dm, const DgammaSum& dg) {
  const int slice = dm.D * dm.D / 1024 * dm.Hkv;
  return dg.part ? (dg.tiles() + slice - 1) / slice : 0;
}

// per: products that a state spans
template <int D, bool REV>
void launch_scan_kernel(const LayerDims& dm, int per, const float* U, void* states, int nchunks, int nst, int head,
                        void* subset, const void* restart, int m, hipStream_t st,
                        const DgammaSum& dg = DgammaSum{}) {
  const dim3 grid(D * D / 1024, dm.Hkv, dm.B + dgamma_layers(dm, dg));
#define RATTN_SCAN(PER_)                                                                                                \
  rla_scan_kernel<D, REV, PER_><<<grid, 256, 0, st>>>(U, (uint16_t*)states, nchunks, nst, head, (uint16_t*)subset, \
                                                      (const uint16_t*)restart, m, dm.B, dg)
  if (REV && per == 8) RATTN_SCAN(REV ? 8 : 2);
  else if (REV && per == 6) RATTN_SCAN(REV ? 6 : 2);
  else if (REV && per == 4) RATTN_SCAN(REV ? 4 : 2);
  else if (REV && per == 3) RATTN_SCAN(REV ? 3 : 2);
  else if (per == 2) RATTN_SCAN(2);
  else RATTN_SCAN(1);
#undef RATTN_SCAN
}

}  // namespace

void rla_forward_states(const LayerDims& dm, const FastFwdPlan& pl, const SeqTensors& t, float* U, void* states,
                        hipStream_t st, void* subset_out, const void* restart, int m) {
  if (pl.nstf <= 0) return;
  if (m < 2) { m = 1; subset_out = nullptr; restart = nullptr; }
  const int head = pl.base > 0 ? 1 : 0;  // products in front of state 0: the 64 keys before it when it sits at key 64
  // Forward without saving in us, two launches | one: one product, 8 pairs of batch and kv head 28.2 | 23.4, 128 pairs 74.4 | 65.1;
  // two, 8 pairs 26.0 | 23.0, 64 pairs 37.4 | 34.1; three, 8 pairs 39.2 | 37.3 (D = 64 24.2 | 22.6), 64 pairs 49.2 | 47.8, 128 pairs
  // 123.4 | 125.8, where the work-groups no longer have a CU each
  if (m == 1 && t.P == 0 && pl.ckeys == 128 && pl.nchunks <= (dm.Hkv * (long long)dm.B <= 64 ? 3 : 2)) {
    const WalkArgs p = {(const uint16_t*)t.k, (const uint16_t*)t.v, (uint16_t*)states, dm.Hkv, t.Tb, dm.B, head, pl.nchunks, pl.nstf};
    ProfScope ps("rla_walk_kernel", st);
    if (dm.D == 64) launch_walk<64>(dm.phi, p, st); else launch_walk<128>(dm.phi, p, st);
    return;
  }
  if (pl.nchunks > 0) {
    ChunkArgs p;
    p.a = {(const uint16_t*)t.k_front, (const uint16_t*)t.k, t.P, t.Tb};
    p.b = {(const uint16_t*)t.v_front, (const uint16_t*)t.v, t.P, t.Tb};
    p.U = U;
    p.H = dm.Hkv; p.GA = p.GS = 1; p.tok_off = 0;
    p.ckeys = pl.ckeys;
    p.first_lo = 0; p.first_n = head ? 64 : pl.ckeys; p.rest_lo = p.first_n; p.tok_end = 1 << 30;
    p.skip_m = restart ? m : 0; p.skip_head = head; p.skip_per = 128 / pl.ckeys;
    ProfScope ps("rla_chunk_kernel", st);
    const dim3 grid(pl.nchunks, dm.Hkv, dm.B);
    if (dm.D == 64) launch_chunk_kernel<64>(dm.phi, grid, p, st); else launch_chunk_kernel<128>(dm.phi, grid, p, st);
  }
  ProfScope ps("rla_scan_kernel", st);
  if (dm.D == 64) launch_scan_kernel<64, false>(dm, 128 / pl.ckeys, U, states, pl.nchunks, pl.nstf, head, subset_out, restart, m, st);
  else launch_scan_kernel<128, false>(dm, 128 / pl.ckeys, U, states, pl.nchunks, pl.nstf, head, subset_out, restart, m, st);
}

void rla_reverse_states(const LayerDims& dm, const FastBwdPlan& pl, const void* q, int Tb, const void* dxr, float* U,
                        void* rstates, hipStream_t st, const DgammaSum& dg) {
  if (pl.nk <= 0) {
    if (dg.part) dgamma_reduce(dg, st);
    return;
  }
  const int W = pl.fwd.W, Tp = dm.T - W, ck = pl.fwd.ckeys;
  if (pl.nrchunks > 0) {
    ChunkArgs p;
    p.a = {nullptr, (const uint16_t*)q, 0, Tb};
    p.b = {nullptr, (const uint16_t*)dxr, 0, dm.T};   // a workspace tensor of the padded length
    p.U = U;
    p.H = dm.Hq; p.GA = dm.G; p.GS = pl.rsplit; p.tok_off = W;
    p.ckeys = ck;
    p.first_lo = 128; p.first_n = ck; p.rest_lo = 128 + ck; p.tok_end = Tp;
    p.skip_m = 0; p.skip_head = 0; p.skip_per = 1;
    ProfScope ps("rla_chunk_kernel(rev)", st);
    const dim3 grid(pl.nrchunks * pl.rsplit, dm.Hkv, dm.B);
    if (dm.D == 64) launch_chunk_kernel<64>(dm.phi, grid, p, st); else launch_chunk_kernel<128>(dm.phi, grid, p, st);
  }
  DgammaSum in_scan = dg;
  if (dm.B + dgamma_layers(dm, dg) > 65535) {   // a grid has no more layers than that
    dgamma_reduce(dg, st);
    in_scan.part = nullptr;
  }
  ProfScope ps("rla_scan_kernel(rev)", st);
  const int per = 128 / ck * pl.rsplit, n = pl.nrchunks * pl.rsplit;
  if (dm.D == 64) launch_scan_kernel<64, true>(dm, per, U, rstates, n, pl.nk, 0, nullptr, nullptr, 1, st, in_scan);
  else launch_scan_kernel<128, true>(dm, per, U, rstates, n, pl.nk, 0, nullptr, nullptr, 1, st, in_scan);
}

}  // namespace rattn
