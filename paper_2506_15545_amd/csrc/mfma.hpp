// gfx950 matrix-core and LDS helpers shared by the MFMA kernels.
//
// v_mfma_f32_32x32x16_bf16 operand layout (wave of 64 lanes, lane = 32*h + r):
//   A (32 x 16): lane holds row r, contraction slots 8h..8h+7 (8 bf16 in 4 VGPRs)
//   B (16 x 32): lane holds column r, contraction slots 8h..8h+7
//   C (32 x 32): lane holds column r; register i (0..15) is row 8*(i/4) + 4h + i%4
// ds_read_b64_tr_b16 (16-lane groups): if source lane 4j+c of a group points at M[k0+j][n0+4c..+3],
//   lane i of the group receives M[k0+0..3][n0+i]: a 4(k) x 16(n) block of a row-major matrix is
//   delivered k-contiguous per lane, which is what an MFMA operand wants when memory is n-contiguous.
// Tiles in LDS are rows of D bf16 (D = 128 or 64: 16 or 8 chunks of 16 bytes); the chunk index is XOR-swizzled with
//   D = 128:  swz(row) = ((row & 3) << 2) | ((row >> 2) & 3)
//   D =  64:  swz(row) = ((row >> 1 & 1) << 2) | ((row >> 2) & 3)
// so that both access patterns are bank-conflict free without padding (64 banks of 4 bytes = 16 chunks; two D = 64
// rows share one sweep of the banks):
//   row reads (ds_read_b128, 16 lanes on 16 consecutive rows, same logical chunk): (row, swz) spread over all 16 chunks
//   tr reads  (ds_read_b64_tr_b16, 4 consecutive rows x 64 bytes per half-wave): the upper bits of swz (with D = 64,
//             together with the row's parity) differ between the 4 rows, so the four 64-byte pieces land in different
//             bank groups
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rattn {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

#define RATTN_LDS(p) ((__attribute__((address_space(3))) void*)(p))

template <int D> struct TileGeom {
  static constexpr int ROWB = 2 * D;          // bytes of a row
  static constexpr int CH = D / 8;            // 16-byte chunks of a row
  static constexpr int RPB = 1024 / ROWB;     // rows that one wave's direct-to-LDS load covers (a "block")
  static constexpr int KT = 64 * ROWB;        // bytes of a 64-row tile
  static constexpr int NB = 64 / RPB;         // blocks of a 64-row tile
  static constexpr int NV = D == 128 ? 4 : 2; // the swizzle of a block's rows depends on the block index modulo NV only
};
template <int D> __device__ __forceinline__ int swz(int row) {
  return D == 128 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

__device__ __forceinline__ f32x16_t mfma32(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// wait until every outstanding vector-memory operation of this wave (incl. direct-to-LDS loads) is done
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// 16 bytes per lane from global memory straight into LDS at lds_addr + 16*lane (lds_addr wave-uniform).
// Issued through inline assembly on purpose: the compiler then does not put its own conservative
// vmcnt waits in front of later LDS reads, so a tile prefetch really overlaps the math on the current
// tile; completion is awaited explicitly with wait_vmem() before the barrier that publishes the tile.
__device__ __forceinline__ void dma16(const void* g, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
}

// The same load with a wave-uniform base in scalar registers and a 32-bit per-lane byte offset: no per-lane 64-bit
// address arithmetic per load.
__device__ __forceinline__ void dma16s(const void* sbase, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds_addr)) : "memory", "m0");
}
// Asynchronously copy `NBLK` blocks from global memory into an LDS tile, direct to LDS (no VGPR staging).  Block index
// blk0 + i, lane l lands at tile + blk*1024 + l*16, i.e. row RPB*blk + l/CH, physical chunk l%CH; it fetches the logical
// chunk that the swizzle maps there.  Rows from `nrows` on are read as row nrows - 1 (nrows may be <= 0: a row of the
// same sequence further up).
constexpr int ALL_ROWS = 1 << 30;
template <int D, int NBLK>
__device__ __forceinline__ void tile_load_async(const uint16_t* gbase, size_t row_stride, unsigned char* tile,
                                                int blk0, int lane, int nrows = ALL_ROWS) {
  typedef TileGeom<D> G;
#pragma unroll
  for (int i = 0; i < NBLK; ++i) {
    const int blk = blk0 + i;
    const int r = blk * G::RPB + lane / G::CH;
    const int c = (lane % G::CH) ^ swz<D>(r);
    const uint16_t* g = gbase + (ptrdiff_t)(nrows == ALL_ROWS ? r : min(r, nrows - 1)) * (ptrdiff_t)row_stride + c * 8;
    dma16(g, (unsigned)(size_t)RATTN_LDS(tile + blk * 1024));
  }
}
// Per-lane byte offsets of that access pattern inside a block, one per value of (block % NV); computed once per kernel.
template <int D> struct DmaLane { unsigned off[TileGeom<D>::NV]; };
template <int D> __device__ __forceinline__ DmaLane<D> make_dma_lane(int lane, size_t row_stride_elems) {
  typedef TileGeom<D> G;
  DmaLane<D> d;
  const int lr = lane / G::CH, p = lane % G::CH;
#pragma unroll
  for (int i = 0; i < G::NV; ++i)
    d.off[i] = (unsigned)(lr * row_stride_elems * 2) + (unsigned)((p ^ swz<D>(i * G::RPB + lr)) << 4);
  return d;
}
// tile_load_async for NBLK consecutive blocks starting at blk0 (wave-uniform, a multiple of NV)
template <int D, int NBLK>
__device__ __forceinline__ void tile_load_async_s(const uint16_t* gbase, size_t row_stride, unsigned char* tile, int blk0,
                                                  const DmaLane<D>& dl) {
  typedef TileGeom<D> G;
#pragma unroll
  for (int i = 0; i < NBLK; ++i) {
    const int blk = blk0 + i;
    dma16s(gbase + (size_t)blk * G::RPB * row_stride, dl.off[i % G::NV], (unsigned)(size_t)RATTN_LDS(tile + blk * 1024));
  }
}
// A run of tile rows in global memory: `p` = its first row, `n` = rows that exist from there on (see split_rows).
// Whole tiles take the scalar-base loads, a tile that reaches past the last row the ones that clamp every row.
struct TileRows { const uint16_t* p; int n; };
template <int D, int NBLK>
__device__ __forceinline__ void tile_load_async_s(const TileRows& src, size_t row_stride, unsigned char* tile, int blk0,
                                                  const DmaLane<D>& dl, int lane) {
  if (src.n >= 64) tile_load_async_s<D, NBLK>(src.p, row_stride, tile, blk0, dl);
  else tile_load_async<D, NBLK>(src.p, row_stride, tile, blk0, lane, src.n);
}

// Per-lane LDS byte offsets, computed once per kernel so that the hot loops issue ds_read with a
// register offset plus an immediate (the XOR swizzle is not affine, the compiler cannot fold it).
template <int D> struct LaneOff {
  int row[D / 16];     // row read: logical chunk 2*c2 + h of row (lane % 32)
  int trp[D / 32][2];  // transposed read, contraction slots in accumulator order: rows 4h + 8*ab + (0..3), columns 32*ct + lane%32
};
template <int D> struct LaneOffN {
  int trn[D / 32][2];  // transposed read, natural contraction order: rows 8h + 4*ab + (0..3), columns 32*ct + lane%32
};
template <int D> __device__ __forceinline__ int tr_lane_off(int rl, int ct, int lane) {
  const int i = lane & 15, gi = lane >> 4;
  const int r = rl + (i >> 2);
  const int c = 4 * ct + 2 * (gi & 1) + ((i & 3) >> 1);
  return r * TileGeom<D>::ROWB + ((c ^ swz<D>(r)) << 4) + ((i & 1) << 3);
}
template <int D> __device__ __forceinline__ LaneOff<D> make_lane_off(int lane) {
  LaneOff<D> lo;
  const int r32 = lane & 31, h = lane >> 5;
#pragma unroll
  for (int c2 = 0; c2 < D / 16; ++c2) lo.row[c2] = r32 * TileGeom<D>::ROWB + (((2 * c2 + h) ^ swz<D>(r32)) << 4);
#pragma unroll
  for (int ct = 0; ct < D / 32; ++ct)
#pragma unroll
    for (int ab = 0; ab < 2; ++ab) lo.trp[ct][ab] = tr_lane_off<D>(4 * h + 8 * ab, ct, lane);
  return lo;
}
template <int D> __device__ __forceinline__ LaneOffN<D> make_lane_off_n(int lane) {
  LaneOffN<D> lo;
  const int h = lane >> 5;
#pragma unroll
  for (int ct = 0; ct < D / 32; ++ct)
#pragma unroll
    for (int ab = 0; ab < 2; ++ab) lo.trn[ct][ab] = tr_lane_off<D>(8 * h + 4 * ab, ct, lane);
  return lo;
}
// A/B operand = rows R0 + lane%32 of the tile (R0 % 16 == 0), elements 16*c2 + 8h .. +7
template <int D> __device__ __forceinline__ bf16x8_t lds_row(const unsigned char* tile, const LaneOff<D>& lo, int R0, int c2) {
  return *reinterpret_cast<const bf16x8_t*>(tile + lo.row[c2] + R0 * TileGeom<D>::ROWB);
}
__device__ __forceinline__ bf16x8_t lds_tr2(const unsigned char* pa, const unsigned char* pb) {
  s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(pa));
  s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(pb));
  union { struct { s16x4_t lo, hi; } s; bf16x8_t v; } u;
  u.s.lo = lo; u.s.hi = hi;
  return u.v;
}
// operand = columns 32*ct + lane%32 of the tile; slot e of half h is tile row K0 + 8(e/4) + 4h + e%4
// (the order in which a 32x32 accumulator holds its rows), K0 % 16 == 0
template <int D> __device__ __forceinline__ bf16x8_t lds_trp(const unsigned char* tile, const LaneOff<D>& lo, int K0, int ct) {
  return lds_tr2(tile + lo.trp[ct][0] + K0 * TileGeom<D>::ROWB, tile + lo.trp[ct][1] + K0 * TileGeom<D>::ROWB);
}
// same with natural order: slot e of half h is tile row K0 + 8h + e, K0 % 16 == 0
template <int D> __device__ __forceinline__ bf16x8_t lds_trn(const unsigned char* tile, const LaneOffN<D>& lo, int K0, int ct) {
  return lds_tr2(tile + lo.trn[ct][0] + K0 * TileGeom<D>::ROWB, tile + lo.trn[ct][1] + K0 * TileGeom<D>::ROWB);
}

__device__ __forceinline__ bf16x8_t pack_bf16x8(const float* x) {
  f32x8_t v = {x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]};
  return __builtin_convertvector(v, bf16x8_t);
}

__device__ __forceinline__ void unpack_bf16x8(bf16x8_t v, float* x) {
  f32x8_t f = __builtin_convertvector(v, f32x8_t);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = f[i];
}

// combine a value with the one held by lane ^ 32 (v_permlane32_swap: one VALU op, no LDS traffic)
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// largest of three, NaN operands ignored: one v_max3_f32 (fmaxf puts a quieting instruction in front of every operand that
// comes from a matrix instruction).  Not inline assembly: the compiler keeps the distance that a vector instruction needs from
// the matrix instruction whose result it reads for its own instructions only.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximumnum(a, __builtin_elementwise_maximumnum(b, c));
}
// 2^x on the transcendental unit (v_exp_f32): 2^-inf = 0, no denormal fix-up code
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Rows of one head of a sequence that lies in memory in two parts: rows 0 .. P-1 in `front` [B, P, H, D] (P a multiple of
// 128, 0 = no such part), the rows after them in `back` [B, Tb, H, D].  The kernels work on whole 128-row tiles of the
// length P + Tb rounded up; a tile (or 64-row half) lies in one part, and rows past the last one are read as the last row:
// what is computed for them is never stored, and nothing that is stored depends on them (the layer is causal; their dO is
// zero).
struct SeqRows {
  const uint16_t *front, *back;
  int P, Tb;
};
__device__ __forceinline__ TileRows split_rows(const SeqRows& s, int b, int row, int H, int h, int D) {
  TileRows t;
  if (row < s.P) {
    t.p = s.front + ((size_t)((size_t)b * s.P + row) * H + h) * D;
    t.n = s.P - row;
  } else {  // (a start past the last row gives n <= 0: the loads then reach back to the last row)
    t.p = s.back + ((ptrdiff_t)((size_t)b * s.Tb + (row - s.P)) * H + h) * D;
    t.n = s.Tb - (row - s.P);
  }
  return t;
}

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Feature map of the linear branch as a compile-time choice of the matrix-core kernels:
//   FM_SOFTMAX    softmax over the 128 features of a row (Sec. 3.1)
//   FM_RELU       max(x, 0) per feature, FM_IDENTITY  x itself (the ablation's maps, Sec. 4.5)
enum { FM_SOFTMAX = 0, FM_RELU = 1, FM_IDENTITY = 2 };

// phi of a row whose two halves sit in lanes l and l^32 (N = D/2 values each: x[8c + e] = feature 16c + 8h + e);
// result packed as N/8 MFMA operand registers in the same order.
template <int FM, int N>
__device__ __forceinline__ void phi_rows(float (&x)[N], bf16x8_t (&op)[N / 8]) {
  if (FM == FM_RELU) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = fmaxf(x[i], 0.f);
  } else if (FM == FM_SOFTMAX) {
    float m = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) m = fmaxf(m, x[i]);
    m = half_max(m);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) { x[i] = fast_exp2((x[i] - m) * LOG2E); s += x[i]; }
    s = half_sum(s);
    const float inv = 1.f / s;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] *= inv;
  }
#pragma unroll
  for (int c = 0; c < N / 8; ++c) op[c] = pack_bf16x8(&x[8 * c]);
}

// phi applied in place to rows of LDS tiles by groups of TPR neighbouring threads per row (2 or 4), thread `part` of the
// group on features D/TPR * part ..; `tile` null: nothing to do for this thread.  The caller synchronises around it.
template <int FM, int D, int TPR>
__device__ __forceinline__ void phi_row_inplace(unsigned char* tile, int row, int part) {
  if (FM == FM_IDENTITY || !tile) return;
  constexpr int N = D / TPR;
  float x[N];
  unsigned char* rp = tile + row * TileGeom<D>::ROWB;
  const int sw = swz<D>(row);
#pragma unroll
  for (int j = 0; j < N / 8; ++j)
    unpack_bf16x8(*reinterpret_cast<const bf16x8_t*>(rp + (((N / 8 * part + j) ^ sw) << 4)), &x[8 * j]);
  if (FM == FM_RELU) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = fmaxf(x[i], 0.f);
  } else {
    float m = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) m = fmaxf(m, x[i]);
    m = fmaxf(m, __shfl_xor(m, 1, 64));
    if (TPR == 4) m = fmaxf(m, __shfl_xor(m, 2, 64));
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) { x[i] = fast_exp2((x[i] - m) * LOG2E); s += x[i]; }
    s += __shfl_xor(s, 1, 64);
    if (TPR == 4) s += __shfl_xor(s, 2, 64);
    const float inv = 1.f / s;
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] *= inv;
  }
#pragma unroll
  for (int j = 0; j < N / 8; ++j)
    *reinterpret_cast<bf16x8_t*>(rp + (((N / 8 * part + j) ^ sw) << 4)) = pack_bf16x8(&x[8 * j]);
}
// 256 threads, two per row: thread pair r works on row r of tile A (r < 64) or row r-64 of tile B (r >= 64); a null tile
// pointer skips that half.  Tiles A and B contiguous = one 128-row tile.
template <int FM, int D>
__device__ __forceinline__ void phi_tiles_inplace(unsigned char* tileA, unsigned char* tileB) {
  const int r = threadIdx.x >> 1;
  phi_row_inplace<FM, D, 2>(r < 64 ? tileA : tileB, r & 63, threadIdx.x & 1);
}
// first `nrows` (64 or 128) rows of one contiguous tile
template <int FM, int D>
__device__ __forceinline__ void phi_tile_inplace(unsigned char* tile, int nrows) {
  phi_tiles_inplace<FM, D>(tile, nrows > 64 ? tile + TileGeom<D>::KT : nullptr);
}

// Write a [128 rows x D] bf16 tile held transposed in accumulators (lane = tile row 32w + lane%32,
// register (dt,i) = column 32dt + 8(i/4) + 4h + i%4) to global rows of stride `row_stride`, through
// LDS so that the global stores are 16 bytes per lane and row-contiguous; rows from `nrows` on are not written.
// All 256 threads call it; smem[0..128 rows) is used and is free again on return.
template <int D>
__device__ __forceinline__ void store_tile_transposed(unsigned char* smem, const float (&vals)[D / 32][16], uint16_t* dst,
                                                      size_t row_stride, int w, int lane, int nrows = 128) {
  typedef TileGeom<D> G;
  const int r32 = lane & 31, h = lane >> 5;
  const int row = 32 * w + r32;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      f32x4_t f = {vals[dt][4 * i4], vals[dt][4 * i4 + 1], vals[dt][4 * i4 + 2], vals[dt][4 * i4 + 3]};
      bf16x4_t pk = __builtin_convertvector(f, bf16x4_t);
      const int c = 4 * dt + i4;
      *reinterpret_cast<bf16x4_t*>(smem + row * G::ROWB + ((c ^ swz<D>(row)) << 4) + 8 * h) = pk;
    }
  __syncthreads();
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 128 * G::CH / 256; ++i) {
    const int id = tid + 256 * i;
    const int r = id / G::CH, p = id % G::CH;
    const int c = p ^ swz<D>(r);
    const u32x4_t val = *reinterpret_cast<const u32x4_t*>(smem + r * G::ROWB + (p << 4));
    // written once, not read again by the kernel that writes it: keep it from displacing the shared K/V tiles in L2
    if (r < nrows) __builtin_nontemporal_store(val, reinterpret_cast<u32x4_t*>(dst + (size_t)r * row_stride + c * 8));
  }
  __syncthreads();
}

}  // namespace rattn
