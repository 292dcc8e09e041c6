// Decode step of the RAttention layer: one new token per sequence with constant memory
// (Sec. 2.1: cache of the last W keys;  Sec. 2.2: fixed D x D state;  Eq. 4: the linear branch reads
// the state lagging W tokens behind).  Memory bound: per (sequence, kv head) the kernel streams the
// K and V rings once (all query heads of the group share that read) and reads-modifies-writes the
// fp32 state once, with 16-byte-per-lane loads.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include <type_traits>

namespace rattn {

namespace {

__device__ __forceinline__ f32x4_t mfma16_f32(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Memory behind a buffer resource: accesses past its `bytes` touch nothing (reads return zero), so the last set of a ring
// needs no per-row address selection, and a lane's address is one 32-bit offset.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
// Keeps the compiler from reasoning about a per-lane value: offsets built from it stay one register plus an immediate,
// and what is computed from it inside a loop is not hoisted out of it into registers.
__device__ __forceinline__ int opaque(int x) { asm volatile("" : "+v"(x)); return x; }
// ONCE: marked non-temporal
template <typename V, bool ONCE = false> __device__ __forceinline__ V buf_load(rsrc_t r, int off) {
  if constexpr (sizeof(V) == 16) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, ONCE ? 2 : 0));
  else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, ONCE ? 2 : 0));
}
__device__ __forceinline__ void buf_store(rsrc_t r, f32x4_t v, int off) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), r, off, 0, 0);
}

// A set of ring rows as one wave holds it (lane = 16*q4 + r16), for the two window contractions on 16 x 16 matrix-core
// tiles whose columns are the query heads of the group:
//   S^T[key][head] = K Q^T : A rows are keys, read straight from the ring in operand layout (lane = key row r16, a
//       16-byte piece of its features per lane group q4; the feature order of the contraction is free as long as the q
//       operand follows it).  The result has key 16c + 4*q4 + i of head r16 in register i of tile c.
//   O^T[d][head] = V^T P^T : the probabilities stay in the registers the first product left them in; as a B operand
//       they pin which keys contraction slot (q4, .) stands for, and lane group q4 loads the V rows of exactly those
//       keys, lane r16 taking the r16-th piece (EV features) of each row.
// bf16: 32 keys, 16x16x32 tiles; fp32: 16 keys, 16x16x4 tiles (exact fp32 products and sums).
template <typename IO, int D, bool ONCE> struct RingSet;

template <int D, bool ONCE> struct RingSet<bf16_t, D, ONCE> {
  static constexpr int KEYS = 32, EV = D / 16;
  typedef uint32_t vrow_t __attribute__((ext_vector_type(EV / 2)));
  bf16x8_t k[2][D / 32];
  vrow_t v[8];
  __device__ __forceinline__ void load_k(rsrc_t rows, int r16, int q4) {
    const int off = opaque(2 * D * r16 + 16 * q4);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int offc = c ? opaque(off + 32 * D) : off;
#pragma unroll
      for (int j = 0; j < D / 32; ++j) k[c][j] = buf_load<bf16x8_t, ONCE>(rows, offc + 64 * j);
    }
  }
  __device__ __forceinline__ void load_v(rsrc_t rows, int r16, int q4) {
    const int off = opaque(8 * D * q4 + 2 * EV * r16), off1 = opaque(off + 32 * D);
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = buf_load<vrow_t, ONCE>(rows, (u < 4 ? off : off1) + 2 * D * (u & 3));
  }
  // q: this lane's head in LDS
  __device__ __forceinline__ void scores(const bf16_t* q, int q4, f32x4_t (&s)[2]) const {
    s[0] = s[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < D / 32; ++j) {
      const bf16x8_t op = *reinterpret_cast<const bf16x8_t*>(q + 32 * j + 8 * q4);
#pragma unroll
      for (int c = 0; c < 2; ++c) s[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[c][j], op, s[c], 0, 0, 0);
    }
  }
  static __device__ __forceinline__ float pexp(float x, float m) { return fast_exp2(x - m); }
  // acc[e] += V^T P^T for feature EV*r16 + e of each lane's piece; two rows are interleaved per dword with v_perm_b32.  The
  // fp32 probabilities pass through the bf16 tiles as three terms of 8 bits whose products share one accumulator, which is
  // as good as fp32 products with the bf16 values (one term: 1.12 - 1.16 times the error of the output against fp64,
  // which is mostly the output's own rounding).  The extra products hide behind the rings: 24 x 8 KV heads, W = 2048, 39.9 us
  // either way; one sequence, where they are part of the chain, 11.2 us against 10.8.
  __device__ __forceinline__ void accumulate(const f32x4_t (&p)[2], f32x4_t (&acc)[EV]) const {
    constexpr int TERMS = 3;
    float r[8] = {p[0][0], p[0][1], p[0][2], p[0][3], p[1][0], p[1][1], p[1][2], p[1][3]};
    bf16x8_t pop[TERMS];
#pragma unroll
    for (int term = 0; term < TERMS; ++term) {
      float t[8];
      pop[term] = pack_bf16x8(r);
      unpack_bf16x8(pop[term], t);
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] -= t[i];  // exact
    }
#pragma unroll
    for (int e = 0; e < EV; ++e) {
      const int j = e >> 1;
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      u32x4_t a;
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = __builtin_amdgcn_perm(v[2 * i + 1][j], v[2 * i][j], sel);
#pragma unroll
      for (int term = TERMS - 1; term >= 0; --term)
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), pop[term], acc[e], 0, 0, 0);
    }
  }
  // feature held by element (e, i) of a lane's accumulators
  static __device__ __forceinline__ int feature0(int e4, int i, int q4) { return EV * (4 * q4 + i) + 4 * e4; }
};

template <int D, bool ONCE> struct RingSet<float, D, ONCE> {
  static constexpr int KEYS = 16, EV = D / 16;
  f32x4_t k[D / 16];
  f32x4_t v[4][D / 64];
  __device__ __forceinline__ void load_k(rsrc_t rows, int r16, int q4) {
    const int off = opaque(4 * D * r16 + 16 * q4);
#pragma unroll
    for (int j = 0; j < D / 16; ++j) k[j] = buf_load<f32x4_t, ONCE>(rows, off + 64 * j);
  }
  __device__ __forceinline__ void load_v(rsrc_t rows, int r16, int q4) {
    const int off = opaque(16 * D * q4 + 16 * r16);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hf = 0; hf < D / 64; ++hf) v[i][hf] = buf_load<f32x4_t, ONCE>(rows, off + 4 * D * i + 256 * hf);
  }
  // Short chains of products and a tree of sums: the rounding of the logits grows with the chain.  With all features in two
  // chains it was 2.1 times that of the sums of partial sums per lane before (error of o at logits of std 4: 5.5e-7, 2.7e-7).
  __device__ __forceinline__ void scores(const float* q, int q4, f32x4_t (&s)[1]) const {
    f32x4_t t[D / 16];
#pragma unroll
    for (int j = 0; j < D / 16; ++j) {
      const f32x4_t op = *reinterpret_cast<const f32x4_t*>(q + 16 * j + 4 * q4);
      f32x4_t u[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e & 1] = mfma16_f32(k[j][e], op[e], u[e & 1]);
      t[j] = u[0] + u[1];
    }
#pragma unroll
    for (int n = D / 32; n > 0; n >>= 1)
#pragma unroll
      for (int j = 0; j < n; ++j) t[j] += t[j + n];
    s[0] = t[0];
  }
  static __device__ __forceinline__ float pexp(float x, float m) { return expf(x - m); }
  __device__ __forceinline__ void accumulate(const f32x4_t (&p)[1], f32x4_t (&acc)[EV]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int hf = 0; hf < D / 64; ++hf)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * hf + e] = mfma16_f32(v[i][hf][e], p[0][i], acc[4 * hf + e]);
  }
  static __device__ __forceinline__ int feature0(int e4, int i, int q4) { return 64 * e4 + 4 * (4 * q4 + i); }
};

constexpr int DEC_HB = 16;  // query heads per pass over the rings (columns of a matrix-core tile)

// bytes of LDS for hb query heads at a time and nw waves: q (rows padded by 16 bytes: the lanes of a read sit on
// different heads), phi(q), phi(k_old), v_old, the new token's logits, and per wave (m, l) and the partial results of
// both branches
constexpr size_t decode_lds_bytes(int D, int esize, int hb, int nw) {
  return (size_t)hb * (D * esize + 16) + ((size_t)(hb + 2) * D + DEC_HB + (size_t)nw * DEC_HB * 2 + (size_t)2 * nw * hb * D) * 4;
}

// Where few (sequence, kv head) pairs have long rings, several work-groups share each (decode_split, with times): a CU takes in
// some 59 bytes a nanosecond, a hundredth of what the memory delivers.  Every work-group leaves the partial
// results of its share of ring and state rows in the workspace; the one that arrives last adds them up in order (no matter who
// that is), forms the output and puts the new token into its slot, from which everyone has taken the evicted one by then.
// Nobody waits for anybody.
// Arrivals are counted in a ticket per pair, nonce | count.  The workspace is not initialised: a ticket whose upper 56 bits are
// not this call's nonce counts as zero, and the last arrival clears it, so that a captured launch finds none of its own
// when it is replayed.  (A ticket that holds the nonce by accident, one in 2^56, is the one case that goes wrong.)
struct SplitArgs {
  float* part;                   // [pair][work-group][head][row]: window sums, state sums, maximum, sum of exponentials
  unsigned long long* ticket;    // [pair]
  unsigned long long nonce;      // low 8 bits zero
  int n, rows;                   // work-groups per pair, 2 .. DEC_MAX_SPLIT, and ring rows for each before there is another
  static constexpr __host__ __device__ int row(int D) { return 2 * D + 4; }
};
struct NoSplit {
  static constexpr float* part = nullptr;
  static constexpr unsigned long long *ticket = nullptr, nonce = 0;
  static constexpr int n = 1, rows = 1;
};
// Stores and loads of agent scope meet in memory, past the caches of an XCD.  So the order of a wave's own accesses is all
// that an arrival needs: its stores are complete (vmcnt) before its work-group is counted, and the last one's loads are issued
// after it was.  A release and an acquire of agent scope instead write back and drop the XCD's whole L2 for every
// work-group: 12.0 -> 22.8 us at 16 work-groups for each of 4 pairs, 24 -> 83 at 4 for 256, where this way takes 18.2 and 30.4.
__device__ __forceinline__ void put_shared(float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float get_shared(const float* p) { return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Called by the whole work-group after its put_shared; true in the one that arrives last, whose get_shared then see everyone's
__device__ __forceinline__ bool arrive_last(unsigned long long* ticket, unsigned long long nonce, int n) {
  __shared__ int last;
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  wait_vmem();  // this wave's stores are in memory
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (threadIdx.x == 0) {
    // A cleared ticket gets the nonce from whoever comes first, and one more arrival is counted, in one trip to memory
    unsigned long long old = 0, now;
    __hip_atomic_compare_exchange_strong(ticket, &old, nonce, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    now = __hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    // Added to something else: counted again by exchange (which fails only because another of the n arrivals came in between,
    // n rounds at most for each of its two kinds)
    if ((now & ~255ull) != nonce) {
      old = now;
      do now = (old & ~255ull) == nonce ? old + 1 : nonce + 1;
      while (!__hip_atomic_compare_exchange_strong(ticket, &old, now, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    last = (int)(now & 255) == n;
    if (last) __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return last != 0;
}

// Waves per SIMD the kernel is compiled for.  A set in flight and the accumulators take 96 registers, the sums of fp32 logits
// of 128 features some 32 more; the loop over several groups of query heads keeps more alive.
constexpr int decode_occ(int D, int esize, bool multi) { return multi || D * esize == 512 ? 2 : 4; }

// grid (Hkv, N), NW waves: one (sequence, kv head).  Every wave runs its own online softmax over its share of the ring
// (K and V of a set are requested together; in fp32 the next set's K already behind the first product), so
// W is not limited by LDS, and takes its share of the state rows; the waves' partial results meet in LDS once.  The
// new token is not read back from the ring: its slot is masked there and it enters the merge as a partial of its own.
// Bound: HBM.  NW is chosen so that the chip is full of waves (pick_decode).  Measured, rings and states cold in the
// caches: 128 sequences x 8 KV heads, 4 query heads each, W = 512: 64.5 us = 6.3 TB/s (84 with the rings kept in the caches, see
// pick_decode); 24 x 8, 5 heads, W = 2048, half of the rings partly filled: 39 us (271 us with the scores of all W keys in LDS and
// vector arithmetic for more than four heads); one sequence, 4 KV heads, W = 512: 11.2 us by one work-group per KV head (18 us
// with four waves of it), 8.9 shared.
// More than 16 query heads per KV head (MULTI) are served in several passes over the rings.
// SPLIT: nsplit work-groups share a (sequence, kv head), see SplitArgs.
// ONCE: the ring is read past the caches; of the kernel: rings of once_rows rows and more (see pick_decode).
template <typename IO, int D, int NW, bool MULTI, bool SPLIT, bool ONCE>
__device__ __forceinline__ void decode_group(
    const IO* __restrict__ q, const IO* __restrict__ k_new, const IO* __restrict__ v_new, const int32_t* __restrict__ pos,
    IO* __restrict__ k_ring, IO* __restrict__ v_ring, float* __restrict__ state, const float* __restrict__ gs,
    const float* __restrict__ gr, IO* __restrict__ o, DecodeDims dd,
    std::conditional_t<SPLIT, SplitArgs, NoSplit> split) {
  typedef RingSet<IO, D, ONCE> Set;
  constexpr int EPL = D / 64, EV = Set::EV, NT = Set::KEYS / 16, NH = D / 64, QS = D + 16 / (int)sizeof(IO);
  const int W = dd.W, G = dd.G, Hq = dd.Hq, Hkv = dd.Hkv;
  const int HBmax = min(G, DEC_HB);
  extern __shared__ __align__(16) float lds[];
  IO* qs = reinterpret_cast<IO*>(lds);  // [HBmax][QS]
  float* qf = reinterpret_cast<float*>(qs + HBmax * QS);  // [HBmax][D]
  float* kfo = qf + HBmax * D;          // [D]
  float* vo = kfo + D;                  // [D]
  float* lnew = vo + D;                 // [16]
  float* ml = lnew + DEC_HB;            // [NW][16][2]
  float* part_s = ml + NW * DEC_HB * 2; // [NW][HBmax][D]
  float* part_r = part_s + NW * HBmax * D;

  // SPLIT: the pairs' first work-groups come first, so that where they are the only ones with work all XCDs have some of it.  (Those of
  // a pair side by side: every n-th has work, on 8 / n XCDs.  64 pairs, W = 1024, 380 tokens 10.0 | 9.0 us, unshared 9.5.)
  const int g = blockIdx.x, sp = SPLIT ? blockIdx.y / dd.N : 0, n = SPLIT ? blockIdx.y % dd.N : blockIdx.y;
  const int lane = lane_id(), w = wave_id();
  const int r16 = lane & 15, q4 = lane >> 4;
  const int p = pos[n];
  const int slot = p % W;
  const bool evict = p >= W;
  const int nvalid = min(p, W);  // ring rows written by earlier steps (with a full ring, row `slot` is the evicted token)
  // A ring that is not full yet takes fewer work-groups, a short one a single one; the others leave at once.  (56 pairs, W = 589,
  // 177 - 281 tokens: 9.2 us with two, 8.7 with one.)
  const int nsplit = !SPLIT || nvalid <= 3 * split.rows ? 1 : min(split.n, (nvalid - 1) / split.rows + 1);
  if (SPLIT && sp >= nsplit) return;
  const int w0 = SPLIT ? w * nsplit + sp : w, nw = SPLIT ? NW * nsplit : NW;  // this wave among those of the (sequence, kv head)
  IO* kr = k_ring + (size_t)(n * Hkv + g) * W * D;
  IO* vr = v_ring + (size_t)(n * Hkv + g) * W * D;
  const IO* knr = k_new + (size_t)(n * Hkv + g) * D;
  const IO* vnr = v_new + (size_t)(n * Hkv + g) * D;
  float* S = state + (size_t)(n * Hkv + g) * D * D;
  const int nset = (nvalid + Set::KEYS - 1) / Set::KEYS;
  // Work-groups run in lockstep over rings that lie a multiple of W*D elements apart; starting each one at a different
  // set spreads the simultaneous requests over the memory channels.
  const int rot = (int)((n * Hkv + g) % (unsigned)max(nset, 1));
  auto set_base = [&](int it) { const int s = it + rot; return (s < nset ? s : s - nset) * Set::KEYS; };
  auto rows = [&](const IO* ring, int base) {
    return make_rsrc(ring + (size_t)base * D, (unsigned)(min(Set::KEYS, nvalid - base) * D * (int)sizeof(IO)));
  };
  // logits in log2 units for bf16, natural for fp32 (see pexp)
  const float sc = sizeof(IO) == 2 ? dd.scale * LOG2E : dd.scale;

  int hb = 0;
  do {
    const int nh = MULTI ? min(DEC_HB, G - hb) : G;
    const size_t q0 = (size_t)(n * Hq + g * G + hb) * D;
    const bool upd = evict && hb == 0;
    Set set;
    // ---- phi(q), the new token's logits and (first pass) phi(k_old), v_old of the token leaving the window; item i of
    // nh + 1 is wave i's, and its rows are requested ahead of the ring (requests complete in order)
    const int nitem = nh + (hb == 0 ? 1 : 0);
    IO xr_[EPL], yr_[EPL];
    auto load_item = [&](int item) {
      const IO* xp = item < nh ? q + q0 + (size_t)item * D : kr + (size_t)slot * D;
      const IO* yp = item < nh ? knr : vr + (size_t)slot * D;
#pragma unroll
      for (int e = 0; e < EPL; ++e) { xr_[e] = xp[lane + 64 * e]; yr_[e] = yp[lane + 64 * e]; }
    };
    auto stage_item = [&](int item) {
      float x[EPL], y[EPL], ex[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) { x[e] = io_traits<IO>::ld(&xr_[e]); y[e] = io_traits<IO>::ld(&yr_[e]); }
      feature_row<EPL>(x, ex, dd.phi);
      if (item < nh) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          dot += x[e] * y[e];
          qs[item * QS + lane + 64 * e] = xr_[e];
          qf[item * D + lane + 64 * e] = ex[e];
        }
        dot = wave_sum(dot);
        if (lane == 0) lnew[item] = dot * sc;
      } else {
#pragma unroll
        for (int e = 0; e < EPL; ++e) { kfo[lane + 64 * e] = ex[e]; vo[lane + 64 * e] = y[e]; }
      }
    };
    auto wanted = [&](int item) { return item < nh || (item < nitem && evict); };
    if (wanted(w)) load_item(w);
    if (w0 < nset) {
      set.load_k(rows(kr, set_base(w0)), r16, q4);
      set.load_v(rows(vr, set_base(w0)), r16, q4);
    }
    if (wanted(w)) stage_item(w);
    for (int item = w + NW; item < nitem; item += NW)
      if (wanted(item)) { load_item(item); stage_item(item); }
    __syncthreads();
    // ---- the new token takes the slot of the evicted one (whose content now sits in LDS; SPLIT: in everyone's, see below)
    auto put_new = [&]() {
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        kr[(size_t)slot * D + lane + 64 * e] = knr[lane + 64 * e];
        vr[(size_t)slot * D + lane + 64 * e] = vnr[lane + 64 * e];
      }
    };
    if (nsplit == 1 && hb == 0 && w == NW - 1) put_new();
    // ---- softmax branch
    auto window_branch = [&]() {
      f32x4_t acc[EV];
#pragma unroll
      for (int e = 0; e < EV; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      float m = -1.0e30f, l = 0.f;
      const int qoff = min(r16, nh - 1) * QS;  // columns >= nh are never read back
      for (int it = w0; it < nset;) {
        const int base = set_base(it);
        it += nw;
        const int next = it < nset ? set_base(it) : 0;
        f32x4_t s[NT];
        set.scores(qs + opaque(qoff), q4, s);
        // fp32: the next set's K arrives behind the softmax and the second product; bf16: its registers hold the operands of
        // the second product there
        if (sizeof(IO) == 4 && it < nset) set.load_k(rows(kr, next), r16, q4);
#pragma unroll
        for (int c = 0; c < NT; ++c) s[c] *= sc;
        if (base + Set::KEYS > nvalid || (unsigned)(slot - base) < (unsigned)Set::KEYS) {  // wave-uniform
          const int key0 = opaque(base + 4 * q4);
#pragma unroll
          for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              s[c][i] = key0 + 16 * c + i < nvalid && key0 + 16 * c + i != slot ? s[c][i] : -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[c][i]);
        const float m_new = fmaxf(m, rows_max(mx));
        const float alpha = Set::pexp(m, m_new);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) { s[c][i] = Set::pexp(s[c][i], m); l += s[c][i]; }
#pragma unroll
        for (int e = 0; e < EV; ++e) acc[e] *= alpha;
        set.accumulate(s, acc);
        if (it >= nset) break;  // (not a condition on the loads: the old rows would stay alive across the products)
        if (sizeof(IO) == 2) set.load_k(rows(kr, next), r16, q4);
        set.load_v(rows(vr, next), r16, q4);
      }
      l = rows_sum(l);
      if (r16 < nh) {
        if (q4 == 0) { ml[(w * DEC_HB + r16) * 2] = m; ml[(w * DEC_HB + r16) * 2 + 1] = l; }
#pragma unroll
        for (int e4 = 0; e4 < EV / 4; ++e4)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4_t*>(part_s + (w * HBmax + r16) * D + Set::feature0(e4, i, q4)) =
                f32x4_t{acc[4 * e4][i], acc[4 * e4 + 1][i], acc[4 * e4 + 2][i], acc[4 * e4 + 3][i]};
      }
    };
    // ---- linear branch: state += phi(k_old)^T v_old, X_r^T[d][head] = S^T phi(Q)^T in fp32, eight state rows (two per
    // lane group) at a time, in the V layout of the fp32 ring set
    auto linear_branch = [&]() {
      f32x4_t xr[4 * NH];
#pragma unroll
      for (int e = 0; e < 4 * NH; ++e) xr[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      f32x4_t vold[NH];
#pragma unroll
      for (int hf = 0; hf < NH; ++hf) vold[hf] = upd ? *reinterpret_cast<const f32x4_t*>(vo + 64 * hf + 4 * r16) : f32x4_t{0.f, 0.f, 0.f, 0.f};
      const float* qfh = qf + min(r16, nh - 1) * D;
      constexpr int NSTEP = D / 8, SPW = (NSTEP + NW - 1) / NW;
      // steps past the last one, and all stores of a state that is not updated, fall outside their resource
      const rsrc_t src = make_rsrc(S, D * D * 4), dst = make_rsrc(S, upd ? D * D * 4 : 0);
      const int off0 = opaque(4 * ((8 * w0 + 2 * q4) * D + 4 * r16));
      f32x4_t sv[SPW][2][NH];
#pragma unroll
      for (int j = 0; j < SPW; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int hf = 0; hf < NH; ++hf) sv[j][i][hf] = buf_load<f32x4_t>(src, off0 + 4 * (8 * nw * D * j + D * i + 64 * hf));
#pragma unroll
      for (int j = 0; j < SPW; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int f = min(8 * (w0 + nw * j), D - 8) + 2 * q4 + i;
          const float qv = qfh[f];
          const float kf = upd ? kfo[f] : 0.f;
#pragma unroll
          for (int hf = 0; hf < NH; ++hf) {
            const f32x4_t s = sv[j][i][hf] + kf * vold[hf];
            buf_store(dst, s, off0 + 4 * (8 * nw * D * j + D * i + 64 * hf));
            if ((!SPLIT && NSTEP % NW == 0) || w0 + nw * j < NSTEP) {
#pragma unroll
              for (int e = 0; e < 4; ++e) xr[4 * hf + e] = mfma16_f32(s[e], qv, xr[4 * hf + e]);
            }
          }
        }
      if (r16 < nh) {
#pragma unroll
        for (int hf = 0; hf < NH; ++hf)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4_t*>(part_r + (w * HBmax + r16) * D + 64 * hf + 4 * (4 * q4 + i)) =
                f32x4_t{xr[4 * hf][i], xr[4 * hf + 1][i], xr[4 * hf + 2][i], xr[4 * hf + 3][i]};
      }
    };
    window_branch();
    __builtin_amdgcn_sched_barrier(0);  // (the registers of one branch at a time)
    linear_branch();
    __syncthreads();
    // sums over the waves of this work-group for head hh, relative to the maximum M, on top of `own` times the values v:
    // exponentials in den, both branches' accumulators in a, c.  (Fused by name: of two products and a sum the compiler
    // fuses either one, and not the same one in every instantiation.)
    auto wave_sums = [&](int hh, float M, float own, const float (&v)[EPL], float& den, float (&a)[EPL], float (&c)[EPL]) {
      den = own;
#pragma unroll
      for (int r = 0; r < NW; ++r) {
        const float sw = Set::pexp(ml[(r * DEC_HB + hh) * 2], M);
        den = __builtin_fmaf(sw, ml[(r * DEC_HB + hh) * 2 + 1], den);
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const float x = part_s[(r * HBmax + hh) * D + lane + 64 * e], y = part_r[(r * HBmax + hh) * D + lane + 64 * e];
          if (r == 0) {
            a[e] = __builtin_fmaf(own, v[e], sw * x);
            c[e] = y;
          } else {
            a[e] = __builtin_fmaf(sw, x, a[e]);
            c[e] += y;
          }
        }
      }
    };
    auto wave_max_of = [&](int hh, float M) {
#pragma unroll
      for (int r = 0; r < NW; ++r) M = fmaxf(M, ml[(r * DEC_HB + hh) * 2]);
      return M;
    };
    const size_t grp = (size_t)n * Hkv + g;
    if (SPLIT && nsplit > 1) {
      for (int hh = w; hh < nh; hh += NW) {
        const float M = wave_max_of(hh, -1.0e30f);
        float a[EPL], c[EPL], den;
        const float none[EPL] = {};
        wave_sums(hh, M, 0.f, none, den, a, c);
        float* dst = split.part + ((grp * split.n + sp) * G + hh) * SplitArgs::row(D);
#pragma unroll
        for (int e = 0; e < EPL; ++e) { put_shared(dst + lane + 64 * e, a[e]); put_shared(dst + D + lane + 64 * e, c[e]); }
        if (lane == 0) { put_shared(dst + 2 * D, M); put_shared(dst + 2 * D + 1, den); }
      }
      if (!arrive_last(split.ticket + grp, split.nonce, nsplit)) return;
      if (w == NW - 1) put_new();  // every work-group has taken the evicted token out of the slot
    }
    // ---- the partial results, the new token's, and the combination (Sec. 3.2); one wave per head
    for (int hh = w; hh < nh; hh += NW) {
      const int h = g * G + hb + hh;
      float a[EPL], c[EPL], den, M;
      float vn[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) vn[e] = io_traits<IO>::ld(vnr + lane + 64 * e);
      if (SPLIT && nsplit > 1) {
        const float* src = split.part + (grp * split.n * G + hh) * SplitArgs::row(D);
        const size_t step = (size_t)G * SplitArgs::row(D);
        const float* mine = src + min(lane, nsplit - 1) * step + 2 * D;  // lane i: maximum and sum of work-group i
        const float Mi = get_shared(mine), Li = get_shared(mine + 1);
        float x[DEC_MAX_SPLIT][2 * EPL];
#pragma unroll
        for (int i = 0; i < DEC_MAX_SPLIT; ++i)
          if (i < nsplit) {
#pragma unroll
            for (int e = 0; e < 2 * EPL; ++e) x[i][e] = get_shared(src + i * step + lane + 64 * e);
          }
        M = fmaxf(lnew[hh], wave_max(Mi));
        const float own = Set::pexp(lnew[hh], M), sw = lane < nsplit ? Set::pexp(Mi, M) : 0.f;
        den = own + wave_sum(sw * Li);
#pragma unroll
        for (int e = 0; e < EPL; ++e) { a[e] = own * vn[e]; c[e] = 0.f; }
#pragma unroll
        for (int i = 0; i < DEC_MAX_SPLIT; ++i)
          if (i < nsplit) {
            const float wi = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sw), i));
#pragma unroll
            for (int e = 0; e < EPL; ++e) { a[e] += wi * x[i][e]; c[e] += x[i][EPL + e]; }
          }
      } else {
        M = wave_max_of(hh, lnew[hh]);
        wave_sums(hh, M, Set::pexp(lnew[hh], M), vn, den, a, c);
      }
      // The window branch read the slot, while it changed from the evicted row to the new one, at a probability of 0, and
      // 0 times an infinite or NaN value is not 0.  A feature that came out without a number is formed again, key by key
      // without the slot.  (Dropping the row inside the branch costs every call: 24 x 8 KV heads, W = 2048, 41.0 -> 42.1 us.)
      float z = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) z += a[e] * 0.f;
      if (evict && __any(z != 0.f)) {
        float again[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) again[e] = Set::pexp(lnew[hh], M) * vn[e];
        for (int s = 0; s < W; ++s) {
          if (s == slot) continue;
          float dot = 0.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e)
            dot += io_traits<IO>::ld(qs + hh * QS + lane + 64 * e) * io_traits<IO>::ld(kr + (size_t)s * D + lane + 64 * e);
          const float prob = Set::pexp(wave_sum(dot) * sc, M);
#pragma unroll
          for (int e = 0; e < EPL; ++e) again[e] += prob * io_traits<IO>::ld(vr + (size_t)s * D + lane + 64 * e);
        }
#pragma unroll
        for (int e = 0; e < EPL; ++e) a[e] = a[e] * 0.f == 0.f ? a[e] : again[e];
      }
      const float inv = 1.f / den;
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) { a[e] *= inv; s1 += a[e] * a[e]; s2 += c[e] * c[e]; }
      const float r1 = rsqrtf(wave_sum(s1) / D + dd.eps), r2 = rsqrtf(wave_sum(s2) / D + dd.eps);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const int d = lane + 64 * e;
        const float g1 = gs ? gs[h * D + d] : 1.f, g2 = gr ? gr[h * D + d] : 1.f;
        io_traits<IO>::st(o + (size_t)(n * Hq + h) * D + d, g1 * a[e] * r1 + g2 * c[e] * r2);
      }
    }
    hb += DEC_HB;
    if (MULTI && hb < G) __syncthreads();
  } while (MULTI && hb < G);
}

template <typename IO, int D, int NW, bool MULTI, bool SPLIT, bool ONCE>
__global__ __launch_bounds__(NW * 64, decode_occ(D, sizeof(IO), MULTI)) void decode_kernel(
    const IO* __restrict__ q, const IO* __restrict__ k_new, const IO* __restrict__ v_new, const int32_t* __restrict__ pos,
    IO* __restrict__ k_ring, IO* __restrict__ v_ring, float* __restrict__ state, const float* __restrict__ gs,
    const float* __restrict__ gr, IO* __restrict__ o, DecodeDims dd,
    std::conditional_t<SPLIT, SplitArgs, NoSplit> split) {
  // (whole bodies: a branch around the loads alone merges their registers, and 64 of them spill)
  if (ONCE && min(pos[blockIdx.y], dd.W) >= dd.once_rows)
    decode_group<IO, D, NW, MULTI, SPLIT, ONCE>(q, k_new, v_new, pos, k_ring, v_ring, state, gs, gr, o, dd, split);
  else
    decode_group<IO, D, NW, MULTI, SPLIT, false>(q, k_new, v_new, pos, k_ring, v_ring, state, gs, gr, o, dd, split);
}

struct DecodeTensors {
  const void *q, *k_new, *v_new;
  const int32_t* pos;
  void *k_ring, *v_ring;
  float* state;
  const float *gs, *gr;
  void* o;
};

template <typename IO, int D, int NW, bool MULTI, bool SPLIT, bool ONCE = false>
void launch_decode(const DecodeDims& dd, const DecodeTensors& t, std::conditional_t<SPLIT, SplitArgs, NoSplit> split, hipStream_t st) {
  const int hb = dd.G < DEC_HB ? dd.G : DEC_HB;
  const size_t bytes = decode_lds_bytes(D, sizeof(IO), hb, NW);
  static const bool attr = hipFuncSetAttribute(reinterpret_cast<const void*>(decode_kernel<IO, D, NW, MULTI, SPLIT, ONCE>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256) == hipSuccess;
  (void)attr;
  decode_kernel<IO, D, NW, MULTI, SPLIT, ONCE><<<dim3(dd.Hkv, dd.N * (SPLIT ? split.n : 1)), NW * 64, bytes, st>>>(
      (const IO*)t.q, (const IO*)t.k_new, (const IO*)t.v_new, t.pos, (IO*)t.k_ring, (IO*)t.v_ring, t.state, t.gs, t.gr,
      (IO*)t.o, dd, split);
}

// Waves per (sequence, kv head): the fewer work-groups there are for the 256 CUs, the more of the waves a CU can hold
// (4 SIMDs of decode_occ waves) each of them needs to keep its CU's share of the memory requests in flight.
template <typename IO, int D, bool MULTI>
void pick_decode(const DecodeDims& dd, const DecodeTensors& t, hipStream_t st) {
  if constexpr (!MULTI) {
    const DecodeSplit ds = decode_split(dd, sizeof(IO));
    if (dd.workspace && ds.n > 1) {
      const SplitArgs split = {(float*)((char*)dd.workspace + ds.part_off), (unsigned long long*)dd.workspace, dd.nonce, ds.n, ds.rows};
      launch_decode<IO, D, 8, false, true>(dd, t, split, st);
      return;
    }
  }
  const NoSplit none;
  constexpr int cap = decode_occ(D, sizeof(IO), MULTI) == 4 ? 16 : 8;
  const long long groups = (long long)dd.N * dd.Hkv;
  int nw = 4;
  while (nw < cap && groups * nw < 256 * cap) nw *= 2;
  while (nw > 4 && decode_lds_bytes(D, sizeof(IO), dd.G < DEC_HB ? dd.G : DEC_HB, nw) > 160 * 1024 - 256) nw /= 2;
  // Enough work-groups to be bound by the memory, and so much in one layer that the memory-side cache (256 MB) cannot hold two:
  // rings that are read once need no place there.  Three layers stepped in turn, us, as usual | non-temporal: 1024 pairs, W = 512
  // (336 MB) 84.0 | 64.5; 512, W = 512 (168 MB) 42.4 | 35.7, W = 384 (134 MB) 35.0 | 30.4; fp32, W = 256 44.7 | 36.6; D = 64,
  // W = 900 (126 MB) 27.0 | 24.5, W = 512 (75 MB) 15.0 | 16.6; 256, W = 512 (84 MB) 18.2 | 19.3.  (A single layer that is stepped
  // again and again has it in that cache up to some 300 MB: 168 MB 31.7 | 34.8, 268 MB 53.0 | 53.2, 403 MB 87.1 | 75.7.)
  // With fewer work-groups the two halves of a row of K, which come with two loads, are fetched twice: 192 pairs, W = 2048
  // 40.2 | 44.0, 128 38.4 | 41.1.
  // Rings that are not full yet count as far as they are filled, in the kernel: one that would make 128 MB if all were filled like
  // it is read past the caches.  Two layers, through the caches | past them | chosen: 344 pairs, D = 64, W = 2933, 543 - 573 tokens
  // (55 MB) 14.85 | 16.1 | 14.9; 256 pairs, fp32, W = 512, 100 - 300 tokens 15.8 | 17.3 | 16.1; full rings (1024 pairs, W = 512)
  // 76.9 | 64.2 | 64.6.
  const long long once_rows = ((128ll << 20) / groups - D * D * 4ll) / (2ll * D * (int)sizeof(IO));
  if (!MULTI && groups >= 256 && dd.W >= once_rows) {
    DecodeDims dim = dd;
    dim.once_rows = (int)(once_rows > 0 ? once_rows : 0);
    if (nw == 4) launch_decode<IO, D, 4, false, false, !MULTI>(dim, t, none, st);
    else if (nw == 8) launch_decode<IO, D, 8, false, false, !MULTI>(dim, t, none, st);
    else if constexpr (cap == 16) launch_decode<IO, D, 16, false, false, !MULTI>(dim, t, none, st);
    return;
  }
  if (nw == 4) launch_decode<IO, D, 4, MULTI, false>(dd, t, none, st);
  else if (nw == 8) launch_decode<IO, D, 8, MULTI, false>(dd, t, none, st);
  else if constexpr (cap == 16) launch_decode<IO, D, 16, false, false>(dd, t, none, st);
}

}  // namespace

void decode_step(const DecodeDims& dd, int dtype, const void* q, const void* k_new, const void* v_new,
                 const int32_t* pos, void* k_ring, void* v_ring, float* state, const float* gs, const float* gr,
                 void* o, hipStream_t st) {
  ProfScope ps("decode_kernel", st);
  const DecodeTensors t = {q, k_new, v_new, pos, k_ring, v_ring, state, gs, gr, o};
#define RATTN_DECODE(IO, DD)                            \
  do {                                                  \
    if (dd.G <= DEC_HB) pick_decode<IO, DD, false>(dd, t, st);  \
    else pick_decode<IO, DD, true>(dd, t, st);          \
  } while (0)
  if (dtype == 0) {
    if (dd.D == 64) RATTN_DECODE(float, 64); else RATTN_DECODE(float, 128);
  } else {
    if (dd.D == 64) RATTN_DECODE(bf16_t, 64); else RATTN_DECODE(bf16_t, 128);
  }
#undef RATTN_DECODE
}

}  // namespace rattn
