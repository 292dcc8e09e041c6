// Shape planning shared by the C ABI and the kernel launchers: which shapes the matrix-core kernels take, how many
// chunk states a call needs and how large its scratch areas are.  Host arithmetic only (nothing here touches a
// device), so this file is also part of the CPU build of the host layer that runs under the sanitizers.
#include "kernels.hpp"

namespace rattn {

// dm: the dimensions the kernels would see, i.e. with the sequence length rounded up to whole tiles
bool fast_fwd_supported(const LayerDims& dm, int dtype) {
  if (dtype != 1 || dm.T % 128 != 0) return false;
  if (!(dm.scale > 0.f)) return false;
  // Windows below 8 keys stay on the general path: their softmax rows are close to one-hot, so the backward's
  // dS = P (dP - delta) is a near-cancellation (exact for W = 1) that bf16 operands turn into rounding noise
  // above the gradient tolerance (measured: worst element 4 % of RMS at W = 2, 3 % at W = 4, 2.5 % from W = 8 on)
  if (dm.W < 8) return false;
  return true;
}

int generic_chunk(const LayerDims& dm, int Tp) {
  const long long groups = (long long)((dm.T + 15) / 16) * dm.Hq * dm.B;
  return Tp > 64 && Tp <= (groups <= 256 ? 320 : groups <= 512 ? 224 : 128) ? Tp : 64;
}

FastFwdPlan fast_fwd_plan(const LayerDims& dm) {
  FastFwdPlan p;
  const int wt = dm.W >= dm.T ? dm.T : dm.W;
  p.W = (wt + 63) / 64 * 64;
  p.gap = p.W - wt;
  p.base = p.W % 128;
  p.nstf = dm.T / 128 - (p.W + 127) / 128;
  if (p.nstf < 0) p.nstf = 0;
  // chunk-local products of `ckeys` keys each (128 unless the caller asks for `chunk` = 64); with 128 and states at the 64
  // alignment the first product covers the 64 keys in front of state 0
  p.ckeys = dm.chunk_req == 64 ? 64 : 128;
  p.nchunks = p.nstf > 0 ? (p.nstf - 1) * (128 / p.ckeys) + (p.base > 0 ? 1 : 0) : 0;
  p.u_bytes = (size_t)dm.B * dm.Hkv * p.nchunks * dm.D * dm.D * 4;
  p.state_bytes = (size_t)dm.B * dm.Hkv * p.nstf * dm.D * dm.D * 2;
  return p;
}

ChunkPlan chunk_plan(const LayerDims& dm, int P, int R, int Tc) {
  ChunkPlan c = {0, 0, 0, 0, 0, 0};
  const FastFwdPlan pl = fast_fwd_plan(dm);
  const long long bg = (long long)dm.B * dm.Hkv;
  c.end = P + Tc - dm.W;
  // Every call whose forward reads states that hold a key shares its products; with a carried state every call does.  (One
  // sequence of one KV head, 128 new tokens, ring of 128: separate launches 30.1 us, shared 26.2.)
  if (pl.nstf <= 0 || R + Tc <= dm.W) return c;
  c.head = pl.base > 0 ? 1 : 0;
  // (the last state is in front of the last row that leaves the window: at least one product follows it)
  const int rest = c.end - 64 * c.head, n = (rest + 127) / 128;
  // Products of 64 rows where those of 128 leave half of the chip idle, as long as the scan's chain stays short: 32/8 heads,
  // W = 512, products of 64 | 128 rows: 700 tokens 41.2 | 41.9 us, 1024 41.4 | 42.7, 1500 50.6 | 52.3, two sequences of 1500
  // 74.9 | 71.9; 16/2 heads, 2048 tokens (16 products of 128 rows in a chain) 41.8 | 40.8.
  c.ckeys = dm.chunk_req == 64 || (n <= 12 && n * bg <= 128) ? 64 : 128;
  c.nprod = c.head + (rest + c.ckeys - 1) / c.ckeys;
  // Chains of 64 keys as in the prefill export, of 128 where that has more tiles than two work-groups per CU (export_plan): another
  // 64 registers and additions, 4 x 2048 tokens after 2048, 8 KV heads 134.6 -> 137.8 us
  c.piece = (R + Tc - dm.W + 63) / 64 * bg > 512 ? c.ckeys : 64;
  c.u_bytes = (size_t)bg * c.nprod * dm.D * dm.D * 4;
  return c;
}

FastBwdPlan fast_bwd_plan(const LayerDims& dm) {
  FastBwdPlan p;
  p.fwd = fast_fwd_plan(dm);
  const int Tp = dm.T - p.fwd.W;
  p.nk = Tp > 0 ? (Tp + 127) / 128 : 0;
  // reverse-time chunk products: query rows t' in [128, Tp) in pieces of ckeys
  p.nrchunks = Tp > 128 ? (Tp - 128 + p.fwd.ckeys - 1) / p.fwd.ckeys : 0;
  // A work-group visits the query heads of its product in turn; where there are few products the heads are split over two
  // or four work-groups, as long as those fit on the chip together (two per CU).  2 x 1000 tokens, 4 KV heads of 4 query
  // heads: 24 -> 96 work-groups, 19 -> 8.5 us.  Every further product is written, and read again in the scan's one chain of
  // additions per element.  So a doubling must take at least as many keys (heads x keys of a product) off the longest
  // work-group as it adds products, and eight times the products that it adds to a chain.  Backward at D = 128, one | two |
  // four work-groups: 64 products of 4 heads in chains of 8 96.6 | 90.2 | 89.7 us, of 16 97.1 | 91.2 | 92.4; 96 products of
  // 4 heads 102.6 | 97.7 | 99.3; 128 of 2 heads 82.5 | 81.1, of 3 98.6 | 98.8, of 8 in chains of 8 228.7 | 216.6 | 215.0, of
  // 32 224.8 | 215.4 | 217.1; 192 of 2 heads 88.7 | 89.6, of 3 124.9 | 127.0; 256 of 4 heads 228.6 | 226.5 | 243.7.
  const long long chains = (long long)dm.Hkv * dm.B;
  auto longest = [&](int s) { return (long long)((dm.G + s - 1) / s) * p.fwd.ckeys; };   // keys
  p.rsplit = 1;
  for (int s = 1; s < 4 && 2 * s <= dm.G && chains * p.nrchunks * 2 * s <= 512; s *= 2) {
    const long long added = (long long)p.nrchunks * s, fewer = longest(s) - longest(2 * s);
    if (chains * added > fewer || 8 * added > fewer) break;
    p.rsplit = 2 * s;
  }
  const int heads = (dm.G + p.rsplit - 1) / p.rsplit;
  p.rsplit = (dm.G + heads - 1) / heads;   // 5, 6 or 9 heads: the fourth work-group would have none
  const int nrev = p.nrchunks * p.rsplit, nch = p.fwd.nchunks > nrev ? p.fwd.nchunks : nrev;
  p.u_bytes = (size_t)dm.B * dm.Hkv * (nch > 0 ? nch : 0) * dm.D * dm.D * 4;
  p.rstate_bytes = (size_t)dm.B * dm.Hkv * p.nk * dm.D * dm.D * 2;
  p.RB = 4 * (dm.T / 128) * dm.B;  // one gain-gradient partial per wave of the dq kernel
  // The dk/dv kernel holds one work-group per CU (two at D = 64), which visits the G query heads of its key tile in turn.  With few key
  // tiles the heads are split over several work-groups (partial sums in fp32, added in order): the split with the fewest
  // head visits on the busiest CU, where a work-group costs about half a visit on top of its own.
  const long long tiles = (long long)(dm.T / 128) * dm.Hkv * dm.B, slots = dm.D == 64 ? 512 : 256;
  p.nsplit = 1;
  double best = 0.0;
  for (int s = 1; s <= dm.G; ++s) {
    const int hps = (dm.G + s - 1) / s, used = (dm.G + hps - 1) / hps;
    if (used != s) continue;   // the same heads per work-group with fewer of them
    const double cost = (double)((tiles * s + slots - 1) / slots) * (hps + 0.5) + (s > 1 ? 0.5 : 0.0);
    if (s == 1 || cost < best) { best = cost; p.nsplit = s; }
  }
  p.dkv_part_bytes = p.nsplit > 1 ? (size_t)2 * p.nsplit * dm.B * dm.T * dm.Hkv * dm.D * 4 : 0;
  return p;
}

DecodeSplit decode_split(const DecodeDims& dd, int esize) {
  // A work-group of eight waves for every 64 KB of rings, up to 128 of them in all: more are bound by what the memory delivers.
  // Captured steps in us, one work-group per pair (16 waves) | as split, bf16, D = 128, full rings:
  //   4 pairs, W = 512 11.1 | 9.0;  1024 14.5 | 9.5;  2048 23.4 | 10.8;  4096 41.0 | 12.1;  16, 512 11.2 | 9.3;  2048 23.6 | 11.7
  //   32, 512 10.9 | 9.5;  2048 24.7 | 13.4;  64, 512 12.1 | 11.4;  1024 16.1 | 14.3;  2048 25.7 | 19.6;  4096 44.2 | 29.5
  //   D = 64, 4 pairs, W = 1024 9.6 | 7.8;  4096 25.2 | 9.4;  fp32, 4 pairs, W = 512 17.9 | 10.6;  16 pairs, 4096 91.7 | 21.5
  // Rings that are not full, 100 tokens 7.3 | 6.9 (4 pairs), 7.5 | 7.1 (64);  380, one work-group of eight waves, 9.4 | 8.7, 9.5 | 9.0;
  // slower by up to 3 % remain D = 64, 4 pairs, 550 - 768 tokens 7.6 | 7.8 and fp32, 100 tokens 9.0 | 9.3.
  // How many were compared eagerly, when the host took 8 of each step and 9.5 with a workspace (now 3.6 and 3.9); one | 2 | 4 | 8 | 16:
  //   4 pairs, W = 512 12.0 | 10.7 | 9.5 | 9.5 | 10.3;  W = 2048 25.0 | 18.6 | 13.4 | 11.5 | 11.5;  W = 4096 42.8 | 29.0 | 18.6 | 13.7 | 12.7
  //   16 pairs, W = 1024 15.9 | 13.4 | 11.0 | 11.0 | 12.4;  64, W = 512 14.3 | 13.3 | 13.4 | 15.1 | 26.5
  //   128 pairs, W = 512 16.1 | 16.8 | 17.4;  W = 2048 38.1 | 34.1 | 34.2 | 39.4 (not taken: rings with 100 - 400 tokens
  //   10.7 | 11.6);  192, W = 2048 35.5 | 39.2 | 39.6
  //   32 pairs, D = 64, W = 512 7.8 | 9.9;  4 pairs, fp32, W = 512 18.5 | 15.4 | 12.6 | 11.2 | 11.8
  DecodeSplit s = {1, dd.W, 0, 0};
  const long long pairs = (long long)dd.N * dd.Hkv, ring = 2ll * dd.W * dd.D * esize;
  if (dd.G > 16 || ring < 256 << 10) return s;
  const int share = 64 << 10;
  s.n = DEC_MAX_SPLIT;
  while (s.n > 1 && (ring / s.n < share || pairs * s.n > 128)) s.n /= 2;
  if (s.n < 2) return s;
  s.rows = (int)(share * (long long)dd.W / ring);
  s.part_off = ((size_t)pairs * 8 + 255) / 256 * 256;
  s.bytes = s.part_off + (size_t)pairs * s.n * dd.G * (2 * dd.D + 4) * 4;
  return s;
}

ExportPlan export_plan(const LayerDims& dm) {
  ExportPlan pl;
  pl.Tp = dm.T > dm.W ? dm.T - dm.W : 0;
  // Segments of 64-key tiles, enough of them for two work-groups on every CU: more only add partial states to write
  // and read back (each as large as 128 keys and values of a bf16 head)
  const int tiles = (pl.Tp + 63) / 64, most = 512 / (dm.B * dm.Hkv) > 1 ? 512 / (dm.B * dm.Hkv) : 1;
  const int per = (tiles + most - 1) / most;
  pl.seg_len = 64 * per;
  pl.nseg = per > 0 ? (tiles + per - 1) / per : 0;
  pl.partial_bytes = (size_t)dm.B * dm.Hkv * pl.nseg * dm.D * dm.D * sizeof(float);
  return pl;
}

}  // namespace rattn
