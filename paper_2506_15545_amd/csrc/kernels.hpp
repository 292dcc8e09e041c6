// Host-side declarations shared by the C ABI (api.hip) and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rattn {

// per-kernel event timing (see rattn_profile_* in rattn.h); no-ops while profiling is off.  Scopes do not nest: an inner
// one leaves the outer one's record without its second event.
void prof_begin(const char* name, hipStream_t st);
void prof_end(hipStream_t st);
struct ProfScope {
  hipStream_t st;
  ProfScope(const char* name, hipStream_t s) : st(s) { prof_begin(name, s); }
  ~ProfScope() { prof_end(st); }
};

// feature map of the linear branch (values of rattn_feature_map)
enum { PHI_SOFTMAX = 0, PHI_RELU = 1, PHI_IDENTITY = 2 };

struct LayerDims {
  int B, T, Hq, Hkv, D, W, C, G;
  int chunk_req;  // the caller's `chunk` parameter as given (0 = unspecified); C above is what the general kernels use
  int nst;  // number of chunk states per (batch, kv head): ceil(max(T-W,0) / C)
  float scale, eps;
  int phi;  // feature map of the linear branch: PHI_SOFTMAX (Sec. 3.1), PHI_RELU, PHI_IDENTITY (Sec. 4.5 ablation)
};

// views into the opaque `saved` buffer: pre-norm branch outputs ([B,T,Hq,D]; the I/O dtype on the MFMA path, fp32
// on the general path: the backward through the second RMS norm projects the upstream gradient off x^r, and where
// the state has very low rank - the first rows past the window - rounding x^r to bf16 leaves an error that the
// state multiplies back up) and the
// row statistics (fp32, [B,Hq,T]): log-sum-exp of the softmax branch and the two RMS reciprocals, and the
// linear-branch chunk states (MFMA path: bf16, transposed; general path: fp32), where backward is not to rebuild them
struct SavedPtrs {
  void* xs;
  void* xr;
  float* lse;
  float* rs;
  float* rr;
  void* states;
  int state_stride;  // `states` holds every chunk state (0 or 1) or states 0, m, 2m, ... only (m = 2, 4): the
                     // forward then works on the full set in its workspace and backward rebuilds the states in
                     // between from the stored ones (Sec. 3.2: store every m-th state, recompute the others)
};

struct GenericBwdWs {
  float* rstates;  // [B,Hkv,nst,D,D]; the forward states first, where `saved` does not hold them
  float* dxs;      // [B,T,Hq,D]
  float* dxr;      // [B,T,Hq,D]
  float* delta;    // [B,Hq,T]
  float* dgpart;   // [2,RB,Hq,D], one gain-gradient partial per 16-row tile (RB = B ceil(T/16))
};

// Keys per chunk of the general kernels where the caller names none, Tp = the keys that leave some query's window.  Few
// enough of them form one chunk: no query sees a whole chunk then, so no states are formed (two launches less in each
// direction) and the consumers multiply out more pairs.  That is a question of idle compute units: forward + backward in
// us, fp32, D = 64, chunks of 64 | one chunk; work-groups of 16 query rows, Tp:
//   32, 224: 51.5 | 42.0;  50, 344: 55.2 | 55.4;  64, 384: 57.6 | 58.2;  200, 344: 66.6 | 67.2
//   384, 176: 66.8 | 54.6;  512, 224: 69.0 | 65.4;  672, 320: 86.1 | 104.9
//   2048, 112: 150 | 132;  3072, 176: 211 | 231;  4096, 224: 268 | 384
// (D = 128 alike: 32, 224: 87.9 | 72.6;  512, 224: 131 | 114;  3072, 176: 443 | 452.)
int generic_chunk(const LayerDims& dm, int Tp);

// Only rows q0 .. T-1 have queries (q, o and the saved tensors hold just those); `states` receives the chunk states
// (B*Hkv*nst*D*D floats; nothing where nst is 1); state0 (fp32 [B,Hkv,D,D], may be NULL): a linear-branch state that precedes key 0.
void generic_fwd(const LayerDims& dm, int dtype, const void* q, const void* k, const void* v, const float* gs,
                 const float* gr, void* o, const SavedPtrs& sv, float* states, hipStream_t st, int q0 = 0,
                 const float* state0 = nullptr);
// sv.states: the chunk states as the forward left them, or NULL: rebuilt from k and v
void generic_bwd(const LayerDims& dm, int dtype, const void* q, const void* k, const void* v, const float* gs,
                 const float* gr, const SavedPtrs& sv, const void* dO, void* dq, void* dk, void* dv, float* dgs,
                 float* dgr, const GenericBwdWs& ws, hipStream_t st);

// partial linear-branch states of key segments of fp32 k, v [B,T,Hkv,D], out[b][kv head][segment][feature][value]:
// segment c covers keys [c seg_len, (c+1) seg_len) below Tp
void generic_chunk_products(const LayerDims& dm, int T, const void* k, const void* v, float* out, int Tp, int nseg,
                            int seg_len, hipStream_t st);

// gain gradients [HD] from RB partials each, summed in a fixed order: part[2][RB][HD], HD a multiple of 32; either output
// may be NULL (part NULL: nothing to sum)
struct DgammaSum {
  const float* part;
  float *dgs, *dgr;
  int RB, HD;
  int tiles() const { return HD / 32 * 2; }   // work-groups
};
void dgamma_reduce(const DgammaSum& dg, hipStream_t st);

// Keys and values of the matrix-core kernels.  They work in 128-row tiles over a padded length (LayerDims::T); a sequence
// has P rows in `*_front` tensors [B,P,Hkv,D] (chunked prefill: the ring in time order behind zero rows that fill the
// first tile; P is a multiple of 128, else 0), then Tb rows in k, v [B,Tb,Hkv,D], and nothing after them.
struct ChunkHandover;
struct SeqTensors {
  const void *k, *v;
  int Tb;
  void *k_front = nullptr, *v_front = nullptr;
  int P = 0;
  int kmin = 0;   // keys in front of this row do not exist for the softmax branch
  const ChunkHandover* handover = nullptr;   // see there
};

// MFMA forward path (bf16, padded length T % 128 == 0, any W >= 8)
struct FastFwdPlan {
  int W;        // window the tiles and states are laid out for: min(W, T) rounded up to a multiple of 64
  int gap;      // that minus the true window (0..63): masks and the reach of the intra-chunk part
  int base;     // key position of state 0 (0 or 64); state i sits at base + 128*i
  int nstf;     // number of states per (batch, kv head) = query tiles that have a linear branch
  int ckeys;    // keys per chunk-local product (64 or 128): the chunk size C of Eqs. 2-3 on this path
  int nchunks;  // chunk-local products needed to build them
  size_t u_bytes, state_bytes;
};
bool fast_fwd_supported(const LayerDims& dm, int dtype);
FastFwdPlan fast_fwd_plan(const LayerDims& dm);

// Chunked prefill on the matrix cores: how the products of the forward's states and of the state that the call leaves are
// shared (see chunk_kernels.hip)
struct ChunkPlan {
  int nprod;   // products per (batch, kv head); 0: nothing to share
  int head;    // 1: product 0 covers the 64 rows in front of state 0
  int ckeys;   // rows of every other product (64 or 128)
  int piece;   // rows of a product that are summed for themselves (64, or ckeys)
  int end;     // row behind the last one that leaves the window
  size_t u_bytes;
};
// dm: padded, D = 128, softmax or ReLU map; P, R: front rows and how many of them are ring rows; Tc new rows
ChunkPlan chunk_plan(const LayerDims& dm, int P, int R, int Tc);
// Given to fast_fwd, which then also does what chunk_ring and prefill_export do: fills the front tensors from the rings,
// and leaves rings and state advanced by the chunk.  U of fast_fwd: plan.u_bytes.
struct ChunkHandover {
  ChunkPlan plan;
  void *k_ring, *v_ring;
  float* state;
  int R, pos0, carried;   // ring rows, position of the chunk's first row, whether `state` holds anything yet
};
void chunk_states(const LayerDims& dm, const SeqTensors& t, float* U, void* states, hipStream_t st);
// dm.T: the padded length.  The query tiles computed are those of the Tb rows behind the front part; q, o and the saved
// tensors hold just those rows ([B,Tb,Hq,D]; the saved tensors rounded up to whole tiles).
void fast_fwd(const LayerDims& dm, const SeqTensors& t, const void* q, const float* gs, const float* gr, void* o,
              const SavedPtrs& sv, float* U, void* states, hipStream_t st);

// linear-branch chunk states for the MFMA paths (bf16 [d][f] per state, fp32 scratch U per chunk)
// With m > 1: `subset_out` (forward) also receives states 0, m, 2m, ...; `restart` (backward) holds those states from
// the forward pass: only the chunk products that lead to a state in between are formed, and the scan restarts from
// every stored state.
void rla_forward_states(const LayerDims& dm, const FastFwdPlan& pl, const SeqTensors& t, float* U, void* states,
                        hipStream_t st, void* subset_out = nullptr, const void* restart = nullptr, int m = 1);
// MFMA backward path (same shape class as the MFMA forward)
struct FastBwdPlan {
  FastFwdPlan fwd;
  int nk;  // key tiles that have a linear branch = number of reverse states
  int nrchunks;  // reverse-time chunk-local products
  int rsplit;    // work-groups that share the query heads of such a product (each leaves one of its own)
  int RB;  // gain-gradient partials: one per wave of the dq kernel
  int nsplit;  // work-groups that share the query heads of a key tile in the dk/dv kernel
  size_t u_bytes, rstate_bytes, dkv_part_bytes;
};
struct FastBwdWs {
  void *dxs, *dxr;       // bf16 [B,T,Hq,D]
  float* delta;          // [2][B,Hq,T]: <dx_s, x_s> * scale, then the log-sum-exp in log2 units
  float* U;              // chunk scratch
  void *states, *rstates;
  float* dgpart;         // [2,RB,Hq,D]
  float* dkv_part;       // partial dk, then dv: [2][nsplit][B,Tc,Hkv,D] (nsplit > 1)
};
FastBwdPlan fast_bwd_plan(const LayerDims& dm);
// reverse-time states R_i = sum over t' >= 128(i+1) and over the group's heads of phi(q_{t'+W})^T dxr_{t'+W},
// i in [0, nk), nk = ceil((T-W)/128); stored transposed [d][f] bf16.  U: see FastBwdPlan.
// q [B,Tb,Hq,D], dxr [B,T,Hq,D] (padded length, zero in rows >= Tb).  `dg`: gain gradients summed on the way.
void rla_reverse_states(const LayerDims& dm, const FastBwdPlan& pl, const void* q, int Tb, const void* dxr, float* U,
                        void* rstates, hipStream_t st, const DgammaSum& dg);
// dm.T: the padded length; the caller's tensors hold Tc rows per sequence.  dO rows from 128 * (Tc / 128) on are read from
// dO_tail [B,128,Hq,D], zero past row Tc (may be NULL when Tc is a multiple of 128).
void fast_bwd(const LayerDims& dm, int Tc, const void* q, const void* k, const void* v, const float* gs, const float* gr,
              const SavedPtrs& sv, const void* dO, const void* dO_tail, void* dq, void* dk, void* dv, float* dgs, float* dgr,
              const FastBwdWs& ws, hipStream_t st);

// prefill -> decode hand-over: rings of the last min(T, W) tokens and the state of all keys before them
struct ExportPlan {
  int Tp;        // keys folded into the state (T - W, or 0)
  int nseg;      // key segments with their own partial state
  int seg_len;   // keys per segment (a multiple of 64)
  size_t partial_bytes;
};
ExportPlan export_plan(const LayerDims& dm);
// dm.T: the rows the plan counts (keys folded into the state + window).  Row s of the back part of `t` is token tok0 + s
// of its sequence: the last min(Tb, W) of them go to their ring slots.  The keys folded into the state are the plan's Tp
// rows from row t.kmin of the two-part sequence on; with `accumulate` they are added to what `state` already holds.
// (A front part: bf16 only.)
void prefill_export(const LayerDims& dm, int dtype, const SeqTensors& t, void* k_ring, void* v_ring, float* state,
                    float* partial, hipStream_t st, int tok0 = 0, bool accumulate = false);

// chunked prefill (see chunk_kernels.hip): R ring rows and Tc new rows as one [B,R+Tc,Hkv,D] tensor each ...
void chunk_concat(const LayerDims& dmc, int dtype, int Tc, int R, int pos0, const void* k, const void* v,
                  const void* k_ring, const void* v_ring, void* kc, void* vc, hipStream_t st);
// ... or (bf16) the ring rows alone as [B,P,Hkv,D], P = R rounded up to 128, zero rows in front
void chunk_ring(const LayerDims& dmc, int P, int R, int pos0, const void* k_ring, const void* v_ring, void* k_front,
                void* v_front, hipStream_t st);

// rows 128 * (T / 128) .. of a [B,T,H,D] bf16 tensor into its [B,128,H,D] tail buffer, zero from row T on
void gather_tail(const void* src, void* tail, int B, int T, int H, int D, hipStream_t st);

// launches the matrix-core probe loop; returns the FLOPs it issues
double probe_mfma(float* sink, int iters, int blocks, hipStream_t st);

struct DecodeDims {
  int N, Hq, Hkv, D, W, G;
  float scale, eps;
  int phi;  // as LayerDims::phi
  void* workspace = nullptr;         // NULL, or decode_split(..).bytes
  unsigned long long nonce = 0;      // with a workspace: a number no other call has, low 8 bits zero
  int once_rows = 0;                 // set by pick_decode: filled rows from which on a ring is read past the caches
};
// Work-groups that share a (sequence, kv head) in a decode step with a workspace (1: the step needs none)
constexpr int DEC_MAX_SPLIT = 16;
struct DecodeSplit {
  int n, rows;   // work-groups, and ring rows for each before there is another (rings that are not full yet)
  size_t part_off, bytes;   // tickets from offset 0
};
DecodeSplit decode_split(const DecodeDims& dd, int esize);
void decode_step(const DecodeDims& dd, int dtype, const void* q, const void* k_new, const void* v_new,
                 const int32_t* pos, void* k_ring, void* v_ring, float* state, const float* gs, const float* gr,
                 void* o, hipStream_t st);

}  // namespace rattn
