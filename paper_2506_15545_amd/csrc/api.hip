// C ABI of librattn: argument validation, workspace layout, path selection, launches.
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "kernels.hpp"
#include "rattn.h"

namespace rattn {
namespace {
// Event pairs come from a pool created by rattn_profile_enable(1): recording inside the layer calls allocates nothing.
struct ProfRec { const char* name; hipEvent_t a, b; };
bool g_prof_on = false;
ProfRec g_pool[RATTN_PROFILE_MAX_RECORDS];
int g_pool_size = 0;   // event pairs that exist
int g_prof_count = 0;  // records in use
bool g_prof_open = false;
}  // namespace
void prof_begin(const char* name, hipStream_t st) {
  g_prof_open = false;
  if (!g_prof_on || g_prof_count >= g_pool_size) return;
  ProfRec& r = g_pool[g_prof_count];
  r.name = name;
  if (hipEventRecord(r.a, st) != hipSuccess) return;  // tracing aid: the launch itself is not affected
  ++g_prof_count;
  g_prof_open = true;
}
void prof_end(hipStream_t st) {
  if (!g_prof_on || !g_prof_open) return;
  (void)hipEventRecord(g_pool[g_prof_count - 1].b, st);
  g_prof_open = false;
}
}  // namespace rattn

namespace {

thread_local char g_err[512] = "";

rattn_status fail(rattn_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return s;
}

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Sequence lengths from this size on run on the matrix-core kernels (bf16) whether or not they are a multiple of
// the 128-row tile.  Shorter ones (less than one tile) stay on the general kernels.
constexpr int FAST_MIN_T = 128;

struct Layout {
  rattn::LayerDims dm;
  rattn::LayerDims dmf;  // what the matrix-core kernels see: dm with T rounded up to whole 128-row tiles
  size_t esize;
  // saved
  size_t sv_xs, sv_xr, sv_lse, sv_rs, sv_rr, sv_states, saved_bytes;
  int state_stride;   // chunk states kept in `saved`: 0 = none, 1 = all, m = every m-th
  // generic forward / backward workspace
  size_t gen_fwd_bytes;
  size_t gb_rstates, gb_dxs, gb_dxr, gb_delta, gb_dgpart, gen_bwd_bytes;
  // MFMA forward / backward workspace
  bool fast_fwd;
  size_t ff_u, ff_states, fast_fwd_bytes;
  size_t fb_dxs, fb_dxr, fb_delta, fb_u, fb_states, fb_rstates, fb_dgpart, fb_dkv, fb_dO_tail, fast_bwd_bytes;
  size_t fwd_bytes, bwd_bytes;
};

// Scratch of the matrix-core kernels for dims `d` (padded length): offsets into L and totals
void fast_scratch(const rattn::LayerDims& d, Layout* L, size_t* fwd, size_t* bwd) {
  const rattn::FastFwdPlan pl = rattn::fast_fwd_plan(d);
  const rattn::FastBwdPlan bp = rattn::fast_bwd_plan(d);
  const size_t nq = (size_t)d.B * d.T * d.Hq * d.D, nrow = (size_t)d.B * d.Hq * d.T;
  size_t off = 0;
  L->ff_u = off; off += align_up(pl.u_bytes);
  L->ff_states = off; off += align_up(pl.state_bytes);
  *fwd = off;
  off = 0;
  L->fb_dxs = off; off += align_up(nq * 2);
  L->fb_dxr = off; off += align_up(nq * 2);
  L->fb_delta = off; off += align_up(nrow * 8);  // delta, then log-sum-exp in log2 units
  L->fb_u = off; off += align_up(bp.u_bytes);
  L->fb_states = off; off += align_up(bp.fwd.state_bytes);
  L->fb_rstates = off; off += align_up(bp.rstate_bytes);
  L->fb_dgpart = off; off += align_up((size_t)2 * bp.RB * d.Hq * d.D * 4);
  L->fb_dkv = off; off += align_up(bp.dkv_part_bytes);
  *bwd = off;
}

rattn_status make_layout(const rattn_params* p, Layout* L) {
  if (!p) return fail(RATTN_ERR_INVALID_ARG, "params is NULL");
  if (p->B < 1 || p->T < 1 || p->Hq < 1 || p->Hkv < 1)
    return fail(RATTN_ERR_INVALID_ARG, "B, T, Hq, Hkv must be >= 1 (got %d, %d, %d, %d)", p->B, p->T, p->Hq, p->Hkv);
  if (p->Hq % p->Hkv != 0)
    return fail(RATTN_ERR_INVALID_ARG, "Hq (%d) must be a multiple of Hkv (%d)", p->Hq, p->Hkv);
  if (p->B > 65535 || p->Hq > 65535)
    return fail(RATTN_ERR_UNSUPPORTED, "B and Hq must be <= 65535 (got %d, %d)", p->B, p->Hq);
  if (p->D != 64 && p->D != 128) return fail(RATTN_ERR_UNSUPPORTED, "head_dim D must be 64 or 128 (got %d)", p->D);
  if (p->window < 1) return fail(RATTN_ERR_INVALID_ARG, "window must be >= 1 (got %d)", p->window);
  if (p->chunk < 0) return fail(RATTN_ERR_INVALID_ARG, "chunk must be >= 0 (got %d)", p->chunk);
  if (p->dtype != RATTN_F32 && p->dtype != RATTN_BF16) return fail(RATTN_ERR_UNSUPPORTED, "unknown dtype %d", p->dtype);
  if (p->feature_map < RATTN_PHI_SOFTMAX || p->feature_map > RATTN_PHI_IDENTITY)
    return fail(RATTN_ERR_UNSUPPORTED, "unknown feature_map %d", p->feature_map);
  if (p->kernel_path != RATTN_PATH_AUTO && p->kernel_path != RATTN_PATH_GENERAL)
    return fail(RATTN_ERR_UNSUPPORTED, "unknown kernel_path %d", p->kernel_path);
  if (p->state_policy != RATTN_STATES_KEEP && p->state_policy != RATTN_STATES_REBUILD &&
      p->state_policy != RATTN_STATES_KEEP_EVERY_2ND && p->state_policy != RATTN_STATES_KEEP_EVERY_4TH)
    return fail(RATTN_ERR_UNSUPPORTED, "unknown state_policy %d", p->state_policy);
  if (!(p->rms_eps > 0.f)) return fail(RATTN_ERR_INVALID_ARG, "rms_eps must be > 0");
  if (!(p->softmax_scale == p->softmax_scale) || p->softmax_scale == 0.f)
    return fail(RATTN_ERR_INVALID_ARG, "softmax_scale must be a non-zero number");
  if ((long long)p->B * p->T >= (1ll << 31) / 4 || (long long)p->B * p->T * p->Hq * p->D >= (1ll << 40))
    return fail(RATTN_ERR_UNSUPPORTED, "tensor too large for 32-bit row indexing");

  rattn::LayerDims& dm = L->dm;
  dm.B = p->B; dm.T = p->T; dm.Hq = p->Hq; dm.Hkv = p->Hkv; dm.D = p->D;
  dm.W = p->window; dm.G = p->Hq / p->Hkv;
  const int Tp = p->T > p->window ? p->T - p->window : 0;
  dm.C = p->chunk > 0 ? p->chunk : rattn::generic_chunk(dm, Tp);
  dm.chunk_req = p->chunk;
  dm.nst = Tp > 0 ? (Tp - 1) / dm.C + 1 : 0;
  dm.scale = p->softmax_scale; dm.eps = p->rms_eps; dm.phi = p->feature_map;
  L->esize = p->dtype == RATTN_F32 ? 4 : 2;

  // What the matrix-core kernels would see: the sequence length rounded up to whole 128-row tiles
  L->dmf = dm;
  const bool ragged = dm.T % 128 != 0;
  if (dm.T >= FAST_MIN_T) L->dmf.T = (dm.T + 127) / 128 * 128;
  const rattn::LayerDims& dmf = L->dmf;
  // Identity feature map: only calls that keep nothing for a backward pass (inference, prefill) run on the matrix
  // cores.  Its backward with bf16 operands is not accurate enough: on the first rows past the window the state has
  // rank 1, 2, ..., d x^r is orthogonal to the few value rows x^r is made of, and with features of size ~1 (not ~1/D
  // as after the softmax map) the 2^-9 that rounding leaves of that cancellation reaches single dq elements at
  // 0.1 .. 2 times the gradient's RMS (GPU and the CPU model of the roundings agree on every such case).
  const bool identity_training = dm.phi == rattn::PHI_IDENTITY && p->save_for_bwd;
  L->fast_fwd = p->kernel_path != RATTN_PATH_GENERAL && !identity_training && rattn::fast_fwd_supported(dmf, p->dtype);
  if (!L->fast_fwd) L->dmf = dm;
  // `saved` is sized for the padded length
  const size_t nq = (size_t)dm.B * dm.T * dm.Hq * dm.D;
  const size_t nrow = (size_t)dm.B * dm.Hq * dm.T;
  const size_t nq_f = (size_t)dmf.B * dmf.T * dmf.Hq * dmf.D;
  const size_t nrow_f = (size_t)dmf.B * dmf.Hq * dmf.T;
  size_t off = 0;
  // pre-norm branch outputs: tensor dtype for the matrix-core kernels, fp32 for the general kernels
  const size_t sv_esize = L->fast_fwd ? L->esize : 4;
  L->sv_xs = off; off += align_up(nq_f * sv_esize);
  L->sv_xr = off; off += align_up(nq_f * sv_esize);
  L->sv_lse = off; off += align_up(nrow_f * 4);
  L->sv_rs = off; off += align_up(nrow_f * 4);
  L->sv_rr = off; off += align_up(nrow_f * 4);
  L->sv_states = off;
  // general kernels; with all keys in the first chunk there are none.  (The forward's workspace keeps room for that one: a call
  // without it is refused for every chunk size or for none.)
  const size_t nstate_fwd = (size_t)dm.B * dm.Hkv * dm.nst * dm.D * dm.D, nstate = dm.nst > 1 ? nstate_fwd : 0;
  if (L->fast_fwd)
    L->state_stride = p->state_policy == RATTN_STATES_KEEP ? 1 : p->state_policy == RATTN_STATES_REBUILD ? 0 : p->state_policy;
  else  // general kernels: all or none; all only where a chunk's states take no more room than its branch outputs
    L->state_stride = p->state_policy == RATTN_STATES_KEEP && dm.D <= 2ll * dm.G * dm.C ? 1 : 0;
  if (!L->fast_fwd) {
    off += L->state_stride ? align_up(nstate * 4) : 0;
  } else if (L->state_stride > 0) {
    const int nstf = rattn::fast_fwd_plan(dmf).nstf;
    off += align_up((size_t)dmf.B * dmf.Hkv * ((nstf + L->state_stride - 1) / L->state_stride) * dmf.D * dmf.D * 2);
  }
  L->saved_bytes = off;

  L->gen_fwd_bytes = align_up(nstate_fwd * 4);   // the same for both kinds of call (states that are kept are built in `saved`)

  off = 0;
  L->gb_rstates = off; off += align_up(nstate * 4);   // states that were not kept are rebuilt here first
  L->gb_dxs = off; off += align_up(nq * 4);
  L->gb_dxr = off; off += align_up(nq * 4);
  L->gb_delta = off; off += align_up(nrow * 4);
  L->gb_dgpart = off; off += align_up((size_t)2 * dm.B * ((dm.T + 15) / 16) * dm.Hq * dm.D * 4);
  L->gen_bwd_bytes = off;

  L->ff_u = L->ff_states = L->fast_fwd_bytes = L->fast_bwd_bytes = 0;
  if (L->fast_fwd) {
    fast_scratch(dmf, L, &L->fast_fwd_bytes, &L->fast_bwd_bytes);
    L->fb_dO_tail = L->fast_bwd_bytes;
    if (ragged) L->fast_bwd_bytes += align_up((size_t)dm.B * 128 * dm.Hq * dm.D * 2);
  }
  L->fwd_bytes = L->fast_fwd ? L->fast_fwd_bytes : L->gen_fwd_bytes;
  L->bwd_bytes = L->fast_fwd ? L->fast_bwd_bytes : L->gen_bwd_bytes;
  return RATTN_OK;
}

rattn::SavedPtrs saved_views(const Layout& L, void* saved) {
  rattn::SavedPtrs sv = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0};
  if (saved) {
    char* s = (char*)saved;
    sv.xs = s + L.sv_xs; sv.xr = s + L.sv_xr;
    sv.lse = (float*)(s + L.sv_lse); sv.rs = (float*)(s + L.sv_rs); sv.rr = (float*)(s + L.sv_rr);
    if (L.state_stride > 0) { sv.states = s + L.sv_states; sv.state_stride = L.state_stride; }
  }
  return sv;
}

// chunked prefill: the forward runs over R ring rows + the chunk's T rows
struct ChunkLayout {
  rattn_params p2;
  Layout L2;
  int R;   // ring rows in front of the chunk
  int P;   // matrix-core kernels: R rounded up to whole tiles, so that the chunk starts at a tile
  rattn::ChunkPlan plan;   // matrix-core kernels
  size_t kc, vc, fwdws, partial, states, bytes;
};

rattn_status make_chunk_layout(const rattn_params* p, int32_t pos0, ChunkLayout* C) {
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (pos0 < 0) return fail(RATTN_ERR_INVALID_ARG, "pos0 must be >= 0 (got %d)", pos0);
  if ((long long)pos0 + p->T >= (1ll << 31)) return fail(RATTN_ERR_UNSUPPORTED, "pos0 + T must stay below 2^31");
  C->R = pos0 < p->window ? pos0 : p->window;
  C->P = (int)(((long long)C->R + 127) / 128 * 128);
  C->p2 = *p;
  C->p2.save_for_bwd = 0;
  if ((long long)C->P + p->T >= (1ll << 31)) return fail(RATTN_ERR_UNSUPPORTED, "window + T must stay below 2^31");
  C->p2.T = C->P + p->T;
  // Head size 64 and the identity map keep the fp32 arithmetic of the general kernels: their outputs are the exact result
  // rounded once (error against fp64 1.65e-3, all of it the rounding of o), on bf16 operands they are 2.1 - 2.3e-3 off.
  if (C->R + p->T < FAST_MIN_T || p->D == 64 || p->feature_map == RATTN_PHI_IDENTITY) C->p2.kernel_path = RATTN_PATH_GENERAL;
  s = make_layout(&C->p2, &C->L2);
  if (s != RATTN_OK) return s;
  if (!C->L2.fast_fwd) {   // general kernels: exactly the rows there are
    C->P = 0;
    C->p2.T = C->R + p->T;
    s = make_layout(&C->p2, &C->L2);
    if (s != RATTN_OK) return s;
  }
  rattn::LayerDims dmx = C->L2.dm;   // rows the state update counts
  dmx.T = C->R + p->T;
  const int front = C->L2.fast_fwd ? C->P : dmx.T;
  const size_t nkv = (size_t)dmx.B * front * dmx.Hkv * dmx.D * C->L2.esize;
  size_t off = 0;
  C->kc = off; off += align_up(nkv);
  C->vc = off; off += align_up(nkv);
  C->fwdws = off;
  C->plan.nprod = 0;
  if (C->L2.fast_fwd) C->plan = rattn::chunk_plan(C->L2.dmf, C->P, C->R, p->T);
  if (C->plan.nprod > 0) {   // products, then states
    off += align_up(C->plan.u_bytes);
    C->states = off; off += align_up(rattn::fast_fwd_plan(C->L2.dmf).state_bytes);
    C->partial = off;
  } else {
    C->states = off + C->L2.ff_states;
    off += align_up(C->L2.fwd_bytes);
    C->partial = off; off += align_up(rattn::export_plan(dmx).partial_bytes);
  }
  C->bytes = off > 0 ? off : 256;
  return RATTN_OK;
}

rattn_status check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(RATTN_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
  return RATTN_OK;
}

}  // namespace

extern "C" {

const char* rattn_status_string(rattn_status s) {
  switch (s) {
    case RATTN_OK: return "ok";
    case RATTN_ERR_INVALID_ARG: return "invalid argument";
    case RATTN_ERR_UNSUPPORTED: return "unsupported configuration";
    case RATTN_ERR_WORKSPACE: return "workspace too small";
    case RATTN_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

const char* rattn_last_error(void) { return g_err; }

void rattn_profile_reset(void) {
  rattn::g_prof_count = 0;
  rattn::g_prof_open = false;
}
void rattn_profile_enable(int on) {
  rattn_profile_reset();
  if (on) {  // fill the event pool once; the layer calls only record into it
    while (rattn::g_pool_size < RATTN_PROFILE_MAX_RECORDS) {
      rattn::ProfRec& r = rattn::g_pool[rattn::g_pool_size];
      if (hipEventCreate(&r.a) != hipSuccess) break;
      if (hipEventCreate(&r.b) != hipSuccess) { (void)hipEventDestroy(r.a); break; }
      ++rattn::g_pool_size;
    }
  }
  rattn::g_prof_on = on != 0;
}
int rattn_profile_count(void) { return rattn::g_prof_count; }
rattn_status rattn_profile_get(int idx, const char** name, float* ms) {
  if (idx < 0 || idx >= rattn::g_prof_count) return fail(RATTN_ERR_INVALID_ARG, "profile index %d out of range", idx);
  const auto& r = rattn::g_pool[idx];
  if (hipEventSynchronize(r.b) != hipSuccess) return fail(RATTN_ERR_HIP, "hipEventSynchronize failed");
  float t = 0.f;
  if (hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) return fail(RATTN_ERR_HIP, "hipEventElapsedTime failed");
  if (name) *name = r.name;
  if (ms) *ms = t;
  return RATTN_OK;
}
const char* rattn_version(void) { return "0.1"; }

rattn_status rattn_workspace_bytes(const rattn_params* p, size_t* fwd_bytes, size_t* bwd_bytes, size_t* saved_bytes) {
  if (!p) return fail(RATTN_ERR_INVALID_ARG, "params is NULL");
  // sizes do not depend on save_for_bwd: `saved` and the backward scratch are those of a call that saves, the
  // forward scratch covers both kinds of call (they differ only where the kernel family depends on it)
  rattn_params q = *p;
  Layout L;
  q.save_for_bwd = 1;
  rattn_status s = make_layout(&q, &L);
  if (s != RATTN_OK) return s;
  size_t fwd = L.fwd_bytes;
  Layout L0;
  q.save_for_bwd = 0;
  s = make_layout(&q, &L0);
  if (s != RATTN_OK) return s;
  if (L0.fwd_bytes > fwd) fwd = L0.fwd_bytes;
  if (fwd_bytes) *fwd_bytes = fwd;
  if (bwd_bytes) *bwd_bytes = L.bwd_bytes;
  if (saved_bytes) *saved_bytes = L.saved_bytes;
  return RATTN_OK;
}

rattn_status rattn_fwd(const rattn_params* p, const void* q, const void* k, const void* v, const float* gamma_swa,
                       const float* gamma_rla, void* o, void* saved, void* workspace, size_t workspace_bytes,
                       void* stream) {
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (!q || !k || !v || !o) return fail(RATTN_ERR_INVALID_ARG, "q, k, v, o must be non-NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(saved) || !aligned16(workspace))
    return fail(RATTN_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  if (p->save_for_bwd && !saved) return fail(RATTN_ERR_INVALID_ARG, "save_for_bwd set but saved is NULL");
  if (L.fwd_bytes > 0 && (!workspace || workspace_bytes < L.fwd_bytes))
    return fail(RATTN_ERR_WORKSPACE, "forward needs %zu workspace bytes, got %zu", L.fwd_bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  rattn::SavedPtrs sv = saved_views(L, p->save_for_bwd ? saved : nullptr);
  if (L.fast_fwd) {
    char* w = (char*)workspace;
    rattn::SeqTensors t;
    t.k = k; t.v = v; t.Tb = L.dm.T;
    rattn::fast_fwd(L.dmf, t, q, gamma_swa, gamma_rla, o, sv, (float*)(w + L.ff_u),
                    sv.states && sv.state_stride <= 1 ? sv.states : (void*)(w + L.ff_states), st);
  } else
    rattn::generic_fwd(L.dm, p->dtype, q, k, v, gamma_swa, gamma_rla, o, sv,
                       sv.states ? (float*)sv.states : (float*)workspace, st);
  return check_launch("rattn_fwd");
}

// ---- rattn_fwd_static: the forward with its scratch memory inside the library's device image
// BEGIN-STATIC-ENTRY
namespace {
// One copy per GPU that loads this library, alive until the process ends.  In host code the array's name is only
// a handle for hipGetSymbolAddress; the kernels get the looked-up device address like any other workspace.
static __device__ __align__(256) unsigned char scratch[RATTN_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES] = {nullptr};  // device address of `scratch`, per device, looked up once
}  // namespace

rattn_status rattn_fwd_static(const rattn_params* p, const void* q, const void* k, const void* v,
                              const float* gamma_swa, const float* gamma_rla, void* o, void* saved, void* stream) {
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (L.fwd_bytes > RATTN_STATIC_SCRATCH_BYTES)
    return fail(RATTN_ERR_WORKSPACE, "rattn_fwd_static: this shape needs %zu bytes of forward scratch, the built-in buffer "
                "holds %zu; use rattn_fwd with a caller-provided workspace", L.fwd_bytes, (size_t)RATTN_STATIC_SCRATCH_BYTES);
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES)
    return fail(RATTN_ERR_HIP, "rattn_fwd_static: no current HIP device (or device index >= %d)", MAX_DEVICES);
  void* ws = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
  if (!ws) {  // first call on this device (every thread that gets here looks up the same address)
    const hipError_t e = hipGetSymbolAddress(&ws, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ws)
      return fail(RATTN_ERR_HIP, "rattn_fwd_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
    __atomic_store_n(&g_scratch_ptr[dev], ws, __ATOMIC_RELEASE);
  }
  // Every part of the scratch that the forward kernels read is written earlier in the same call (chunk products,
  // then the scanned states), so nothing has to be cleared.
  return rattn_fwd(p, q, k, v, gamma_swa, gamma_rla, o, saved, ws, RATTN_STATIC_SCRATCH_BYTES, stream);
}
// END-STATIC-ENTRY

rattn_status rattn_bwd(const rattn_params* p, const void* q, const void* k, const void* v, const float* gamma_swa,
                       const float* gamma_rla, const void* saved, const void* dO, void* dq, void* dk, void* dv,
                       float* dgamma_swa, float* dgamma_rla, void* workspace, size_t workspace_bytes, void* stream) {
  if (!p) return fail(RATTN_ERR_INVALID_ARG, "params is NULL");
  rattn_params pb = *p;
  pb.save_for_bwd = 1;   // `saved` comes from a forward call that saved, whatever this copy of the parameters says
  p = &pb;
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (!q || !k || !v || !saved || !dO || !dq || !dk || !dv)
    return fail(RATTN_ERR_INVALID_ARG, "q, k, v, saved, dO, dq, dk, dv must be non-NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(saved) || !aligned16(dO) || !aligned16(dq) ||
      !aligned16(dk) || !aligned16(dv) || !aligned16(workspace))
    return fail(RATTN_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  if (!workspace || workspace_bytes < L.bwd_bytes)
    return fail(RATTN_ERR_WORKSPACE, "backward needs %zu workspace bytes, got %zu", L.bwd_bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  rattn::SavedPtrs sv = saved_views(L, const_cast<void*>(saved));
  char* w = (char*)workspace;
  if (L.fast_fwd) {
    rattn::FastBwdWs fw;
    fw.dxs = w + L.fb_dxs; fw.dxr = w + L.fb_dxr; fw.delta = (float*)(w + L.fb_delta); fw.U = (float*)(w + L.fb_u);
    fw.states = w + L.fb_states; fw.rstates = w + L.fb_rstates; fw.dgpart = (float*)(w + L.fb_dgpart);
    fw.dkv_part = (float*)(w + L.fb_dkv);
    // the rows of dO past the last whole tile, zero-filled: what the kernels compute for the rows of a tile that do not
    // exist then adds nothing to any gradient
    const bool ragged = L.dm.T % 128 != 0;
    if (ragged) rattn::gather_tail(dO, w + L.fb_dO_tail, L.dm.B, L.dm.T, L.dm.Hq, L.dm.D, st);
    rattn::fast_bwd(L.dmf, L.dm.T, q, k, v, gamma_swa, gamma_rla, sv, dO, ragged ? w + L.fb_dO_tail : nullptr, dq, dk, dv,
                    dgamma_swa, dgamma_rla, fw, st);
    return check_launch("rattn_bwd");
  }
  rattn::GenericBwdWs ws;
  ws.rstates = (float*)(w + L.gb_rstates);
  ws.dxs = (float*)(w + L.gb_dxs); ws.dxr = (float*)(w + L.gb_dxr);
  ws.delta = (float*)(w + L.gb_delta); ws.dgpart = (float*)(w + L.gb_dgpart);
  rattn::generic_bwd(L.dm, p->dtype, q, k, v, gamma_swa, gamma_rla, sv, dO, dq, dk, dv, dgamma_swa, dgamma_rla, ws, st);
  return check_launch("rattn_bwd");
}

namespace {
rattn_status decode_dims(const rattn_decode_params* p, rattn::DecodeDims* dd) {
  if (!p) return fail(RATTN_ERR_INVALID_ARG, "params is NULL");
  if (p->N < 1 || p->Hq < 1 || p->Hkv < 1)
    return fail(RATTN_ERR_INVALID_ARG, "N, Hq, Hkv must be >= 1 (got %d, %d, %d)", p->N, p->Hq, p->Hkv);
  if (p->Hq % p->Hkv != 0)
    return fail(RATTN_ERR_INVALID_ARG, "Hq (%d) must be a multiple of Hkv (%d)", p->Hq, p->Hkv);
  if (p->D != 64 && p->D != 128) return fail(RATTN_ERR_UNSUPPORTED, "head_dim D must be 64 or 128 (got %d)", p->D);
  if (p->window < 1) return fail(RATTN_ERR_INVALID_ARG, "window must be >= 1 (got %d)", p->window);
  if (p->dtype != RATTN_F32 && p->dtype != RATTN_BF16) return fail(RATTN_ERR_UNSUPPORTED, "unknown dtype %d", p->dtype);
  if (p->feature_map < RATTN_PHI_SOFTMAX || p->feature_map > RATTN_PHI_IDENTITY)
    return fail(RATTN_ERR_UNSUPPORTED, "unknown feature_map %d", p->feature_map);
  if (!(p->rms_eps > 0.f)) return fail(RATTN_ERR_INVALID_ARG, "rms_eps must be > 0");
  if (!(p->softmax_scale == p->softmax_scale) || p->softmax_scale == 0.f)
    return fail(RATTN_ERR_INVALID_ARG, "softmax_scale must be a non-zero number");
  if (p->N > 65535) return fail(RATTN_ERR_UNSUPPORTED, "N must be <= 65535 (got %d)", p->N);
  if ((long long)p->N * p->Hkv * p->window * p->D >= (1ll << 40))
    return fail(RATTN_ERR_UNSUPPORTED, "ring buffers too large");
  dd->N = p->N; dd->Hq = p->Hq; dd->Hkv = p->Hkv; dd->D = p->D; dd->W = p->window; dd->G = p->Hq / p->Hkv;
  dd->scale = p->softmax_scale; dd->eps = p->rms_eps; dd->phi = p->feature_map;
  return RATTN_OK;
}
// A number that no other call of this process has, spread over the upper 56 bits (the multiplier is odd: no two counts give
// the same), so that what happens to lie in memory does not look like one
unsigned long long decode_nonce() {
  static unsigned long long count = 0;
  return (__atomic_add_fetch(&count, 1, __ATOMIC_RELAXED) * 0x9E3779B97F4A7C15ull) << 8;
}
}  // namespace

rattn_status rattn_decode_workspace_bytes(const rattn_decode_params* p, size_t* bytes) {
  rattn::DecodeDims dd;
  rattn_status s = decode_dims(p, &dd);
  if (s != RATTN_OK) return s;
  if (bytes) *bytes = rattn::decode_split(dd, p->dtype == RATTN_F32 ? 4 : 2).bytes;
  return RATTN_OK;
}

rattn_status rattn_decode_step_ws(const rattn_decode_params* p, const void* q, const void* k_new, const void* v_new,
                                  const int32_t* pos, void* k_ring, void* v_ring, float* state, const float* gamma_swa,
                                  const float* gamma_rla, void* o, void* workspace, size_t workspace_bytes, void* stream) {
  rattn::DecodeDims dd;
  rattn_status s = decode_dims(p, &dd);
  if (s != RATTN_OK) return s;
  if (!q || !k_new || !v_new || !pos || !k_ring || !v_ring || !state || !o)
    return fail(RATTN_ERR_INVALID_ARG, "q, k_new, v_new, pos, k_ring, v_ring, state, o must be non-NULL");
  if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(k_ring) || !aligned16(v_ring) ||
      !aligned16(state) || !aligned16(o) || !aligned16(workspace))
    return fail(RATTN_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  const size_t need = rattn::decode_split(dd, p->dtype == RATTN_F32 ? 4 : 2).bytes;
  if (workspace && workspace_bytes < need)
    return fail(RATTN_ERR_WORKSPACE, "decode step needs %zu workspace bytes (or none), got %zu", need, workspace_bytes);
  if (workspace && need > 0) { dd.workspace = workspace; dd.nonce = decode_nonce(); }
  rattn::decode_step(dd, p->dtype, q, k_new, v_new, pos, k_ring, v_ring, state, gamma_swa, gamma_rla, o,
                     (hipStream_t)stream);
  return check_launch("rattn_decode_step");
}

rattn_status rattn_decode_step(const rattn_decode_params* p, const void* q, const void* k_new, const void* v_new,
                               const int32_t* pos, void* k_ring, void* v_ring, float* state, const float* gamma_swa,
                               const float* gamma_rla, void* o, void* stream) {
  return rattn_decode_step_ws(p, q, k_new, v_new, pos, k_ring, v_ring, state, gamma_swa, gamma_rla, o, nullptr, 0, stream);
}

rattn_status rattn_prefill_export_workspace_bytes(const rattn_params* p, size_t* bytes) {
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (bytes) *bytes = align_up(rattn::export_plan(L.dm).partial_bytes);
  return RATTN_OK;
}

rattn_status rattn_prefill_export(const rattn_params* p, const void* k, const void* v, void* k_ring, void* v_ring,
                                  float* state, void* workspace, size_t workspace_bytes, void* stream) {
  Layout L;
  rattn_status s = make_layout(p, &L);
  if (s != RATTN_OK) return s;
  if (!k || !v || !k_ring || !v_ring || !state) return fail(RATTN_ERR_INVALID_ARG, "k, v, k_ring, v_ring, state must be non-NULL");
  if (!aligned16(k) || !aligned16(v) || !aligned16(k_ring) || !aligned16(v_ring) || !aligned16(state) ||
      !aligned16(workspace))
    return fail(RATTN_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  const size_t need = align_up(rattn::export_plan(L.dm).partial_bytes);
  if (need > 0 && (!workspace || workspace_bytes < need))
    return fail(RATTN_ERR_WORKSPACE, "prefill export needs %zu workspace bytes, got %zu", need, workspace_bytes);
  rattn::SeqTensors t;
  t.k = k; t.v = v; t.Tb = L.dm.T;
  rattn::prefill_export(L.dm, p->dtype, t, k_ring, v_ring, state, (float*)workspace, (hipStream_t)stream);
  return check_launch("rattn_prefill_export");
}

rattn_status rattn_prefill_chunk_workspace_bytes(const rattn_params* p, int32_t pos0, size_t* bytes) {
  ChunkLayout C;
  rattn_status s = make_chunk_layout(p, pos0, &C);
  if (s != RATTN_OK) return s;
  if (bytes) *bytes = C.bytes;
  return RATTN_OK;
}

rattn_status rattn_prefill_chunk(const rattn_params* p, int32_t pos0, const void* q, const void* k, const void* v,
                                 const float* gamma_swa, const float* gamma_rla, void* k_ring, void* v_ring,
                                 float* state, void* o, void* workspace, size_t workspace_bytes, void* stream) {
  ChunkLayout C;
  rattn_status s = make_chunk_layout(p, pos0, &C);
  if (s != RATTN_OK) return s;
  if (!q || !k || !v || !o || !k_ring || !v_ring || !state)
    return fail(RATTN_ERR_INVALID_ARG, "q, k, v, o, k_ring, v_ring, state must be non-NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(k_ring) || !aligned16(v_ring) ||
      !aligned16(state) || !aligned16(workspace))
    return fail(RATTN_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  if (!workspace || workspace_bytes < C.bytes)
    return fail(RATTN_ERR_WORKSPACE, "chunked prefill needs %zu workspace bytes, got %zu", C.bytes, workspace_bytes);
  hipStream_t st = (hipStream_t)stream;
  char* w = (char*)workspace;
  const rattn::LayerDims& dm = C.L2.dm;
  // keys before the ring exist only once more than `window` tokens have been seen; until then the state is zero
  // by definition and what the caller's buffer holds is not read
  const bool carried = pos0 > p->window;
  rattn::LayerDims dmx = dm;   // rows the state update counts
  dmx.T = C.R + p->T;
  rattn::SavedPtrs none = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0};
  rattn::SeqTensors t;
  // The forward computes the chunk's rows only, straight from q into o; a carried state is the initial value of the
  // chunk-state scan, of which every chunk row reads a state (the keys before it number at least `window` then).
  if (C.L2.fast_fwd) {
    // only the ring rows are gathered, as the whole 128-row tiles in front of the chunk's
    t.k = k; t.v = v; t.Tb = p->T; t.P = C.P; t.kmin = C.P - C.R;
    if (C.P > 0) { t.k_front = w + C.kc; t.v_front = w + C.vc; }
    const rattn::ChunkHandover handover = {C.plan, k_ring, v_ring, state, C.R, pos0, carried ? 1 : 0};
    if (C.plan.nprod > 0) t.handover = &handover;
    else if (C.P > 0) rattn::chunk_ring(dm, C.P, C.R, pos0, k_ring, v_ring, w + C.kc, w + C.vc, st);
    rattn::fast_fwd(C.L2.dmf, t, q, gamma_swa, gamma_rla, o, none, (float*)(w + C.fwdws), w + C.states, st);
    // (not shared: nothing is carried either, so the state is what the export forms)
    if (C.plan.nprod == 0) rattn::prefill_export(dmx, p->dtype, t, k_ring, v_ring, state, (float*)(w + C.partial), st, pos0);
  } else {
    t.k = w + C.kc; t.v = w + C.vc; t.Tb = dmx.T;
    rattn::chunk_concat(dm, p->dtype, p->T, C.R, pos0, k, v, k_ring, v_ring, w + C.kc, w + C.vc, st);
    rattn::generic_fwd(dm, p->dtype, q, t.k, t.v, gamma_swa, gamma_rla, o, none, (float*)(w + C.fwdws), st,
                       C.R, carried ? state : nullptr);
    rattn::prefill_export(dmx, p->dtype, t, k_ring, v_ring, state, (float*)(w + C.partial), st, pos0 - C.R, carried);
  }
  return check_launch("rattn_prefill_chunk");
}

rattn_status rattn_cache_bytes(int32_t layers, int32_t global_every, int64_t ctx, int64_t window, int32_t with_state,
                               int32_t Hkv, int32_t D, int32_t elem_bytes, double* out) {
  if (!out) return fail(RATTN_ERR_INVALID_ARG, "out is NULL");
  if (layers < 0 || global_every < 0 || ctx < 0 || window < 0 || Hkv < 1 || D < 1 || elem_bytes < 1)
    return fail(RATTN_ERR_INVALID_ARG, "sizes must be non-negative (Hkv, D, elem_bytes positive)");
  const int n_glob = global_every > 0 ? layers / global_every : 0;
  const int n_loc = layers - n_glob;
  const double tok = 2.0 * Hkv * D * elem_bytes;
  const double loc_tokens = (double)(ctx < window ? ctx : window);
  const double st = with_state ? (double)Hkv * D * D * 4.0 : 0.0;
  *out = n_glob * (double)ctx * tok + n_loc * (loc_tokens * tok + st);
  return RATTN_OK;
}

rattn_status rattn_step_time_model(double batch, double cache_bytes, double param_count, double param_bytes,
                                   double bandwidth, double flops, double* out) {
  if (!out) return fail(RATTN_ERR_INVALID_ARG, "out is NULL");
  if (!(batch >= 0.0) || !(cache_bytes >= 0.0) || !(param_count >= 0.0) || !(param_bytes >= 0.0))
    return fail(RATTN_ERR_INVALID_ARG, "batch, cache_bytes, param_count, param_bytes must be >= 0");
  if (!(bandwidth > 0.0) || !(flops > 0.0)) return fail(RATTN_ERR_INVALID_ARG, "bandwidth and flops must be > 0");
  const double compute = 2.0 * batch * param_count / flops, weights = param_bytes / bandwidth;
  *out = batch * cache_bytes / bandwidth + (compute > weights ? compute : weights);
  return RATTN_OK;
}

rattn_status rattn_probe_mfma(void* sink, int iters, int blocks, double* flops, void* stream) {
  if (!sink || !aligned16(sink)) return fail(RATTN_ERR_INVALID_ARG, "sink must be a 16-byte aligned device pointer");
  if (iters < 1 || iters > (1 << 24) || blocks < 1 || blocks > (1 << 20))
    return fail(RATTN_ERR_INVALID_ARG, "iters must be in [1, 2^24] and blocks in [1, 2^20] (got %d, %d)", iters, blocks);
  const double f = rattn::probe_mfma((float*)sink, iters, blocks, (hipStream_t)stream);
  if (flops) *flops = f;
  return check_launch("rattn_probe_mfma");
}

}  // extern "C"
