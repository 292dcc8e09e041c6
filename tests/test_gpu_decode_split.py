"""Decode steps whose (sequence, KV head) pairs are shared by several work-groups that meet in a workspace, and large ones whose
rings are read past the caches."""
import ctypes
import math

import numpy as np
import pytest
import torch

import parity_metrics as pm

from oracle import rattn_oracle as orc
from paper_2506_15545_amd import binding as rb, synth

pytestmark = pytest.mark.gpu
np64 = lambda t: t.detach().cpu().to(torch.float64).numpy()
NAMES = ("q", "k_new", "v_new", "pos", "k_ring", "v_ring", "state")


def inputs(N, Hq, Hkv, D, W, dtype, pos, seed):
    cfg = synth.DecodeConfig("split", N, Hq, Hkv, D, W, dtype, seed, 0, max(pos), 1.0 / math.sqrt(D))
    return synth.make_decode_inputs(cfg, pos=pos), cfg.scale


def workspace_bytes(N, Hq, Hkv, D, W, dtype):
    n = ctypes.c_size_t()
    p = rb.RattnDecodeParams(N, Hq, Hkv, D, W, rb.RATTN_F32 if dtype == "f32" else rb.RATTN_BF16, 1.0, 1e-6, 0)
    assert rb.lib().rattn_decode_workspace_bytes(ctypes.byref(p), ctypes.byref(n)) == 0
    return p, n.value


@pytest.mark.parametrize("N,Hq,Hkv,D,W,dtype,n,pos", [
    (1, 4, 1, 128, 512, "bf16", 4, [2000]),
    (4, 6, 2, 128, 515, "bf16", 4, [0, 1, 384, 385]),           # one work-group, four: rings that are not full yet
    (4, 6, 2, 128, 515, "bf16", 4, [512, 514, 515, 516]),
    (3, 2, 1, 128, 1024, "bf16", 8, [512, 513, 897]),           # four, five, eight
    (2, 16, 1, 128, 4096, "bf16", 16, [4095, 9000]),            # all sixteen, sixteen heads
    (1, 5, 1, 64, 1025, "bf16", 4, [1024]),
    (3, 3, 1, 64, 1100, "f32", 8, [100, 1099, 5000]),
    (2, 16, 1, 128, 1030, "f32", 16, [700, 3333]),
    (64, 8, 1, 128, 512, "bf16", 2, [400] * 32 + [700] * 32),   # 128 work-groups
    (65, 8, 1, 128, 512, "bf16", 1, [700] * 65),                # one pair more: no split
    (1, 1, 1, 128, 511, "bf16", 1, [700]),                      # rings below 256 KB
])
def test_shared_pairs(N, Hq, Hkv, D, W, dtype, n, pos):
    """Against the oracle: outputs as the unshared step's (bf16 storage; fp32 sums of up to W terms), rings to the bit, the state
    to one fp32 multiply-add; the rule asks for a workspace of n work-groups per pair, and for none without a split."""
    _, nbytes = workspace_bytes(N, Hq, Hkv, D, W, dtype)
    G = Hq // Hkv
    part = N * Hkv * n * G * (2 * D + 4) * 4
    assert nbytes == 0 if n == 1 else part < nbytes <= part + 8 * N * Hkv + 256
    d, scale = inputs(N, Hq, Hkv, D, W, dtype, pos, 5600 + W + N)
    print(f"N={N} Hq={Hq} Hkv={Hkv} D={D} W={W} {dtype}", flush=True)
    o_ref, kr_ref, vr_ref, S_ref = orc.decode_step(*(np64(d[m]) for m in ("q", "k_new", "v_new")), d["pos"].tolist(),
                                                   *(np64(d[m]) for m in ("k_ring", "v_ring", "state")), W, scale=scale)
    x = {m: t.cuda() for m, t in d.items()}
    o = rb.rattn_decode_step(*(x[m] for m in NAMES), softmax_scale=scale)
    if dtype == "bf16":
        pm.assert_out_bf16(np64(o), o_ref, what="o")
    else:
        assert float(np.abs(np64(o) - o_ref).max()) <= 1e-4
    assert np.array_equal(np64(x["k_ring"]), kr_ref) and np.array_equal(np64(x["v_ring"]), vr_ref)
    assert float(np.abs(np64(x["state"]) - S_ref).max()) <= 1e-5 * max(1.0, float(np.abs(S_ref).max()))
    # the same call without a workspace
    y = {m: t.cuda() for m, t in d.items()}
    o2 = torch.empty_like(o)
    p, _ = workspace_bytes(N, Hq, Hkv, D, W, dtype)
    p.softmax_scale = scale
    assert rb.lib().rattn_decode_step(ctypes.byref(p), *(y[m].data_ptr() for m in NAMES), None, None, o2.data_ptr(), rb._stream()) == 0
    err = float((o.float() - o2.float()).norm() / o2.float().norm())
    assert err <= (2e-3 if dtype == "bf16" else 1e-6), err
    assert torch.equal(x["k_ring"], y["k_ring"]) and torch.equal(x["state"], y["state"])


def test_workspace_contents_do_not_matter():
    """Tickets are found cleared, as noise, as what an earlier call would leave or full of ones: the same bits each time, and
    cleared tickets behind every call.  A workspace that is too small is refused."""
    N, Hq, Hkv, D, W = 3, 8, 2, 128, 1024
    d, scale = inputs(N, Hq, Hkv, D, W, "bf16", [700, 1024, 5000], 5700)
    p, nbytes = workspace_bytes(N, Hq, Hkv, D, W, "bf16")
    p.softmax_scale = scale
    tickets = 8 * N * Hkv
    gen = torch.Generator(device="cuda").manual_seed(1)
    noise = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=gen)
    fills = [torch.zeros_like(noise), noise, torch.full_like(noise, 255), torch.full_like(noise, 1), None, None]
    ws, outs = torch.empty_like(noise), []
    for fill in fills:   # None: as the call before left it
        if fill is not None:
            ws.copy_(fill)
        x = {m: t.cuda() for m, t in d.items()}
        o = torch.empty_like(x["q"])
        assert rb.lib().rattn_decode_step_ws(ctypes.byref(p), *(x[m].data_ptr() for m in NAMES), None, None, o.data_ptr(),
                                             ws.data_ptr(), nbytes, rb._stream()) == 0
        outs.append((o, x["state"], x["k_ring"]))
        assert not bool(ws[:tickets].any())
    for out in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out, outs[0]))
    assert rb.lib().rattn_decode_step_ws(ctypes.byref(p), *(x[m].data_ptr() for m in NAMES), None, None, o.data_ptr(),
                                         ws.data_ptr(), nbytes - 1, rb._stream()) == -3


def test_replayed_and_overlapping_calls():
    """A captured step replayed between eager ones, and steps on two streams at once: the bits of single calls."""
    N, Hq, Hkv, D, W = 2, 8, 2, 128, 2048
    case = lambda seed: inputs(N, Hq, Hkv, D, W, "bf16", [1500, 4000], seed)
    d, scale = case(5800)
    want = {}
    for seed in (5800, 5801):
        x = {m: t.cuda() for m, t in case(seed)[0].items()}
        want[seed] = rb.rattn_decode_step(*(x[m] for m in NAMES), softmax_scale=scale), x["state"]
    x = {m: t.cuda() for m, t in d.items()}
    out = torch.empty_like(x["q"])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rb.rattn_decode_step(*(x[m] for m in NAMES), softmax_scale=scale, out=out)
    for _ in range(3):
        for m in ("k_ring", "v_ring", "state"):
            x[m].copy_(d[m])
        out.zero_()
        graph.replay()
        y = {m: t.cuda() for m, t in case(5801)[0].items()}
        eager = rb.rattn_decode_step(*(y[m] for m in NAMES), softmax_scale=scale)
        torch.cuda.synchronize()
        assert torch.equal(out, want[5800][0]) and torch.equal(x["state"], want[5800][1])
        assert torch.equal(eager, want[5801][0]) and torch.equal(y["state"], want[5801][1])
    streams, got = [torch.cuda.Stream() for _ in range(2)], []
    for i in range(8):
        seed = 5800 + i % 2
        y = {m: t.cuda() for m, t in case(seed)[0].items()}
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[i % 2]):
            got.append((seed, rb.rattn_decode_step(*(y[m] for m in NAMES), softmax_scale=scale), y))
    torch.cuda.synchronize()
    for seed, o, y in got:
        assert torch.equal(o, want[seed][0]) and torch.equal(y["state"], want[seed][1])


@pytest.mark.parametrize("N,D,W,dtype", [
    (32, 128, 895, "bf16"), (32, 128, 896, "bf16"),   # 256 pairs, 16 waves: the last window below 128 MB of rings and states, the first above
    (64, 128, 383, "bf16"), (64, 128, 385, "bf16"),   # 512, eight waves
    (128, 128, 128, "bf16"), (128, 64, 450, "bf16"),  # 1024, four waves
    (32, 128, 448, "f32"), (64, 128, 191, "f32"), (64, 128, 193, "f32"), (128, 64, 224, "f32"),
])
def test_large_steps_match_small_ones(N, D, W, dtype):
    """A batch at once and 16 sequences at a time (128 pairs: always the plain kernel): rings and states to the bit, outputs as far
    as sums in another order go (fp32: 4 ulp of a norm; bf16: ties of its rounding)."""
    print(f"N={N} D={D} W={W} {dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5900 + W)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    draw = lambda *shape: torch.randn(*shape, device="cuda", generator=gen).to(dt)
    pos = torch.randint(0, 4 * W, (N,), dtype=torch.int32, device="cuda", generator=gen)
    pos[:4] = torch.tensor([0, W - 1, W, 2 * W - 1], dtype=torch.int32)
    d = dict(q=draw(N, 16, D), k_new=draw(N, 8, D), v_new=draw(N, 8, D), pos=pos, k_ring=draw(N, 8, W, D), v_ring=draw(N, 8, W, D),
             state=draw(N, 8, D, D).float() / D)
    few = {m: t.clone() for m, t in d.items()}
    got = rb.rattn_decode_step(*(d[m] for m in NAMES), softmax_scale=D ** -0.5)
    want = torch.cat([rb.rattn_decode_step(*(few[m][i:i + 16] for m in NAMES), softmax_scale=D ** -0.5) for i in range(0, N, 16)])
    err = float((got.float() - want.float()).norm() / want.float().norm())
    assert err <= (2e-3 if dtype == "bf16" else 5e-7), err
    for m in ("k_ring", "v_ring", "state"):
        assert torch.equal(d[m], few[m]), m


@pytest.mark.parametrize("N,D,W,dtype", [(43, 64, 2933, "bf16"), (32, 128, 1500, "bf16"), (32, 128, 600, "f32")])
def test_large_steps_with_rings_around_the_caches_limit(N, D, W, dtype):
    """Rings that are filled as far as 128 MB of all pairs', one row less and one more, and hardly at all, in one step: those below
    are read through the caches, the others past them.  As above."""
    print(f"N={N} D={D} W={W} {dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5950 + W)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    draw = lambda *shape: torch.randn(*shape, device="cuda", generator=gen).to(dt)
    limit = ((128 << 20) // (8 * N) - 4 * D * D) // (2 * D * dt.itemsize)
    assert 2 < limit < W
    pos = torch.tensor([limit, limit - 1, limit + 1, 1, 0, 40, W - 1, W, 3 * W + 5], dtype=torch.int32, device="cuda").repeat(N)[:N]
    d = dict(q=draw(N, 16, D), k_new=draw(N, 8, D), v_new=draw(N, 8, D), pos=pos, k_ring=draw(N, 8, W, D), v_ring=draw(N, 8, W, D),
             state=draw(N, 8, D, D).float() / D)
    few = {m: t.clone() for m, t in d.items()}
    got = rb.rattn_decode_step(*(d[m] for m in NAMES), softmax_scale=D ** -0.5)
    want = torch.cat([rb.rattn_decode_step(*(few[m][i:i + 16] for m in NAMES), softmax_scale=D ** -0.5) for i in range(0, N, 16)])
    for n in range(N):   # (each sequence by itself: few keys in one ring, many in the next)
        err = float((got[n].float() - want[n].float()).norm() / want[n].float().norm())
        assert err <= (4e-3 if dtype == "bf16" else 1e-6), (int(pos[n]), err)
    for m in ("k_ring", "v_ring", "state"):
        assert torch.equal(d[m], few[m]), m
