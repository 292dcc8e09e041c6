"""Calls on few tokens.  General kernels: one chunk without states or chunks of 64 keys, four or eight waves per work-group, at the
edges of the rules that choose them.  Chunked prefill: products shared between the forward and the hand-over."""
import math

import numpy as np
import pytest
import torch

import parity_metrics as pm

from oracle import rattn_oracle as orc
from paper_2506_15545_amd import binding as rb, synth

pytestmark = pytest.mark.gpu
np64 = lambda t: t.detach().cpu().to(torch.float64).numpy()


def launches(f):
    rb.rattn_profile_enable(True)
    out = f()
    torch.cuda.synchronize()
    names = [n for n, _ in rb.rattn_profile_records()]
    rb.rattn_profile_enable(False)
    return out, names


@pytest.mark.parametrize("D,phi", [(64, "softmax"), (128, "softmax"), (64, "relu")])
@pytest.mark.parametrize("B,T,Hq,Hkv,W,states", [
    (1, 65, 2, 1, 1, False), (1, 66, 2, 1, 1, False),        # one tile of keys more than the 64 of a default chunk
    (1, 352, 2, 2, 32, False), (1, 353, 2, 2, 32, True),     # 320 keys beyond the window, and one more
    (2, 256, 8, 4, 16, False), (2, 257, 8, 4, 16, True),     # 256 work-groups (eight waves), 272 (four; limit 224)
    (4, 256, 8, 4, 32, False), (4, 256, 8, 4, 31, True),     # 512 work-groups: 224 keys, and one more
    (4, 161, 16, 8, 33, False), (4, 162, 16, 8, 33, True),   # 704 work-groups: 128 keys, and one more
])
def test_one_chunk_or_states(B, T, Hq, Hkv, W, states, D, phi):
    """fp32 against fp64: sums of up to T + D terms of fp32 products, with features at most one (softmax) or a few (ReLU)."""
    x = synth.make_random_layer(B, T, Hq, Hkv, D, "f32", 5100 + T + D, with_dO=True, with_gains=True)
    scale = 1.0 / math.sqrt(D)
    print(f"B={B} T={T} Hq={Hq} Hkv={Hkv} D={D} W={W} {phi}", flush=True)
    q, k, v, dO, gs, gr = (x[n].cuda() for n in ("q", "k", "v", "dO", "gamma_swa", "gamma_rla"))
    kw = dict(softmax_scale=scale, feature_map=phi)
    (o, saved), fwd = launches(lambda: rb.rattn_fwd(q, k, v, W, gs, gr, save_for_bwd=True, **kw))
    grads, bwd = launches(lambda: rb.rattn_bwd(q, k, v, saved, dO, W, gs, gr, **kw))
    assert fwd == (["gen_chunk_kernel", "gen_scan_kernel"] if states else []) + ["gen_fwd_kernel"]
    assert ("gen_chunk_kernel(rev)" in bwd) == ("gen_scan_kernel(rev)" in bwd) == states
    okw = dict(scale=scale, gamma_swa=np64(gs), gamma_rla=np64(gr), feature_map=phi)
    args = tuple(np64(x[n]) for n in ("q", "k", "v"))
    want = {"o": orc.fwd_dense(*args, W, **okw)["o"], **orc.bwd_dense(*args, np64(dO), W, **okw)}
    for n, got in zip(("o", "dq", "dk", "dv", "dgamma_swa", "dgamma_rla"), (o,) + tuple(grads)):
        err = float(np.linalg.norm(np64(got) - want[n]) / np.linalg.norm(want[n]))
        print(f"{n}: {err:.2e}", flush=True)
        assert err <= 5e-6, n   # 2^-24 times a random walk over (T + D) terms and the two products in front of them


@pytest.mark.parametrize("B,T,Hq,Hkv,D,W,limit", [
    (1, 200, 2, 1, 64, 16, (1.24, 2.52, 2.58, 1.85)), (4, 256, 8, 4, 64, 32, (1.35, 2.66, 2.74, 2.06)), (4, 256, 8, 4, 128, 32, (1.62, 3.10, 3.17, 2.24)),
    (2, 200, 16, 4, 128, 16, (1.47, 2.79, 2.90, 2.06)), (4, 161, 16, 8, 64, 33, (1.39, 2.63, 2.72, 2.11))])
def test_one_chunk_rounds_no_more_than_states_did(B, T, Hq, Hkv, D, W, limit):
    """o, dq, dk and dv of calls whose keys form one chunk against fp64, in 1e-7 of the norm: not above what these inputs gave when
    the same calls went over states of 64 keys with products in two chains (a sum over the whole chunk in one chain is above)."""
    g = torch.Generator(device="cuda").manual_seed(5200 + T + D)
    q, k, v, dO = (torch.randn(B, T, h, D, device="cuda", generator=g) for h in (Hq, Hkv, Hkv, Hq))
    args, scale = tuple(np64(t) for t in (q, k, v)), D ** -0.5
    want = {"o": orc.fwd_dense(*args, W, scale=scale)["o"], **orc.bwd_dense(*args, np64(dO), W, scale=scale)}
    o, saved = rb.rattn_fwd(q, k, v, W, save_for_bwd=True, softmax_scale=scale)
    got = (o,) + rb.rattn_bwd(q, k, v, saved, dO, W, want_dgamma=False, softmax_scale=scale)[:3]
    err = [1e7 * float(np.linalg.norm(np64(x) - want[n]) / np.linalg.norm(want[n])) for n, x in zip(("o", "dq", "dk", "dv"), got)]
    print("errors %.3f %.3f %.3f %.3f" % tuple(err), flush=True)
    assert all(e <= lim for e, lim in zip(err, limit))


SHARED = ["chunk_products_kernel", "chunk_scan_kernel", "fwd_fused_kernel"]


@pytest.mark.parametrize("phi", ["softmax", "relu"])
@pytest.mark.parametrize("B,Hq,Hkv,W,chunks", [
    (1, 4, 4, 128, [384, 128, 127, 513]),     # no ring yet; whole tiles; one row less
    (2, 8, 4, 64, [65, 191, 64, 300]),        # a ring of half a tile, rows in front of it, states at the 64 alignment
    (1, 8, 8, 100, [150, 90, 70, 129]),       # window off the 64 grid: up to 63 keys more leave than the states hold
    (1, 8, 8, 513, [300, 250, 333, 64]),      # ring filled over several calls, then wrapping
    (3, 8, 8, 129, [257, 1100]),              # more than 128 whole products: 128 keys each
    (1, 16, 16, 8, [140, 1000]),
    (1, 3, 1, 128, [384, 128, 127, 513]),     # one sequence of one KV head
    (1, 2, 2, 200, [1800, 1]),                # more than 12 products in a chain: 128 keys each; one token
])
def test_chunk_products_shared_with_the_hand_over(B, Hq, Hkv, W, chunks, phi):
    """Chunked prefill whose forward states and carried state come out of the same products, at the edges of its plan, against
    the oracle's rows of one forward and its export: outputs to the bf16 bound, rings to the bit, the state to fp32."""
    D, T = 128, sum(chunks)
    x = synth.make_random_layer(B, T, Hq, Hkv, D, "bf16", 5300 + T + W, with_gains=True)
    scale = 1.0 / math.sqrt(D)
    gs, gr = x["gamma_swa"], x["gamma_rla"]
    ref = orc.fwd_dense(np64(x["q"]), np64(x["k"]), np64(x["v"]), W, scale=scale, gamma_swa=np64(gs), gamma_rla=np64(gr),
                        feature_map=phi)["o"]
    q, k, v = (x[n].cuda() for n in ("q", "k", "v"))
    kr, vr = (torch.full((B, Hkv, W, D), float("nan"), dtype=q.dtype, device="cuda") for _ in range(2))
    S = torch.full((B, Hkv, D, D), float("nan"), dtype=torch.float32, device="cuda")
    gmax = max(float(gs.abs().max()), float(gr.abs().max()), 1.0)
    pos0 = 0
    for n in chunks:
        print(f"B={B} Hkv={Hkv} W={W} {phi}: tokens {pos0}..{pos0 + n - 1}", flush=True)
        sl = slice(pos0, pos0 + n)
        o, names = launches(lambda: rb.rattn_prefill_chunk(
            q[:, sl].contiguous(), k[:, sl].contiguous(), v[:, sl].contiguous(), W, pos0, kr, vr, S, gs.cuda(), gr.cuda(),
            softmax_scale=scale, feature_map=phi))
        ring = min(pos0, W)
        tiles = -(-ring // 128) + -(-n // 128)
        shared = ring + n > W and tiles > -(-(-(-W // 64) * 64) // 128)
        assert (names == SHARED) == shared, names
        pm.assert_out_bf16(np64(o), ref[:, sl], gmax, what=f"chunk at {pos0}")
        pos0 += n
        kr_ref, vr_ref, S_ref = orc.prefill_export(np64(x["k"])[:, :pos0], np64(x["v"])[:, :pos0], W, feature_map=phi)
        m = min(pos0, W)   # slots that hold tokens
        assert np.array_equal(np64(kr)[:, :, :m], kr_ref[:, :, :m]) and np.array_equal(np64(vr)[:, :, :m], vr_ref[:, :, :m])
        if pos0 > W:
            assert float(np.max(np.abs(np64(S) - S_ref))) <= 2e-5 * max(1.0, float(np.abs(S_ref).max()))


@pytest.mark.parametrize("B,T,Hkv,W,pos0", [(1, 2048, 2, 129, 4000), (1, 1300, 2, 300, 9000), (4, 2048, 8, 512, 2048), (1, 700, 8, 512, 1531)])
def test_carried_state_of_shared_products_in_fp32(B, T, Hkv, W, pos0):
    """The state after a chunk against fp64, to what sums of 64 keys each (where every CU has two such products: 128), added in runs
    of a quarter of them, leave: measured on these inputs 1.03e-7, 8.5e-8, 1.21e-7 and 9.1e-8 of the norm.  (One chain per 128 keys
    and one over the products: 1.26e-7, 1.20e-7, 1.37e-7, 1.04e-7.)"""
    D = 128
    g = torch.Generator(device="cuda").manual_seed(5450 + T)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v = (r(B, T, Hkv, D).bfloat16() for _ in range(3))
    kr, vr = (r(B, Hkv, W, D).bfloat16() for _ in range(2))
    S = r(B, Hkv, D, D) * math.sqrt((pos0 - W) * math.e) / D
    slots = [(pos0 + i) % W for i in range(W)]
    rows = [torch.cat([ring[:, :, slots], x.transpose(1, 2)], 2)[:, :, :T].double() for ring, x in ((kr, k), (vr, v))]
    want = S.double() + torch.softmax(rows[0], -1).transpose(-1, -2) @ rows[1]
    _, names = launches(lambda: rb.rattn_prefill_chunk(q, k, v, W, pos0, kr, vr, S, softmax_scale=0.09))
    assert names == SHARED
    err = float((S.double() - want).norm() / want.norm())
    print(f"{err:.3e}", flush=True)
    assert err <= {4000: 1.03e-7, 9000: 8.5e-8, 2048: 1.21e-7, 1531: 9.1e-8}[pos0] * 1.01   # (inputs differ by 0.5 % at most)


@pytest.mark.parametrize("B,Hkv", [(1, 1), (1, 4), (2, 2)])
def test_chunk_products_of_infinite_values(B, Hkv):
    """An infinite value of one key, met by features of both kinds of zero, reaches its own column of the carried state only: the
    oracle's state of the whole sequence, which has that column and finite values otherwise."""
    D, W, pos0, n = 128, 128, 200, 256
    x = synth.make_random_layer(B, pos0 + n, Hkv, Hkv, D, "bf16", 5400)
    x["v"][0, 250, Hkv - 1, 7] = float("inf")
    q, k, v = (x[m].cuda() for m in ("q", "k", "v"))
    kr, vr, S = rb.rattn_prefill_export(k[:, :pos0].contiguous(), v[:, :pos0].contiguous(), W)
    _, names = launches(lambda: rb.rattn_prefill_chunk(q[:, pos0:].contiguous(), k[:, pos0:].contiguous(), v[:, pos0:].contiguous(),
                                                       W, pos0, kr, vr, S, softmax_scale=0.09))
    assert names == SHARED
    want = orc.prefill_export(np64(x["k"]), np64(x["v"]), W)[2]
    got, fin = np64(S), np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin) and int((~fin).sum()) == D and bool((got[~fin] == np.inf).all())
    assert float(np.abs(got[fin] - want[fin]).max()) <= 2e-5 * max(1.0, float(np.abs(want[fin]).max()))


@pytest.mark.parametrize("phi", ["softmax", "relu"])
@pytest.mark.parametrize("B,T,Hq,Hkv,D,W,products", [
    (1, 256, 2, 1, 128, 100, 0), (2, 384, 4, 2, 128, 128, 1), (1, 384, 3, 3, 64, 190, 1),      # state 0 alone; one more
    (1, 400, 4, 2, 128, 130, 2), (2, 512, 2, 1, 64, 65, 3), (1, 639, 4, 4, 128, 128, 3),      # states at the 64 alignment; three
    (1, 641, 4, 4, 128, 128, 4), (65, 640, 1, 1, 64, 128, 3),                                 # two launches: four products, 65 pairs
])
def test_states_of_few_products(B, T, Hq, Hkv, D, W, products, phi):
    """Forward states out of one launch (few products) or two: outputs and gradients against the general kernels, which form
    them in fp32, at the bound of two bf16 paths; at least the last state is read by a query tile of every case."""
    x = synth.make_random_layer(B, T, Hq, Hkv, D, "bf16", 5500 + T + W, with_dO=True)
    q, k, v, dO = (x[n].cuda() for n in ("q", "k", "v", "dO"))
    print(f"B={B} T={T} Hq={Hq} Hkv={Hkv} D={D} W={W} {phi}", flush=True)
    one = products <= (3 if B * Hkv <= 64 else 2)
    got = {}
    for path in ("auto", "general"):
        kw = dict(softmax_scale=1.0 / math.sqrt(D), kernel_path=path, feature_map=phi)
        (o, saved), names = launches(lambda: rb.rattn_fwd(q, k, v, W, save_for_bwd=True, **kw))
        got[path] = (o,) + rb.rattn_bwd(q, k, v, saved, dO, W, want_dgamma=False, **kw)[:3]
        if path == "auto":
            assert names == (["rla_walk_kernel"] if one else ["rla_chunk_kernel", "rla_scan_kernel"]) + ["fwd_fused_kernel"]
    for n, a, b in zip(("o", "dq", "dk", "dv"), got["auto"], got["general"]):
        rel = float((a.double() - b.double()).norm() / b.double().norm())
        print(f"{n}: {rel:.2e}", flush=True)
        assert rel <= 1e-2, n   # bf16 operands: 2^-9 per factor and term


@pytest.mark.parametrize("phi", ["softmax", "relu"])
@pytest.mark.parametrize("B,T,Hq,Hkv,D,W", [(2, 384, 4, 2, 128, 128), (1, 400, 4, 2, 128, 130), (2, 512, 2, 1, 64, 65), (1, 639, 4, 4, 128, 128)])
def test_states_of_one_launch_or_two_are_the_same_bits(B, T, Hq, Hkv, D, W, phi):
    """One, two and three products: a forward that forms all states in one launch and one whose states are kept by halves, which
    takes two."""
    x = synth.make_random_layer(B, T, Hq, Hkv, D, "bf16", 5500 + T + W)
    q, k, v = (x[n].cuda() for n in ("q", "k", "v"))
    got = {}
    for policy in ("keep", "every2"):
        (got[policy], _), names = launches(lambda: rb.rattn_fwd(q, k, v, W, softmax_scale=1.0 / math.sqrt(D), save_for_bwd=True,
                                                                feature_map=phi, state_policy=policy))
        assert names == (["rla_walk_kernel"] if policy == "keep" else ["rla_chunk_kernel", "rla_scan_kernel"]) + ["fwd_fused_kernel"]
    assert torch.equal(got["keep"], got["every2"])


@pytest.mark.parametrize("B,Hkv,D,dtype,W,out,launched", [
    (2, 3, 128, "bf16", 100, 0, 1), (2, 3, 64, "f32", 100, 0, 1), (1, 2, 128, "bf16", 64, -20, 1),   # nothing leaves the window
    (2, 3, 128, "bf16", 50, 1, 1), (2, 3, 128, "bf16", 50, 64, 1), (2, 3, 128, "bf16", 50, 65, 2),
    (16, 4, 128, "bf16", 50, 128, 1), (16, 4, 128, "bf16", 50, 129, 2), (16, 8, 64, "bf16", 20, 320, 1), (16, 8, 64, "bf16", 20, 321, 2),
    (16, 8, 128, "bf16", 20, 320, 1), (16, 8, 128, "bf16", 20, 321, 2), (2, 3, 64, "bf16", 50, 192, 1), (2, 3, 64, "bf16", 50, 193, 2),
    (1, 2, 64, "f32", 30, 64, 2), (1, 2, 64, "f32", 30, 65, 3), (1, 2, 128, "f32", 30, 64, 2), (1, 2, 128, "f32", 30, 65, 3)])
@pytest.mark.parametrize("phi", ["softmax", "identity"])
def test_export_of_few_keys(B, Hkv, D, dtype, W, out, launched, phi):
    """Prefill export with no key, few keys and one more beyond the window: rings to the bit, the state to fp32, buffers that hold
    noise before."""
    T = W + out
    x = synth.make_random_layer(B, T, Hkv, Hkv, D, dtype, 5600 + T)
    kr, vr = (torch.zeros(B, Hkv, W, D, dtype=x["k"].dtype, device="cuda") for _ in range(2))
    S = torch.full((B, Hkv, D, D), float("nan"), device="cuda")
    _, names = launches(lambda: rb.rattn_prefill_export(x["k"].cuda(), x["v"].cuda(), W, kr, vr, S, feature_map=phi))
    assert len(names) == launched, names
    kr_ref, vr_ref, S_ref = orc.prefill_export(np64(x["k"]), np64(x["v"]), W, feature_map=phi)
    assert np.array_equal(np64(kr), kr_ref) and np.array_equal(np64(vr), vr_ref)
    assert float(np.max(np.abs(np64(S) - S_ref))) <= 2e-5 * max(1.0, float(np.abs(S_ref).max()))


@pytest.mark.parametrize("phi", ["softmax", "relu", "identity"])
@pytest.mark.parametrize("B,Hkv,D,dtype,out", [
    (1, 2, 128, "bf16", 65), (1, 2, 128, "bf16", 128), (1, 2, 128, "bf16", 192), (16, 8, 128, "bf16", 256), (16, 8, 128, "bf16", 193),
    (1, 2, 64, "bf16", 256), (1, 2, 64, "bf16", 257), (1, 2, 64, "bf16", 320), (1, 2, 64, "f32", 65), (1, 2, 64, "f32", 128)])
def test_export_adds_sums_of_64_keys(B, Hkv, D, dtype, out, phi):
    """However many launches: the state is the sum of the states of its tiles of 64 keys in order (five tiles of few pairs: by
    twos), to the bit.  One chain of products over all keys is further from fp64 (320 keys at D = 64: 1.9e-7 of the norm, 1.1e-7)."""
    W = 8
    x = synth.make_random_layer(B, out + W, Hkv, Hkv, D, dtype, 5650 + out)
    k, v = x["k"].cuda(), x["v"].cuda()
    state = lambda a, b: rb.rattn_prefill_export(k[:, a:b + W].contiguous(), v[:, a:b + W].contiguous(), W, feature_map=phi)[2]
    got = state(0, out)
    tiles = [state(a, min(a + 64, out)) for a in range(0, out, 64)]
    if len(tiles) > 4:
        tiles = [sum(tiles[i:i + 2]) for i in range(0, len(tiles), 2)]
    assert torch.equal(got, sum(tiles))


def test_export_of_infinite_values_in_pieces():
    """An infinite value reaches the column of its own feature only, and only through the keys that hold it."""
    D, W, out = 128, 8, 128
    x = synth.make_random_layer(1, out + W, 2, 2, D, "bf16", 5660)
    plain = rb.rattn_prefill_export(x["k"].cuda(), x["v"].cuda(), W)[2]
    x["v"][0, 70, 1, 7] = float("inf")
    S = rb.rattn_prefill_export(x["k"].cuda(), x["v"].cuda(), W)[2]
    assert bool((S[0, 1, :, 7] == float("inf")).all())
    S[0, 1, :, 7] = plain[0, 1, :, 7]
    assert torch.equal(S[0, 0], plain[0, 0]) and float((S - plain).abs().max()) <= 1e-6 * float(plain.abs().max())
