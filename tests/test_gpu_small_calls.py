"""General kernels on few tokens: one chunk without states or chunks of 64 keys, four or eight waves per work-group, at the
edges of the rules that choose them."""
import math

import numpy as np
import pytest
import torch

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
