"""Workloads of the layer library, as a user's program runs them: training steps, prompt prefill with the hand-over to
decoding, chunked prefill, and decode steps.

A case is a dict of plain values; `kind` names what the program does:

  train    rattn_fwd(save_for_bwd) followed by rattn_bwd, as in every layer of a training step
  prompt   rattn_fwd over a whole prompt, then rattn_prefill_export (rings and state for the decode steps to come)
  chunk    rattn_prefill_chunk: the next T tokens of sequences whose first pos0 tokens are rings and state
  decode   rattn_decode_step: one new token for each of N sequences

Buffers that such a program keeps (outputs, `saved`, the workspaces the calls take) are made once in prepare().
"""
import math

import torch

from paper_2506_15545_amd import binding as rb

NOMINAL_CHUNK = 64   # linear-branch chunk of the FLOP count (the benchmark's formula)
EPS = 1e-6


def _layer(name, kind, B, T, Hq, Hkv, D, W, dtype="bf16", gains=True, pos0=0):
    return dict(name=name, kind=kind, B=B, T=T, Hq=Hq, Hkv=Hkv, D=D, W=W, dtype=dtype, gains=gains, pos0=pos0)


def _decode(name, N, Hq, Hkv, D, W, pos_lo, pos_hi, dtype="bf16", gains=True):
    return dict(name=name, kind="decode", N=N, Hq=Hq, Hkv=Hkv, D=D, W=W, pos_lo=pos_lo, pos_hi=pos_hi, dtype=dtype,
                gains=gains)


def listed():
    return [
        # the smallest call: one sequence being generated interactively (16 query / 4 KV heads, the 3B layer of Table 1)
        _decode("decode_one", 1, 16, 4, 128, 512, 2000, 2000),
        # batch serving: the decode benchmark's step
        _decode("decode_batch", 128, 32, 8, 128, 512, 512, 32768, gains=False),
        # a moderate batch on the 12B layer of Table 1 (40 query / 8 KV heads) with a wider window, half of the
        # sequences still inside it
        _decode("decode_wide", 24, 40, 8, 128, 2048, 100, 4000),
        # one prompt of ordinary, ragged length, then the hand-over to decoding
        _layer("prompt_ragged", "prompt", 1, 3001, 16, 4, 128, 512),
        # a long document with the wide window of the sweep
        _layer("prompt_long", "prompt", 1, 32768, 24, 8, 128, 4096, gains=False),
        # chunked prefill of a batch at aligned positions, as the benchmark does it
        _layer("chunk_aligned", "chunk", 4, 2048, 24, 8, 128, 512, gains=False, pos0=2048),
        # the remainder of a prompt after a prefix of arbitrary length (a follow-up turn of a conversation)
        _layer("chunk_ragged", "chunk", 1, 700, 32, 8, 128, 512, pos0=1531),
        # the smallest fp32 configuration (numerical checks, small experiments), as a training step
        _layer("train_f32", "train", 1, 256, 2, 2, 64, 32, dtype="f32", gains=False),
        # short ragged sequences with the paper's window of w = 512 earlier tokens (513 with the current one)
        _layer("train_ragged", "train", 2, 1000, 16, 4, 128, 513),
        # the headline layer
        _layer("train_3b", "train", 4, 4096, 24, 8, 128, 512, gains=False),
        # the same layer at head size 64
        _layer("train_d64", "train", 4, 4096, 24, 8, 64, 512),
        # the 12B-scale layer, with gains and their gradients
        _layer("train_12b", "train", 2, 8192, 32, 8, 128, 512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tf(case):
    return work(case)["flops"] / 1e12


def draw(rng):
    kind = rng.choice(["decode"] * 3 + ["prompt"] * 2 + ["chunk"] * 2 + ["train"] * 4)
    Hkv, G = rng.choice([(8, 3), (8, 4), (8, 5), (4, 4), (4, 2), (2, 8), (2, 1), (8, 1)])
    D = rng.choice([128, 128, 128, 64])
    gains = rng.random() < 0.6
    if kind == "decode":
        W = _log_int(rng, 64, 4096)
        N = max(1, min(_log_int(rng, 1, 128), int(1.3e8 / (2 * W * Hkv * D))))
        hi = _log_int(rng, 64, 32768)
        return dict(kind="decode", N=N, Hq=Hkv * G, Hkv=Hkv, D=D, W=W, pos_lo=rng.randrange(1, hi), pos_hi=hi,
                    dtype=rng.choice(["bf16"] * 4 + ["f32"]), gains=gains)
    f32 = kind == "train" and rng.random() < 0.25
    if f32:    # numerical checks and small experiments
        Hkv, G = rng.choice([(2, 1), (1, 2), (2, 2)])
        B, T, W = rng.choice([1, 2]), _log_int(rng, 64, 512), _log_int(rng, 16, 128)
    elif kind == "chunk":
        B, T, W = _log_int(rng, 1, 4), _log_int(rng, 64, 2048), _log_int(rng, 32, 2048)
    else:
        B, T, W = _log_int(rng, 1, 4), _log_int(rng, 128, 8192), _log_int(rng, 32, 2048)
    if rng.random() < 0.4:   # aligned sizes are as common as odd ones
        W, T = (W + 63) // 64 * 64, (T + 127) // 128 * 128
    case = dict(kind=kind, B=B, T=T, Hq=Hkv * G, Hkv=Hkv, D=D, W=W, dtype="f32" if f32 else "bf16", gains=gains,
                pos0=_log_int(rng, 32, 16384) if kind == "chunk" else 0)
    if kind == "chunk" and rng.random() < 0.4:
        case["pos0"] = (case["pos0"] + 127) // 128 * 128
    # no more work than the training layers' steps; chunks at head size 64 belong to small models
    while _tf(case) > 0.4 or (kind == "chunk" and D == 64 and case["B"] * case["T"] * case["Hq"] > 65536):
        if case["B"] > 1:
            case["B"] -= 1
        else:
            case["T"] = case["T"] * 2 // 3
    return case


def _scale(D):
    return 1.0 / math.sqrt(D)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[case["dtype"]]

    def normal(*shape, dtype=dt):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)

    Hq, Hkv, D, W = case["Hq"], case["Hkv"], case["D"], case["W"]
    s = {"case": case, "gs": None, "gr": None}
    if case["gains"]:
        s["gs"], s["gr"] = (1.0 + 0.1 * normal(Hq, D, dtype=torch.float32) for _ in range(2))

    def cache(N, pos):   # rings and state of N sequences at positions pos (see synth.make_decode_inputs)
        s["k_ring"], s["v_ring"] = normal(N, Hkv, W, D), normal(N, Hkv, W, D)
        std = torch.sqrt(torch.clamp(pos.float() - W, min=0.0) * math.e) / D
        s["state"] = normal(N, Hkv, D, D, dtype=torch.float32) * std.view(N, 1, 1, 1)

    if case["kind"] == "decode":
        N = case["N"]
        s["q"], s["k"], s["v"] = normal(N, Hq, D), normal(N, Hkv, D), normal(N, Hkv, D)
        s["pos"] = torch.randint(case["pos_lo"], case["pos_hi"] + 1, (N,), generator=g, device="cuda", dtype=torch.int32)
        cache(N, s["pos"])
        s["o"] = torch.empty_like(s["q"])
        return s

    B, T = case["B"], case["T"]
    s["q"], s["k"], s["v"] = normal(B, T, Hq, D), normal(B, T, Hkv, D), normal(B, T, Hkv, D)
    s["o"] = torch.empty_like(s["q"])
    if case["kind"] == "chunk":
        cache(B, torch.full((B,), case["pos0"], device="cuda"))
        return s
    train = case["kind"] == "train"
    p = rb.make_params(s["q"], s["k"], W, 0, _scale(D), EPS, train)
    fwd, bwd, saved = rb.rattn_workspace_bytes(p)
    s["ws"] = torch.empty(max(fwd, bwd if train else 0, 16), dtype=torch.uint8, device="cuda")
    if train:
        s["dO"] = normal(B, T, Hq, D)
        s["saved"] = torch.empty(max(saved, 16), dtype=torch.uint8, device="cuda")
        s["grads"] = tuple(torch.empty_like(s[n]) for n in "qkv")
    else:
        s["k_ring"], s["v_ring"] = (torch.zeros(B, Hkv, W, D, dtype=dt, device="cuda") for _ in range(2))
        s["state"] = torch.empty(B, Hkv, D, D, dtype=torch.float32, device="cuda")
    return s


def run(s):
    case = s["case"]
    W, scale = case["W"], _scale(case["D"])
    if case["kind"] == "decode":
        o = rb.rattn_decode_step(s["q"], s["k"], s["v"], s["pos"], s["k_ring"], s["v_ring"], s["state"], s["gs"], s["gr"],
                                 softmax_scale=scale, out=s["o"])
        return {"o": o, "k_ring": s["k_ring"], "v_ring": s["v_ring"], "state": s["state"]}
    if case["kind"] == "chunk":
        o = rb.rattn_prefill_chunk(s["q"], s["k"], s["v"], W, case["pos0"], s["k_ring"], s["v_ring"], s["state"], s["gs"],
                                   s["gr"], softmax_scale=scale, out=s["o"])
        return {"o": o, "k_ring": s["k_ring"], "v_ring": s["v_ring"], "state": s["state"]}
    if case["kind"] == "prompt":
        o = rb.rattn_fwd(s["q"], s["k"], s["v"], W, s["gs"], s["gr"], softmax_scale=scale, out=s["o"], workspace=s["ws"])
        kr, vr, state = rb.rattn_prefill_export(s["k"], s["v"], W, s["k_ring"], s["v_ring"], s["state"])
        return {"o": o, "k_ring": kr, "v_ring": vr, "state": state}
    o, saved = rb.rattn_fwd(s["q"], s["k"], s["v"], W, s["gs"], s["gr"], softmax_scale=scale, save_for_bwd=True,
                            out=s["o"], saved=s["saved"], workspace=s["ws"])
    dq, dk, dv, dgs, dgr = rb.rattn_bwd(s["q"], s["k"], s["v"], saved, s["dO"], W, s["gs"], s["gr"], softmax_scale=scale,
                                        want_dgamma=case["gains"], workspace=s["ws"], out=s["grads"])
    return {"o": o, "dq": dq, "dk": dk, "dv": dv, "dgs": dgs, "dgr": dgr}


def _pairs(T, W, pos0):
    """In-window (query, key) pairs of queries pos0 .. pos0+T-1, and how many of them have keys beyond the window."""
    upto = lambda n: n * (n + 1) // 2 if n <= W else W * n - W * (W - 1) // 2
    return upto(pos0 + T) - upto(pos0), max(pos0 + T - max(W, pos0), 0)


def work(case):
    Hq, Hkv, D, W = case["Hq"], case["Hkv"], case["D"], case["W"]
    e = 4 if case["dtype"] == "f32" else 2
    gains = 2 * Hq * D * 4 if case["gains"] else 0
    if case["kind"] == "decode":
        N, lo, hi = case["N"], case["pos_lo"], case["pos_hi"]
        n = hi - lo + 1                                   # mean of min(pos + 1, W) over pos in lo .. hi
        k = max(0, min(hi, W - 1) - lo + 1)
        valid = (k * (2 * lo + k + 1) / 2 + (n - k) * W) / n
        evict = (n - k) / n                               # share of the sequences that fold a key into the state
        nbytes = N * (2 * Hkv * valid * D * e + 2 * Hkv * D * D * 4 * evict + (2 * Hq + 4 * Hkv) * D * e) + gains
        flops = N * (Hq * 4 * D * valid + evict * (2 * Hq + 2 * Hkv) * D * D)
        return {"bytes": nbytes, "flops": flops}
    B, T, pos0 = case["B"], case["T"], case["pos0"]
    P, Tr = _pairs(T, W, pos0)
    fwd = B * Hq * (4 * D * P + 2 * Tr * D * D + 4 * D * Tr * (NOMINAL_CHUNK + 1) // 2) + B * Hkv * 2 * Tr * D * D
    qo, kv, ring, state = B * T * Hq * D * e, B * T * Hkv * D * e, B * Hkv * W * D * e, B * Hkv * D * D * 4
    if case["kind"] == "train":
        bwd = B * Hq * (10 * D * P + 4 * Tr * D * D + 10 * D * Tr * (NOMINAL_CHUNK + 1) // 2) + B * Hkv * 4 * Tr * D * D
        # q, k, v, dO in; o, dq, dk, dv out
        return {"bytes": 4 * qo + 4 * kv + 2 * gains, "flops": fwd + bwd}
    if case["kind"] == "prompt":   # the state of the decode steps is one more row of chunk products
        return {"bytes": 2 * qo + 2 * kv + gains + 2 * min(1.0, T / W) * ring + state, "flops": fwd}
    seen, new = min(pos0, W), min(T, W)
    return {"bytes": 2 * qo + 2 * kv + gains + 2 * (seen + new) / W * ring + (2 if pos0 > W else 1) * state, "flops": fwd}


def tolerance(case):
    # bf16: operands, probabilities and results are rounded to 8 bits (gradients of single elements by up to a tenth of
    # the tensor's RMS, where they are differences of larger terms); fp32: sums of up to 10^4 terms
    return {"rel": 1e-2, "max": 0.2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}
