"""What a training or serving program asks of this library, as cases to measure.

A case is one pass over one packed stream (or, `new_bin`, over one freshly packed bin):

  step       bf16 forward and backward: one attention layer of a training step
  forward    bf16 forward alone: evaluation and serving (prefill; the mask hides nothing a decoder would not)
  fp8        Q, K, V quantised on the device with per-head scales, then the FP8 forward
  fp8_block  the same with block-wise scales
  new_bin    first-fit packing of a pool of sample lengths, layout and work lists of the first bin, then forward
             and backward on it: what the first layer of every step pays

The sample lengths of a case follow from its `rule`, `pool`, `budget` and `lengths` (a seed); the tensors are
standard normal draws rounded to bfloat16, as in the library's workloads.
"""
import functools
import math

import numpy as np
import torch

from paper_2603_11101_amd import binding as va

MASKS = {
    "causal": va.VA_MASK_CAUSAL,
    "prefix": va.VA_MASK_PREFIX_LM,
    "prefix_causal": va.VA_MASK_PREFIX_LM_CAUSAL,
    "three_block": va.VA_MASK_THREE_BLOCK,
    "window": va.VA_MASK_SLIDING_WINDOW,
}


def _case(kind, rule, lengths, pool, budget, hq, hkv, d, mask, window=0, name=None):
    c = {"kind": kind, "rule": rule, "lengths": lengths, "pool": pool, "budget": budget, "hq": hq, "hkv": hkv, "d": d,
         "mask": mask, "window": window}
    return dict(c, name=name) if name else c


def listed():
    return [
        # configuration 1: a handful of short samples; all latency: host path, launches, kernel start
        _case("step", "tiny", 1, 3, 176, 2, 2, 64, "causal", name="tiny_step"),
        # serving a policy: one observation (three cameras, an instruction) through one layer, batch 1
        _case("forward", "pi05", 11, 1, 1100, 8, 1, 256, "prefix", name="one_observation_forward"),
        # fine-tuning with a small micro-batch: five camera samples on one GPU
        _case("step", "vlm", 12, 5, 4096, 16, 8, 128, "causal", name="micro_batch_step"),
        # configuration 2: the vision-language backbone's packed 16k batch
        _case("step", "vlm", 2, 512, 16384, 16, 8, 128, "causal", name="vlm_step"),
        # configuration 3: bidirectional prefix, one KV head for eight query heads, the widest heads
        _case("step", "pi05", 3, 512, 32768, 8, 1, 256, "prefix", name="pi05_step"),
        # configuration 4: heavy-tailed lengths, 64k tokens
        _case("step", "longtail", 4, 2048, 65536, 16, 8, 128, "causal", name="longtail_step"),
        # configuration 5: FP8 forward on the batch of configuration 2, quantisation included
        _case("fp8", "vlm", 2, 512, 16384, 16, 8, 128, "causal", name="vlm_fp8"),
        # the finest scales on the large batch
        _case("fp8_block", "longtail", 4, 2048, 65536, 16, 8, 128, "causal", name="longtail_fp8_block"),
        # the vision encoder: every patch sees its image, head dimension between two tile geometries
        _case("step", "vit", 5, 512, 16384, 16, 16, 80, "prefix", name="vit_step"),
        # evaluation of a flow-matching policy: prefix, state token, actions
        _case("forward", "pi0", 6, 512, 32768, 8, 1, 256, "three_block", name="pi0_forward"),
        # long contexts with a bounded horizon
        _case("step", "long", 9, 4, 65536, 16, 8, 128, "window", 1024, name="window_step"),
        # every step of a training run brings a new bin: pool to gradients
        _case("new_bin", "longtail", 4, 2048, 65536, 16, 8, 128, "causal", name="new_bin_step"),
    ]


def _pool(c):
    """Sample lengths of the pool and block ends (None, [pool] or [pool, 2]) by the case's rule."""
    r, n = np.random.default_rng(c["lengths"]), c["pool"]
    rule, ends = c["rule"], None
    if rule == "tiny":
        lens = np.array([17, 64, 95]) if c["lengths"] == 1 else r.integers(1, 200, size=n)
    elif rule == "vlm":  # 1 to 3 cameras of 256 tokens, text, 17 state and action tokens
        cams = r.integers(1, 4, size=n)
        lens = 256 * cams + r.integers(10, 61, size=n) + 17
    elif rule in ("pi05", "pi0"):  # three cameras and text, (a state token,) 50 action tokens
        prefix = 768 + r.integers(20, 201, size=n)
        lens, ends = (prefix + 50, prefix) if rule == "pi05" else (prefix + 51, np.stack([prefix, prefix + 1], axis=1))
    elif rule == "vit":  # square images
        lens = r.choice(np.array([16, 24, 32, 38]), size=n) ** 2
        ends = lens
    elif rule == "longtail":
        lens = np.clip(np.rint(np.exp(np.log(600.0) + 0.8 * r.standard_normal(n))), 16, 4096)
    else:  # long: few samples that fill the budget
        lens = np.full(n, c["budget"] // n) - r.integers(0, max(1, c["budget"] // n // 16), size=n)
    lens = lens.astype(np.int32)
    if c["mask"] == "window":
        ends = np.full(n, c["window"])
    elif c["mask"] == "prefix_causal":
        ends = (lens * r.uniform(0.5, 0.95, size=n)).astype(np.int32)
    return lens, None if ends is None or c["mask"] == "causal" else ends.astype(np.int32)


def _first_bin(lens, ends, budget):
    """Packs the pool and lays out its first bin, as a data loader does."""
    bin_of, pos, _ = va.va_pack_first_fit(lens, budget)
    members = np.flatnonzero(bin_of == 0)  # placement order is arrival order
    cu, pl, longest = va.va_bin_layout(lens[members], None if ends is None else ends[members])
    return bin_of, pos, members, cu, pl, longest


def _layout(c):
    lens, ends = _pool(c)
    bin_of, _, members, cu, pl, longest = _first_bin(lens, None if c["mask"] == "window" else ends, c["budget"])
    return cu, ends[members] if c["mask"] == "window" else pl, longest


def _pairs(c):
    """Visible (query, key) pairs of the first bin, per head."""
    cu, pl, _ = _layout(c)
    L = np.diff(cu).astype(np.int64)
    if c["mask"] == "causal":
        return int((L * (L + 1) // 2).sum())
    P = pl.astype(np.int64)
    if c["mask"] == "prefix":
        return int((P * P + (L - P) * L).sum())
    if c["mask"] == "prefix_causal":
        return int((P * P + (L * (L + 1) - P * (P + 1)) // 2).sum())
    if c["mask"] == "three_block":
        return int((P[:, 0] ** 2 + (P[:, 1] - P[:, 0]) * P[:, 1] + (L - P[:, 1]) * L).sum())
    W = np.minimum(P, L)
    return int((W * (W + 1) // 2 + (L - W) * W).sum())


def work(case):
    T, D, hq, hkv = int(_layout(case)[0][-1]), case["d"], case["hq"], case["hkv"]
    products = 14 if case["kind"] in ("step", "new_bin") else 4
    flops = products * D * hq * _pairs(case)
    if case["kind"] in ("step", "new_bin"):  # Q, K, V, dO in; O, LSE, dQ, dK, dV out
        nbytes = 2 * T * D * (4 * hq + 4 * hkv) + 4 * T * hq
    else:  # Q, K, V in; O, LSE out
        nbytes = 2 * T * D * (2 * hq + 2 * hkv) + 4 * T * hq
    if case["kind"] == "fp8":  # and the codes and scales
        nbytes += T * D * (hq + 2 * hkv) + 4 * (hq + 2 * hkv)
    elif case["kind"] == "fp8_block":
        nbytes += T * (D + 4) * (hq + 2 * hkv)
    return {"bytes": nbytes, "flops": flops}


@functools.lru_cache(maxsize=None)
def _largest():
    w = [work(c) for c in listed()]
    return {k: max(x[k] for x in w) for k in w[0]}


def draw(rng):
    """A case from the same ranges: the kinds, masks and head shapes of the list (and the ones between them), from a
    hundred tokens to the largest bin, over the logarithm."""
    kind = rng.choice(["step", "step", "step", "forward", "fp8", "fp8_block", "new_bin"])
    rule = rng.choice(["tiny", "vlm", "vlm", "pi05", "pi0", "vit", "longtail", "longtail", "long"])
    low = {"tiny": 128, "long": 2048}.get(rule, 1500)
    high = {"tiny": 8192}.get(rule, 65536)
    budget = int(math.exp(rng.uniform(math.log(low), math.log(high))))
    mask, window = {"pi05": "prefix", "pi0": "three_block", "vit": "prefix"}.get(rule, "causal"), 0
    if rule in ("tiny", "longtail") and rng.random() < 0.25:
        mask = "prefix_causal"
    elif rule == "long" or (rule == "longtail" and rng.random() < 0.25):
        mask, window = "window", int(math.exp(rng.uniform(math.log(64), math.log(4096))))
    heads = {"tiny": [(2, 2, 64), (4, 2, 64), (8, 8, 64), (8, 1, 128)],
             "pi05": [(8, 1, 256)], "pi0": [(8, 1, 256)],
             "vit": [(16, 16, 80), (16, 16, 64), (12, 12, 64)]}.get(
                 rule, [(16, 8, 128), (16, 8, 128), (32, 8, 128), (16, 2, 128), (16, 16, 64), (8, 4, 96), (8, 4, 256)])
    if kind in ("fp8", "fp8_block"):
        heads = [h for h in heads if h[2] in (64, 128, 256)]
    hq, hkv, d = rng.choice(heads)
    pool = rng.randint(1, 4) if rule == "long" else max(2, 2 * budget // (100 if rule == "tiny" else 400))
    if rule == "vlm" and budget < 6000:  # micro-batches of a few whole samples
        pool = rng.randint(1, 6)
        budget = 900 * pool
    c = _case(kind, rule, rng.randrange(2, 1 << 20), pool, budget, hq, hkv, d, mask, window)
    top = _largest()
    if rule == "longtail":
        c["budget"] = max(c["budget"], 4096)
    while any(v > top[k] for k, v in work(c).items()):
        c["budget"] = max(4096, c["budget"] // 2)
        if rule == "long":
            c["pool"] = min(4, c["pool"] * 2)
    return c


def prepare(case, seed):
    """Tensors in the model's layout, output buffers, and the bin's plan (except where the pass makes it)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    cu, pl, longest = _layout(case)
    T = int(cu[-1])

    def normal(h):
        return torch.randn(T, h, d, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)

    s = {"case": case, "scale": d ** -0.5, "cu": cu, "q": normal(hq), "k": normal(hkv), "v": normal(hkv)}
    s["out"] = torch.empty_like(s["q"])
    s["lse"] = torch.empty(hq, T, device="cuda", dtype=torch.float32)
    if case["kind"] in ("step", "new_bin"):
        s["dout"] = normal(hq)
        s["dq"], s["dk"], s["dv"] = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
    if case["kind"] == "new_bin":
        s["pool"] = _pool(case)
        return s
    passes = (va.VA_PASS_FWD, va.VA_PASS_BWD_DKDV, va.VA_PASS_BWD_DQ) if case["kind"] == "step" else (va.VA_PASS_FWD,)
    s["stream"] = va.PackedStream(cu, pl, MASKS[case["mask"]], hq, hkv, d, max_seqlen=longest, passes=passes)
    if case["kind"] in ("fp8", "fp8_block"):
        s["cu_dev"] = torch.from_numpy(cu).to("cuda")
        for n, h in (("q", hq), ("k", hkv), ("v", hkv)):
            s[n + "8"] = torch.empty(T, h, d, device="cuda", dtype=torch.uint8)
            s[n + "_scale"] = torch.empty((h,) if case["kind"] == "fp8" else (T, h), device="cuda", dtype=torch.float32)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind in ("fp8", "fp8_block"):
        for n in ("q", "k", "v"):
            if kind == "fp8":
                va.va_quantize_e4m3_per_head_device(s[n], s[n + "8"], s[n + "_scale"])
            else:
                va.va_quantize_e4m3_blockwise_device(s[n], s["cu"], s["cu_dev"], s[n + "8"], s[n + "_scale"])
        forward = s["stream"].fwd_fp8 if kind == "fp8" else s["stream"].fwd_fp8_blockwise
        forward(s["q8"], s["k8"], s["v8"], s["q_scale"], s["k_scale"], s["v_scale"], s["scale"], s["out"], s["lse"])
        return [s[n] for n in ("q8", "k8", "v8", "q_scale", "k_scale", "v_scale", "out", "lse")]
    outputs = {"out": s["out"], "lse": s["lse"]}
    stream = s.get("stream")
    if kind == "new_bin":
        c, (lens, ends) = s["case"], s["pool"]
        window = c["mask"] == "window"
        bin_of, pos, members, cu, pl, longest = _first_bin(lens, None if window else ends, c["budget"])
        stream = va.PackedStream(cu, ends[members] if window else pl, MASKS[c["mask"]], c["hq"], c["hkv"], c["d"],
                                 max_seqlen=longest)
        outputs.update(bin_of=bin_of, pos=pos, cu=cu)
    stream.fwd(s["q"], s["k"], s["v"], s["scale"], s["out"], s["lse"])
    if kind != "forward":
        stream.bwd(s["q"], s["k"], s["v"], s["out"], s["lse"], s["dout"], s["scale"], s["dq"], s["dk"], s["dv"])
        outputs.update(dq=s["dq"], dk=s["dk"], dv=s["dv"])
    return outputs


def tolerance(case):
    """bfloat16 results of float32 sums whose second products take bfloat16 (FP8: four-bit) probabilities; codes and
    scales, packing and layout are exact."""
    return {"rel": 0.03, "max": 0.5, "differ": 0.0} if case["kind"] in ("fp8", "fp8_block") else {"rel": 0.01, "max": 0.2, "differ": 0.0}
