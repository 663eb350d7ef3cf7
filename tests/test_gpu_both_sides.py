"""Every instantiation of the bf16 kernels on either side of the line between streams of few works and streams that fill the
chip: the same ragged samples once, and so often that all three passes run on the persistent kernels (which is asserted),
each copy against the oracle.  Copies of a sample inside one stream have equal bits, unless a key tile is split."""
import functools

import numpy as np
import pytest
import torch

from oracle import attn as oa
from paper_2603_11101_amd import binding as va
from paper_2603_11101_amd import workloads as wl

from gpu_util import DEV, DeviceRun, TOL_FWD_REL, TOL_GRAD_REL, TOL_LSE_ABS, from_dev_bf16, max_abs, rel_l2, to_dev_bf16

pytestmark = pytest.mark.gpu

LENS = [70, 0, 129, 33, 200, 1, 300]
MODES = {va.VA_MASK_CAUSAL: oa.MASK_CAUSAL, va.VA_MASK_PREFIX_LM: oa.MASK_PREFIX_BIDIR_SUFFIX,
         va.VA_MASK_PREFIX_LM_CAUSAL: oa.MASK_PREFIX_CAUSAL_SUFFIX, va.VA_MASK_THREE_BLOCK: oa.MASK_THREE_BLOCK,
         va.VA_MASK_SLIDING_WINDOW: oa.MASK_SLIDING_WINDOW}
PASSES = (va.VA_PASS_FWD, va.VA_PASS_BWD_DKDV, va.VA_PASS_BWD_DQ)
NAMES = ("out", "lse", "dq", "dk", "dv")


def ends_of(mode, seed):
    if mode == va.VA_MASK_CAUSAL:
        return None
    if mode == va.VA_MASK_SLIDING_WINDOW:
        return np.array([16, 3, 200, 1, 65, 7, 100], dtype=np.int32)
    if mode == va.VA_MASK_THREE_BLOCK:
        return wl.random_block_ends(seed, LENS)
    return (np.random.default_rng(seed).uniform(0.0, 1.0, size=len(LENS)) * LENS).astype(np.int32)


def tiled(ends, copies):
    return None if ends is None else np.concatenate([ends] * copies)


@functools.lru_cache(maxsize=None)
def copies_for(mode, Hq, Hkv, D, seed):
    """Smallest number of copies for which no pass runs on the kernels for few works."""
    ends, n = ends_of(mode, seed), 1
    while True:
        cu = np.concatenate([[0], np.cumsum(LENS * n)])
        if all(va.va_worklist_few_works(va.va_build_worklist(cu, tiled(ends, n), mode, p, D, Hq, Hkv), Hq, Hkv) == 0
               for p in PASSES):
            return n
        n += max(1, n // 4)


class Copies:
    """A stream of `copies` times the samples of `base` (q, k, v, dout), with its plan and outputs."""

    def __init__(self, base, ends, mode, copies):
        self.copies, self.rows = copies, base[0].shape[0]
        self.cu = np.concatenate([[0], np.cumsum(LENS * copies)]).astype(np.int32)
        (_, Hq, D), Hkv = base[0].shape, base[1].shape[1]
        self.scale = 1.0 / np.sqrt(D)
        self.ps = va.PackedStream(self.cu, tiled(ends, copies), mode, Hq, Hkv, D, device=DEV)
        self.q, self.k, self.v, self.do = (to_dev_bf16(x).repeat(copies, 1, 1) for x in base)

    def run(self, stages=(va.VA_BWD_STAGE_ALL,)):
        """Outputs by name, with the copies as the first dimension."""
        o = {"out": torch.full_like(self.q, 768.0), "dq": torch.full_like(self.q, 768.0), "dk": torch.full_like(self.k, 768.0),
             "dv": torch.full_like(self.v, 768.0)}
        lse = torch.full((self.q.shape[1], self.q.shape[0]), 768.0, dtype=torch.float32, device=DEV)
        self.ps.fwd(self.q, self.k, self.v, self.scale, o["out"], lse)
        for s in stages:
            self.ps.bwd_stages(self.q, self.k, self.v, o["out"], lse, self.do, self.scale, o["dq"], o["dk"], o["dv"], s)
        torch.cuda.synchronize()
        o = {n: t.view(self.copies, self.rows, *t.shape[1:]) for n, t in o.items()}
        o["lse"] = lse.view(lse.shape[0], self.copies, self.rows).transpose(0, 1)
        return o

    def split_key_tiles(self):
        return int(self.ps.worklist_host[va.VA_PASS_BWD_DKDV][1, 7]) > 0


def same_bits(a, b):
    kind = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
    return torch.equal(a.contiguous().view(kind), b.contiguous().view(kind))


def oracle(base, ends, mode, scale):
    q, k, v, do = base
    cu = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int32)
    kw = {"scale": scale, "mask_mode": MODES[mode]}
    out, lse = oa.attn_fwd(q, k, v, cu, ends, **kw)
    return dict(zip(NAMES, (out, lse, *oa.attn_bwd(q, k, v, do, cu, ends, **kw))))


def check(got, want):
    """One copy (numpy, float64) against the oracle, sample by sample."""
    start = np.concatenate([[0], np.cumsum(LENS)])
    assert max_abs(got["lse"], want["lse"]) <= TOL_LSE_ABS
    for n, tol in (("out", TOL_FWD_REL), ("dq", TOL_GRAD_REL), ("dk", TOL_GRAD_REL), ("dv", TOL_GRAD_REL)):
        size = np.sqrt((want[n] ** 2).mean())
        for s, L in enumerate(LENS):
            g, w = (x[n][start[s]:start[s + 1]] for x in (got, want))
            assert np.isfinite(g).all(), (n, s)
            if L and np.sqrt((w ** 2).mean()) > 1e-3 * size:
                assert rel_l2(g, w) <= tol, (n, s)
            elif L:  # a row that sees itself alone has dQ = dK = 0 up to the rounding of dP - delta
                assert np.abs(g).max() <= 1e-3 * size, (n, s)


def stream(seed, Hq, Hkv, D):
    _, _, q, k, v, do = wl.random_stream(seed, LENS, Hq, Hkv, D)
    return q, k, v, do


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("window", [False, True])
@pytest.mark.parametrize("D", [48, 64, 80, 96, 128, 160, 192, 256])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_every_head_dimension_and_stacking_on_either_side(D, G, window, many):
    Hkv = 2 if G <= 2 else 1
    Hq = G * Hkv
    mode = va.VA_MASK_SLIDING_WINDOW if window else list(MODES)[(D // 16 + G.bit_length()) % 4]
    seed = 8000 + 10 * D + G
    base, ends = stream(seed, Hq, Hkv, D), ends_of(mode, seed)
    copies = copies_for(mode, Hq, Hkv, D, seed) if many else 1
    print(f"D={D} heads={Hq}/{Hkv} mode={mode} copies={copies}", flush=True)
    c = Copies(base, ends, mode, copies)
    for p in PASSES:
        assert (va.va_worklist_few_works(c.ps.worklist_host[p], Hq, Hkv) > 0) == (not many), p
    got = c.run()
    want = oracle(base, ends, mode, c.scale)
    split = c.split_key_tiles()
    for n in NAMES:
        if not (split and n in ("dk", "dv")):
            assert same_bits(got[n], got[n][:1].expand_as(got[n])), n
    for i in {0, copies // 2, copies - 1} if split else {0}:
        check({n: t[i].cpu().numpy().astype(np.float64) if n == "lse" else from_dev_bf16(t[i]) for n, t in got.items()}, want)
    if split:  # every copy, at the norm of a whole copy
        for n in ("dk", "dv"):
            w = torch.from_numpy(want[n]).to(DEV)
            off = ((got[n].double() - w) ** 2).flatten(1).sum(1).sqrt() / (w ** 2).sum().sqrt()
            assert float(off.max()) <= TOL_GRAD_REL, n


@pytest.mark.parametrize("mode,Hq,Hkv,D", [
    (va.VA_MASK_CAUSAL, 4, 2, 128), (va.VA_MASK_PREFIX_LM, 8, 1, 256), (va.VA_MASK_SLIDING_WINDOW, 8, 2, 128),
    (va.VA_MASK_PREFIX_LM_CAUSAL, 2, 2, 64), (va.VA_MASK_THREE_BLOCK, 4, 4, 80)])
def test_nothing_of_one_sample_reaches_another_on_the_persistent_kernels(mode, Hq, Hkv, D):
    seed = 8900 + D + mode
    base, ends = stream(seed, Hq, Hkv, D), ends_of(mode, seed)
    copies = copies_for(mode, Hq, Hkv, D, seed)
    print(f"no leak D={D} heads={Hq}/{Hkv} mode={mode} copies={copies}", flush=True)
    c = Copies(base, ends, mode, copies)
    clean, again = c.run(), c.run()
    assert all(same_bits(clean[n], again[n]) for n in NAMES)
    bad = copies // 2
    rows = slice(bad * c.rows, (bad + 1) * c.rows)
    c.q[rows], c.k[rows], c.v[rows], c.do[rows] = float("nan"), float("inf"), float("nan"), float("nan")
    poisoned = c.run()
    for n in NAMES:
        for part in (slice(0, bad), slice(bad + 1, copies)):
            assert same_bits(poisoned[n][part], clean[n][part]), n


@pytest.mark.parametrize("Hq,Hkv,D", [(8, 2, 64), (4, 2, 128), (8, 1, 256)])
def test_backward_by_stages_on_the_persistent_kernels(Hq, Hkv, D):
    base = stream(8700 + D, Hq, Hkv, D)
    copies = copies_for(va.VA_MASK_CAUSAL, Hq, Hkv, D, 0)
    print(f"by stages D={D} heads={Hq}/{Hkv} copies={copies}", flush=True)
    c = Copies(base, None, va.VA_MASK_CAUSAL, copies)
    whole = c.run()
    c.ps.workspace().fill_(0xFF)
    first = va.VA_BWD_STAGE_DQ | (va.VA_BWD_STAGE_DELTA if va.va_bwd_has_delta_kernel(D) else 0)
    parts = c.run(stages=(first, va.VA_BWD_STAGE_DKDV))
    assert all(same_bits(whole[n], parts[n]) for n in NAMES)


@pytest.mark.parametrize("Hq,Hkv,D,splits", [(4, 4, 128, (1, 1)), (8, 1, 256, (16, 8))])
def test_bits_of_a_sample_beside_another_on_the_kernels_for_few_works(Hq, Hkv, D, splits):
    # O, LSE and dQ have the bits of the sample alone; dK and dV as long as their steps are dealt to as many workgroups
    L = 430
    cu, _, q, k, v, do = wl.random_stream(8800 + D, [L, L], Hq, Hkv, D)
    scale = 1.0 / np.sqrt(D)
    print(f"beside another D={D} heads={Hq}/{Hkv}", flush=True)
    runs = []
    for n in (1, 2):
        run = DeviceRun(cu[:n + 1], None, va.VA_MASK_CAUSAL, *(x[:n * L] for x in (q, k, v, do)), scale)
        few = [va.va_worklist_few_works(run.ps.worklist_host[p], Hq, Hkv) for p in PASSES]
        assert few == [1, splits[n - 1], 1]
        runs.append(run)
    alone, beside = runs
    assert np.array_equal(beside.out[:L], alone.out) and np.array_equal(beside.lse[:, :L], alone.lse)
    assert np.array_equal(beside.dq[:L], alone.dq)
    for n in ("dk", "dv"):
        a, b = getattr(alone, n), getattr(beside, n)[:L]
        # the sums differ in order alone: float32 rounding, then at most a last place of bfloat16 where that falls on an edge
        assert np.array_equal(a, b) if splits[0] == splits[1] else rel_l2(b, a) <= 2.0 ** -8, n
