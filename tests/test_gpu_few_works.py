"""Streams on both sides of the line between the kernels for few works and the persistent ones (which side is asserted), and
with dK/dV alone on the former, against the oracle: the same ragged samples a few and many times over, so that each kernel
sees the edges of its tiles; and one KV head serving eight query heads over a long sample, whose dK/dV steps are dealt
to several workgroups and merged."""
import numpy as np
import pytest

from oracle import attn as oa
from paper_2603_11101_amd import binding as va
from paper_2603_11101_amd import workloads as wl

from gpu_util import DeviceRun, TOL_FWD_REL, TOL_GRAD_REL, TOL_LSE_ABS, max_abs, rel_l2

pytestmark = pytest.mark.gpu

MODES = {va.VA_MASK_CAUSAL: oa.MASK_CAUSAL, va.VA_MASK_PREFIX_LM: oa.MASK_PREFIX_BIDIR_SUFFIX,
         va.VA_MASK_PREFIX_LM_CAUSAL: oa.MASK_PREFIX_CAUSAL_SUFFIX, va.VA_MASK_THREE_BLOCK: oa.MASK_THREE_BLOCK,
         va.VA_MASK_SLIDING_WINDOW: oa.MASK_SLIDING_WINDOW}
SHORT = [1, 31, 32, 33, 64, 65, 96, 127, 128, 129, 200]


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("Hq,Hkv,D,lens,few", [  # few: forward, dQ and dK/dV run on the kernels for few works
    (2, 2, 64, SHORT, (1, 1, 1)), (4, 4, 64, SHORT * 3, (0, 0, 0)), (2, 1, 128, SHORT, (1, 1, 1)),
    (4, 4, 128, SHORT * 3, (0, 0, 0)), (4, 2, 80, SHORT * 4, (0, 0, 1)), (2, 2, 48, SHORT * 6, (0, 0, 0)),
    (8, 1, 256, SHORT, (1, 1, 1)), (8, 4, 256, SHORT * 3, (0, 0, 0)), (16, 2, 96, SHORT, (0, 0, 1)),
    (3, 1, 160, SHORT * 2, (0, 0, 1)), (8, 1, 256, [1005], (1, 1, 8)), (8, 1, 192, [700, 33], (1, 1, 9)),
    (16, 1, 128, [900], (1, 1, 8)), (8, 1, 64, [1300], (1, 1, 5))])
def test_few_and_many_works_against_the_oracle(mode, Hq, Hkv, D, lens, few):
    seed = 500 + Hq + D + len(lens) + mode
    cu, prefix, q, k, v, do = wl.random_stream(seed, lens, Hq, Hkv, D, prefix_frac=-1.0)
    if mode == va.VA_MASK_CAUSAL:
        prefix = None
    elif mode == va.VA_MASK_THREE_BLOCK:
        prefix = wl.random_block_ends(seed, lens)
    elif mode == va.VA_MASK_SLIDING_WINDOW:
        prefix = np.random.default_rng(seed).integers(1, 150, size=len(lens)).astype(np.int32)
    scale = 1.0 / np.sqrt(D)
    print(f"few / many works mode={mode} Hq={Hq} Hkv={Hkv} D={D} samples={len(lens)}", flush=True)
    run = DeviceRun(cu, prefix, mode, q, k, v, do, scale)
    if mode != va.VA_MASK_SLIDING_WINDOW or len(lens) >= len(SHORT):  # a window shortens the walks of one long sample
        assert tuple(va.va_worklist_few_works(run.ps.worklist_host[p], Hq, Hkv)
                     for p in (va.VA_PASS_FWD, va.VA_PASS_BWD_DQ, va.VA_PASS_BWD_DKDV)) == few
    kw = {"scale": scale, "mask_mode": MODES[mode]}
    out, lse = oa.attn_fwd(q, k, v, cu, prefix, **kw)
    assert rel_l2(run.out, out) <= TOL_FWD_REL and max_abs(run.lse, lse) <= TOL_LSE_ABS
    refs = {"out": out, **dict(zip(("dq", "dk", "dv"), oa.attn_bwd(q, k, v, do, cu, prefix, **kw)))}
    for name, want in refs.items():
        got, tol = getattr(run, name), TOL_FWD_REL if name == "out" else TOL_GRAD_REL
        assert rel_l2(got, want) <= tol, name
        for s in range(len(lens)):  # a bad short sample cannot hide behind long ones (two tokens and up: dQ of one is zero)
            sl = slice(cu[s], cu[s + 1])
            if name == "out" or lens[s] > 8 and np.abs(want[sl]).max() > 0:  # nor has a window of one key any
                assert rel_l2(got[sl], want[sl]) <= 2 * tol, (name, s)
    again = DeviceRun(cu, prefix, mode, q, k, v, do, scale)
    assert all(np.array_equal(getattr(run, n), getattr(again, n)) for n in ("out", "lse", "dq", "dk", "dv"))
    assert run.tail_untouched("out", "dq", "dk", "dv")
