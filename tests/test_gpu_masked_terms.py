"""Boundary terms of -infinity as masks: starts and ends that are forbidden at some positions or for some labels.  The oracle is
given -1e4 in their place, which is as good as forbidden in fp64 (e^-1e4 = 0) and keeps its logarithms finite.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda:0")


@pytest.mark.parametrize("mask", [-np.inf, -1.0e4, np.finfo(np.float32).min])
@pytest.mark.parametrize("T,K,C,extra", [(300, 12, 5, 0), (300, 12, 5, sb.SEMICRF_SEQUENTIAL_SCAN), (700, 20, 24, 0),
                                         (500, 140, 6, 0), (200, 30, 64, 0), (300, 12, 5, sb.SEMICRF_MARGINALS_INTERVAL),
                                         (250, 12, 5, 0), (1000, 12, 5, 0)])
def test_forbidden_starts_and_ends(T, K, C, extra, mask):
    rng = np.random.default_rng(T + C)
    w = synth.small_random(T + K, 2, T, K, C, ragged=False)
    w.lengths[:] = [T, T - 37]
    ps, pe = (0.5 * rng.standard_normal((2, 2, T, C))).astype(np.float32)
    pis, pie = rng.standard_normal((2, C)).astype(np.float32)
    # a segment of label c may start only where t % 3 != c % 3 and end only where that is so for the next position, the
    # sequence itself begins with label 1 and does not end with label 0
    no = (np.arange(T)[:, None] - np.arange(C)[None]) % 3 == 0
    no_start, no_end = no.copy(), np.roll(no, -1, axis=0)
    no_start[0] = False
    no_end[w.lengths - 1] = False
    terms = {}
    for value, kind in ((mask, "gpu"), (-1.0e4, "oracle")):
        s, e, i, o = ps.copy(), pe.copy(), pis.copy(), pie.copy()
        s[:, no_start] = value
        e[:, no_end] = value
        i[np.arange(C) != 1] = value
        o[0] = value
        terms[kind] = (s, e, i, o)
    out = sb.semicrf_fwd_bwd_boundary(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), None,
                                      *[dev(x) for x in terms["gpu"]], flags=sb.SEMICRF_CENTER | extra)
    s, e, i, o = terms["oracle"]
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, proj_start=s, proj_end=e, pi_start=i, pi_end=o, boundary=True)
    assert np.abs(out["logz"].double().cpu().numpy() - r.logz).max() <= 1e-5 * np.abs(r.logz).max()
    for name in ("grad_emis", "pos_marg", "grad_proj_start", "grad_proj_end", "bdy_post", "grad_trans", "grad_dur",
                 "grad_pi_start", "grad_pi_end"):
        g, ref = out[name].double().cpu().numpy(), getattr(r, name)
        assert np.abs(g - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max()), name
    for name, m in (("grad_proj_start", no_start), ("grad_proj_end", no_end)):
        assert (out[name].cpu().numpy()[:, m] == 0).all()
