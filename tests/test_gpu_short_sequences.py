"""GPU parity of the prefix stage that needs no launch before it (up to three chunks of 256 positions, tables of at most 2048
entries), at its edges and on the other side of them: groups of 32 positions, chunks, the largest tables, sequences that are empty or
end at a chunk's edge, half-precision emissions.  Tolerances as elsewhere: 1e-5 of logZ, 1e-4 of a gradient's largest entry."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda:0")


@pytest.mark.parametrize("T", [1, 31, 32, 33, 255, 256, 511, 512, 767, 768])
@pytest.mark.parametrize("K,C", [(1, 1), (6, 3), (16, 24), (2, 44), (3, 44)])
@pytest.mark.parametrize("terms", [False, True])
def test_sums_and_tables_in_one_launch(T, K, C, terms):
    rng = np.random.default_rng(T * 100 + C)
    w = synth.small_random(T + K, 4, T, K, C, ragged=False)
    w.lengths[:] = [T, max(T - 1, 0), T // 256 * 256, 0]
    kw = dict(proj_start=None, proj_end=None, pi_start=None, pi_end=None)
    if terms:
        ps, pe = (3.0 * rng.standard_normal((2, 4, T, C))).astype(np.float32)
        pis, pie = rng.standard_normal((2, C)).astype(np.float32)
        kw = dict(proj_start=ps, proj_end=pe, pi_start=pis, pi_end=pie)
    emis = dev(w.emis)
    if T == 512:  # any storage type of the scores
        emis = emis.to(torch.bfloat16 if terms else torch.float16)
    out = sb.semicrf_fwd_bwd_boundary(emis, dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), None,
                                      *[None if x is None else dev(x) for x in kw.values()])
    r = oracle.fwd_bwd(emis.float().cpu().numpy(), w.lengths, w.trans, w.dur, boundary=True, **kw)
    lz = out["logz"].double().cpu().numpy()
    assert (np.abs(lz - r.logz) <= 1e-5 * np.maximum(np.abs(r.logz), 1.0)).all(), (lz, r.logz)
    for name in ("grad_emis", "pos_marg", "bdy_post", "grad_trans", "grad_dur"):
        g, ref = out[name].double().cpu().numpy(), getattr(r, name)
        assert np.abs(g - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max()), name
    best = sb.semicrf_viterbi(emis, dev(w.lengths, np.int32), dev(w.trans), dev(w.dur))[0].double().cpu().numpy()
    want = oracle.viterbi(emis.float().cpu().numpy(), w.lengths, w.trans, w.dur)[0]
    assert (np.abs(best - want) <= 1e-5 * np.maximum(np.abs(want), 1.0)).all()
