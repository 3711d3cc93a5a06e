"""The scans' window in runs: older runs that are left alone, and inputs for which they must not be.  Durations just beyond the
first run, at the edges of two and of four runs, both task forms, both directions, and mended tasks (a first warm-up far too
short), which start from a whole window."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_parity import assert_outputs_match_oracle

pytestmark = pytest.mark.gpu

FORMS = {"one wave": sb.SEMICRF_ONE_WAVE_SCAN, "two waves": sb.SEMICRF_TWO_WAVE_SCAN}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def case(T, K, C, kind):
    w = synth.small_random(3 * T + K + C, 2, T, K, C, ragged=True)
    w.lengths[:] = [T, T - K // 2 - 1]
    if kind == "only old":  # all labels but the first have no duration of the first run: what is left alone elsewhere is all
        w.dur[: K - 1, 1:] = -1e4
    elif kind == "long":    # weights that rise with the duration as fast as messages grow: every run counts about as much
        w.dur += (1.2 * np.arange(K, dtype=np.float32))[:, None]
    elif kind == "no splits":  # a run of one label is one segment, so that its oldest entry decides; the runs' lengths vary
        w.trans[np.arange(C), np.arange(C)] = -30.0
        w.emis[:, np.arange(T), np.cumsum(np.arange(T) % (K - 2) == 0) % C] += 4.0
    elif kind == "stretches":  # certain scores, then none at all
        w.emis[:, T // 4: T // 2, 0] += 12.0
        w.emis[:, T // 2: 3 * T // 4] = 0.0
    return w


@pytest.mark.parametrize("T,K,C", [(900, 137, 8), (1200, 272, 5), (1300, 273, 8), (700, 69, 16), (800, 256, 9), (500, 33, 24), (500, 64, 19),
                                   (500, 65, 24), (500, 128, 32), (300, 17, 40), (300, 33, 64), (300, 64, 33)])
@pytest.mark.parametrize("kind", ["plain", "only old", "long", "no splits", "stretches"])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_runs_that_count_are_taken(T, K, C, kind, form):
    w = case(T, K, C, kind)
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur)
    delta = (K + 15) // 8 * 8
    for warm in (0, 12):  # as chosen; so short that boundaries are mended or scanned again
        flags = sb.SEMICRF_CENTER | FORMS[form] | sb.SEMICRF_WARMUP(warm)
        args = [dev(a) for a in (w.emis, w.lengths, w.trans, w.dur)]
        ws = sb.alloc_workspace(w.B, T, K, C, delta, 1, "cuda:0").fill_(255)
        out = sb.semicrf_fwd_bwd(*args, None, delta, flags=flags, workspace=ws)
        lz = sb.semicrf_seq_report(ws, w.B, T, K, C, delta, 1)[1].cpu().numpy()
        acc = sb.semicrf_scan_report(ws, w.B, T, K, C, delta, 1)[0].cpu().numpy()
        print(f"[case] {kind} {form} T={T} K={K} C={C} warm-up {warm or 'chosen'} verified at {acc.tolist()}", flush=True)
        assert kind != "plain" or warm or (acc >= 1).all()  # (the sequential scan's results would be right, too)
        assert_outputs_match_oracle([o.double().cpu().numpy() for o in out], r)
        # what is left alone is below 2^-54 of every sum; accepted boundaries agree to 2e-10 each; T sums in 64 bits
        bound = 2e-10 * (T / delta) + 1e-13 * T + 1e-13 * np.abs(r.logz).max()
        assert np.abs(lz - r.logz).max() <= bound
        lf = sb.semicrf_logz_fwd(*args, delta, flags=flags).double().cpu().numpy()
        assert np.abs(lf - r.logz).max() <= 1e-6 * max(1.0, np.abs(r.logz).max())
