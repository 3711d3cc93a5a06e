"""GPU tests of what follows a rejected first attempt of the chunk-parallel scans, in both forms of their tasks: mending of
isolated boundaries, and the warm-up derived from the mismatch of the attempt before.  Results as the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_parity import assert_outputs_match_oracle, run_with_report

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [sb.SEMICRF_ONE_WAVE_SCAN, sb.SEMICRF_TWO_WAVE_SCAN])
@pytest.mark.parametrize("flat", [(590, 680), (600, 700)])
@pytest.mark.parametrize("C,K", [(4, 4), (12, 6), (24, 4), (40, 4)])
def test_isolated_boundaries_are_mended(form, flat, C, K):
    """A deterministic chain pinned by its emissions except on a flat stretch (test_gpu_parity.py has the argument why one
    boundary, or two adjacent ones, fail): accepted with code 2."""
    B, T = 2, 2000
    w = synth.small_random(74, B, T, K, C, ragged=False)
    w.emis[:] = 0.0
    w.emis[:, np.arange(T), (np.arange(T) // 2) % C] = 8.0
    w.emis[:, flat[0]:flat[1], :] = 0.0
    w.trans[:] = -40.0
    w.trans[np.arange(C), (np.arange(C) + 1) % C] = 0.0
    w.dur[:] = -40.0
    w.dur[1, :] = 0.0
    out, acc, mis = run_with_report(w, sb.SEMICRF_CENTER | form, 64)
    print(f"       accepted {acc.ravel()} boundary mismatch {mis.ravel()}", flush=True)
    assert np.all(acc == 2) and np.all(mis <= 1e-10)
    assert_outputs_match_oracle(out, oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur))


@pytest.mark.parametrize("form", [sb.SEMICRF_ONE_WAVE_SCAN, sb.SEMICRF_TWO_WAVE_SCAN])
@pytest.mark.parametrize("flat", [(590, 680), (1900, 2000)])
@pytest.mark.parametrize("C,K", [(4, 12), (24, 11), (40, 21)])
def test_mended_tasks_take_the_whole_window_over(form, flat, C, K):
    """The same chain with segments of five tokens: a mended task's first positions get what they get from window entries further
    back than the newest four, which the two-wave form adds up a block ahead.  Flat at the end of the sequence, the mended
    interval is the forward scan's last one, and no further boundary looks at what it reached."""
    B, T, length = 2, 2000, 5
    w = synth.small_random(75, B, T, K, C, ragged=False)
    w.emis[:] = 0.0
    w.emis[:, np.arange(T), (np.arange(T) // length) % C] = 8.0
    w.emis[:, flat[0]:flat[1], :] = 0.0
    w.trans[:] = -40.0
    w.trans[np.arange(C), (np.arange(C) + 1) % C] = 0.0
    w.dur[:] = -40.0
    w.dur[length - 1, :] = 0.0
    out, acc, mis = run_with_report(w, sb.SEMICRF_CENTER | form, 64, warm_env=32)
    print(f"       accepted {acc.ravel()} boundary mismatch {mis.ravel()}", flush=True)
    assert np.all((acc == 2) | (acc == 1)) and np.any(acc == 2) and np.all(mis <= 1e-10)
    assert_outputs_match_oracle(out, oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur))


@pytest.mark.parametrize("form", [sb.SEMICRF_ONE_WAVE_SCAN, sb.SEMICRF_TWO_WAVE_SCAN])
@pytest.mark.parametrize("T,K,C,delta,warm,sd,band", [
    (3001, 37, 19, 0, 0, 1.0, 2), (1500, 16, 10, 64, 20, 2.0, 0), (1200, 40, 24, 96, 40, 3.0, 2), (900, 12, 50, 48, 12, 1.0, 0),
    (2500, 130, 8, 0, 100, 2.0, 1),
])
def test_slower_models_verify_after_a_longer_warm_up(form, T, K, C, delta, warm, sd, band):
    w = synth.small_random(T, 3, T, K, C, ragged=False)
    w.lengths[:] = [T, T - 1, T // 2]
    w.trans[:] = synth.reshape_transitions(w.trans, sd=sd / 3.0, band=band or None)  # small_random's are N(0, 0.3^2)
    out, acc, mis = run_with_report(w, sb.SEMICRF_CENTER | form, delta, warm_env=warm or None)
    print(f"       accepted {acc.ravel()} boundary mismatch {mis.max():.1e}", flush=True)
    assert np.all(acc >= 2) and np.all(mis <= 1e-10)
    assert_outputs_match_oracle(out, oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur))
