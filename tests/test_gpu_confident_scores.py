"""GPU parity on the scores of a trained encoder: every position has one label far above the others, in segments longer than
K, so that a message falls for the labels that do not hold as fast as the prefix sum of the label that does rises.  What a
scaling block may reach is the sum of the two; a block that is too long for it overflows without the range flag.

Labels score +s where they hold and -s elsewhere, plus unit noise; segments of 40 positions, up to the 300 nats per position
that the entry points promise.  Tolerances as in test_gpu_parity.py.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dev(a, dtype=np.float32):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to(DEV)


def confident(seed, B, T, K, C, s, segment=40):
    w = synth.small_random(seed, B, T, K, C, ragged=False)
    rng = np.random.default_rng(seed + 1)
    w.lengths[:] = rng.integers(T // 2, T + 1, size=B)
    w.lengths[0] = T
    for b in range(B):
        label = np.repeat(rng.integers(0, C, T // segment + 1), segment)[:T]
        f = np.full((T, C), -s) + rng.standard_normal((T, C))
        f[np.arange(T), label] += 2 * s
        w.emis[b] = f
    return w


def close(got, ref, names, per_position):
    for n in names:
        g, r = got[n].double().cpu().numpy(), getattr(ref, n)
        tol = 1e-4 * (1.0 if n in per_position else max(1.0, np.abs(r).max()))
        assert np.all(np.isfinite(g)), n
        assert np.abs(g - r).max() <= tol, (n, np.abs(g - r).max())


CASES = [(2, 12, 1), (2, 14, 1), (2, 15, 1), (2, 30, 1), (2, 60, 0), (2, 140, 1), (2, 250, 0), (3, 10, 1), (3, 20, 1),
         (4, 120, 0), (5, 60, 1), (8, 12, 0), (8, 100, 0), (8, 250, 0)]


# Lengths with sums and headers from one launch (up to three chunks of 256 positions; with projections of two sequences: one), and from two.
@pytest.mark.parametrize("C,s,center", CASES)
def test_training_and_scoring(C, s, center):
    for T, K, extra in ((700, 8, 0), (700, 8, sb.SEMICRF_SEQUENTIAL_SCAN), (700, 8, sb.SEMICRF_MARGINALS_INTERVAL),
                        (700, 8, sb.SEMICRF_TWO_WAVE_SCAN), (700, 150, 0), (1100, 8, 0), (1100, 150, 0)):
        w = confident(10 * C + s, 2, T, K, C, s)
        flags = (sb.SEMICRF_CENTER if center else 0) | extra
        print(f"[case] C={C} s={s} center={center} T={T} K={K} flags={flags}", flush=True)
        x = (dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur))
        ws = sb.alloc_workspace(w.B, w.T, K, C, 0, sb.grad_workspace_kind(flags), DEV)
        out = sb.semicrf_fwd_bwd(*x, flags=flags, workspace=ws)
        exceeded, _ = sb.semicrf_seq_report(ws, w.B, w.T, K, C, 0, sb.grad_workspace_kind(flags))
        score = sb.semicrf_logz_fwd(*x, flags=flags)
        r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, center=bool(center))
        assert exceeded.sum().item() == 0
        for lz in (out[0], score):
            assert np.abs(lz.double().cpu().numpy() - r.logz).max() <= 1e-5 * np.abs(r.logz).max()
        close(dict(zip(("grad_emis", "grad_trans", "grad_dur", "pos_marg"), out[1:])), r,
              ("grad_emis", "grad_trans", "grad_dur", "pos_marg"), ("grad_emis", "pos_marg"))


@pytest.mark.parametrize("C,s,center", CASES)
def test_boundary_terms(C, s, center):
    K, B = 8, 2
    for T, extra in ((700, 0), (700, sb.SEMICRF_MARGINALS_INTERVAL), (250, 0)):
        w = confident(10 * C + s, B, T, K, C, s)
        rng = np.random.default_rng(s)
        q = min(s, 60) / 8
        ps, pe = (q * rng.uniform(-1, 1, (2, B, T, C))).astype(np.float32)
        pis, pie = (q * rng.uniform(-1, 1, (2, C))).astype(np.float32)
        r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, proj_start=ps, proj_end=pe, pi_start=pis, pi_end=pie,
                           center=bool(center))
        out = sb.semicrf_fwd_bwd_boundary(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), None, dev(ps),
                                          dev(pe), dev(pis), dev(pie), flags=(sb.SEMICRF_CENTER if center else 0) | extra)
        assert np.abs(out["logz"].double().cpu().numpy() - r.logz).max() <= 1e-5 * np.abs(r.logz).max()
        per_position = ("grad_emis", "pos_marg", "grad_proj_start", "grad_proj_end", "bdy_post")
        close(out, r, per_position + ("grad_trans", "grad_dur", "grad_pi_start", "grad_pi_end"), per_position)


@pytest.mark.parametrize("C,s,center", CASES)
def test_duration_dependent_transitions(C, s, center):
    w = confident(10 * C + s, 2, 500, 8, C, s)
    trans3 = synth.duration_transitions(w, C, 0.3)
    flags = sb.SEMICRF_CENTER if center else 0
    r = oracle.fwd_bwd_durtrans(w.emis, w.lengths, trans3, w.dur, center=bool(center))
    x = (dev(w.emis), dev(w.lengths, np.int32), dev(trans3), dev(w.dur))
    for extra in (0, sb.SEMICRF_SEQUENTIAL_SCAN):
        out = sb.semicrf_fwd_bwd_durtrans(*x, flags=flags | extra)
        for lz in (out[0], sb.semicrf_logz_fwd_durtrans(*x, flags=flags | extra)):
            assert np.abs(lz.double().cpu().numpy() - r.logz).max() <= 1e-5 * np.abs(r.logz).max()
        close(dict(zip(("grad_emis", "grad_trans", "grad_dur", "pos_marg"), out[1:])), r,
              ("grad_emis", "grad_trans", "grad_dur", "pos_marg"), ("grad_emis", "pos_marg"))


def test_long_sequence_takes_the_headers_of_a_launch_of_their_own():
    """More chunks than the prefix kernel sums up itself: the block length comes from the per-sequence kernel."""
    w = confident(5, 1, 131500, 4, 2, 60)
    lz = sb.semicrf_logz_fwd(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur))
    r = oracle.logz(w.emis, w.lengths, w.trans, w.dur)
    assert np.abs(lz.double().cpu().numpy() - r).max() <= 1e-5 * np.abs(r).max()


def test_many_labels_forward_only():
    """Generic scan (more than 64 labels)."""
    w = confident(6, 2, 400, 6, 70, 40)
    lz = sb.semicrf_logz_fwd(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), flags=0)
    r = oracle.logz(w.emis, w.lengths, w.trans, w.dur, center=False)
    assert np.abs(lz.double().cpu().numpy() - r).max() <= 1e-5 * np.abs(r).max()
