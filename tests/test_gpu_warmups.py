"""Warm-ups from the model: windows that agree only in what they still contribute.  Durations so long that the warm-up is a fraction
of the window (with the gradients of durations that hardly occur, which come from the neighbouring interval's window), label counts
at the edges of the comparison's shares, models that the choice misjudges (long durations favoured, forbidden transitions), one
transition matrix per duration, and a workspace full of NaN."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_parity import assert_outputs_match_oracle

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def case(T, K, C, kind, B=2):
    w = synth.small_random(T + 7 * K + C, B, T, K, C, ragged=True)
    w.lengths[:] = ([T, T - K // 2 - 1, 0] * B)[:B]
    if kind == "band":
        i = np.arange(C)
        d = np.abs(i[:, None] - i[None, :])
        w.trans[np.minimum(d, C - d) > 1] = -1e4
    elif kind == "long":  # what a warm-up of the predicted length leaves out decides
        w.dur += (0.25 * np.arange(K, dtype=np.float32))[:, None]
    elif kind == "forbidden durations":
        w.dur[: K // 2] = -1e4
    elif kind == "confident":
        w.emis[:, :, 0] += 9.0
    return w


def train(w, delta):
    ws = sb.alloc_workspace(w.B, w.T, w.K, w.C, delta, 1, "cuda:0").fill_(255)
    out = sb.semicrf_fwd_bwd(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur), None, delta, workspace=ws)
    acc = sb.semicrf_scan_report(ws, w.B, w.T, w.K, w.C, delta, 1)[0].cpu().numpy()
    return [o.double().cpu().numpy() for o in out], acc


@pytest.mark.parametrize("T,K,C,delta", [(900, 64, 24, 96), (905, 65, 24, 72), (700, 37, 19, 40), (600, 32, 64, 64), (603, 40, 33, 40),
                                         (1500, 130, 8, 136), (2100, 512, 8, 512), (1300, 256, 16, 256), (900, 128, 32, 128),
                                         (500, 17, 3, 24), (400, 8, 2, 8), (330, 60, 15, 64)])
def test_rare_durations(T, K, C, delta):
    w = case(T, K, C, "plain")
    out, acc = train(w, delta)
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur)
    assert (acc[w.lengths > 0] >= 1).all()
    assert_outputs_match_oracle(out, r)
    # every duration, however rare: the scans agree to 2e-10 a boundary, the rest is the rounding of the float (6e-8)
    some = r.grad_dur > 1e-30
    rel = np.abs(out[3] - r.grad_dur)[some] / r.grad_dur[some]
    print(f"[case] T={T} K={K} C={C} relative error of grad_dur {rel.max():.1e} down to {r.grad_dur[some].min():.1e}", flush=True)
    assert rel.max() <= 1e-6
    lz = sb.semicrf_logz_fwd(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur)).double().cpu().numpy()
    assert np.abs(lz - r.logz).max() <= 1e-5 * np.abs(r.logz).max()


@pytest.mark.parametrize("T,K,C", [(800, 60, 10), (1200, 6, 20), (700, 130, 7), (500, 20, 40)])
@pytest.mark.parametrize("kind", ["band", "long", "forbidden durations", "confident"])
def test_models_the_choice_may_misjudge(T, K, C, kind):
    w = case(T, K, C, kind, B=3)
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur)
    for delta in (0, max(K, 40)):
        out, acc = train(w, delta)
        print(f"[case] {kind} T={T} K={K} C={C} interval {delta} verified at {acc.tolist()}", flush=True)
        assert kind != "confident" or (acc[w.lengths > 0] >= 1).all()
        assert_outputs_match_oracle(out, r)


@pytest.mark.parametrize("T,K,C", [(700, 64, 8), (500, 40, 24), (600, 200, 3), (300, 18, 32), (400, 512, 8)])
@pytest.mark.parametrize("kind", ["plain", "band", "long"])
def test_duration_dependent_transitions(T, K, C, kind):
    w = case(T, K, C, kind)
    t3 = synth.duration_transitions(w, 5, 0.2)
    r = oracle.fwd_bwd_durtrans(w.emis, w.lengths, t3, w.dur)
    for delta in (0, 64):
        ws = sb.alloc_durtrans_workspace(w.B, T, K, C, delta, True, "cuda:0").fill_(255)
        out = sb.semicrf_fwd_bwd_durtrans(dev(w.emis), dev(w.lengths), dev(t3), dev(w.dur), None, delta, workspace=ws)
        acc = sb.semicrf_scan_report(ws, w.B, T, K, C, sb.semicrf_durtrans_ckpt_interval(w.B, T, K, C, delta), True)[0].cpu().numpy()
        print(f"[case] {kind} T={T} K={K} C={C} interval {delta} verified at {acc.tolist()}", flush=True)
        assert kind != "plain" or (acc[w.lengths > 0] >= 1).all()  # (not by the whole-sequence scans, whose results are the same)
        assert_outputs_match_oracle([o.double().cpu().numpy() for o in out], r)


@pytest.mark.parametrize("T,K,C", [(900, 64, 24), (905, 65, 20), (700, 37, 9), (600, 32, 40), (1500, 130, 8), (2100, 300, 5), (1300, 90, 3),
                                   (700, 21, 64)])
@pytest.mark.parametrize("kind", ["plain", "band", "long", "forbidden durations", "confident", "no splits"])
def test_best_segmentation(T, K, C, kind):
    w = case(T, K, C, kind, B=3)
    if kind == "no splits":  # a run of one label is one segment: an entry as old as the run decides
        w.trans[np.arange(C), np.arange(C)] = -6.0
        run = np.arange(T) // (K - 2) % C
        w.emis[:, np.arange(T), run] += 4.0
    ws = torch.full((sb.semicrf_viterbi_workspace_bytes(3, T, K, C) + 256,), 255, dtype=torch.uint8, device="cuda:0")
    off = (-ws.data_ptr()) % 256
    score, labels, starts, nseg = sb.semicrf_viterbi(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur),
                                                     workspace=ws[off:ws.numel() - 256 + off])
    acc = sb.semicrf_scan_report(ws[off:ws.numel() - 256 + off], 3, T, K, C, 0, 0)[0][:, 0].cpu().numpy()
    print(f"[case] {kind} T={T} K={K} C={C} verified at {acc.tolist()}", flush=True)
    assert kind not in ("plain", "confident") or (acc[w.lengths > 0] == 1).all()
    ref = oracle.viterbi(w.emis, w.lengths, w.trans, w.dur)[0]
    assert np.abs(score.double().cpu().numpy() - ref).max() <= 1e-6 * max(1.0, np.abs(ref).max())
    for b in range(3):
        L = int(w.lengths[b])
        if L:  # the path is worth what the oracle's best one is (fp64 sums of T terms)
            got = oracle.path_score(w.emis[b], L, w.trans, w.dur, labels[b].cpu().numpy(), starts[b].cpu().numpy())
            assert abs(got - ref[b]) <= 1e-9 * max(1.0, abs(ref[b]))
        assert nseg[b].item() == starts[b].sum().item()


@pytest.mark.parametrize("T,K,C", [(400, 16, 24), (1500, 40, 12), (700, 64, 24)])
def test_a_sequence_does_not_depend_on_its_batch(T, K, C):
    """The same sequence next to others whose scores are certain, or tell nothing at all: the same to the last bit."""
    w = case(T, K, C, "plain", B=4)
    w.lengths[:] = T
    lone = None
    for scale in (0.0, 1.0, 30.0):
        w.emis[1:] *= scale
        ws = sb.alloc_workspace(4, T, K, C, 0, 1, "cuda:0")
        out = sb.semicrf_fwd_bwd(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur), None, 0, workspace=ws)
        rep = sb.semicrf_scan_report(ws, 4, T, K, C, 0, 1) + sb.semicrf_seq_report(ws, 4, T, K, C, 0, 1)
        fws = sb.alloc_workspace(4, T, K, C, 0, 0, "cuda:0")
        sb.semicrf_logz_fwd(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur), workspace=fws)
        rep += sb.semicrf_scan_report(fws, 4, T, K, C, 0, 0) + sb.semicrf_seq_report(fws, 4, T, K, C, 0, 0)
        got = [x[0].cpu().numpy() for x in (out[0], out[1], out[4]) + rep]
        if lone is not None:
            assert all(np.array_equal(a, b) for a, b in zip(got, lone))
        lone = got
        w = case(T, K, C, "plain", B=4)
        w.lengths[:] = T


def labelled(B, T, K, C, sd, own=True, band=None, seed=1):
    """Scores that follow a label path (2 for its label, unit noise) and transitions N(0, sd^2), the labels' own forbidden or not,
    those beyond a band forbidden or not."""
    g = np.random.default_rng(seed)
    trans = (sd * g.standard_normal((C, C))).astype(np.float32)
    d = np.abs(np.arange(C)[:, None] - np.arange(C)[None, :])
    trans[(d == 0) & (not own) | (np.minimum(d, C - d) > (C if band is None else band))] = -1e4
    emis = g.standard_normal((B, T, C)).astype(np.float32)
    label = g.integers(0, C, (B, T + 1))
    path = np.take_along_axis(label, np.cumsum(g.random((B, T)) < 3 / K, axis=1), 1)
    np.put_along_axis(emis, path[:, :, None], np.take_along_axis(emis, path[:, :, None], 2) + 2.0, 2)
    return dev(emis), None, dev(trans), dev((0.1 * g.standard_normal((K, C))).astype(np.float32))


def score(x, B, T, K, C, flags=sb.SEMICRF_CENTER):
    """logZ in 64 bits, and how the scan was verified."""
    ws = sb.alloc_workspace(B, T, K, C, 0, 0, "cuda:0").fill_(255)
    sb.semicrf_logz_fwd(*x, flags=flags, workspace=ws)
    return (sb.semicrf_seq_report(ws, B, T, K, C, 0, 0)[1].cpu().numpy(), sb.semicrf_scan_report(ws, B, T, K, C, 0, 0)[0][:, 0].cpu().numpy())


def test_the_report_tells_a_longer_first_attempt_from_a_second():
    B, T, K, C = 4, 3000, 37, 19
    x = labelled(B, T, K, C, 0.3, band=2)
    assert (score(x, B, T, K, C)[1] == 4).all()
    assert (score(x, B, T, K, C, sb.SEMICRF_CENTER | sb.SEMICRF_WARMUP(40))[1] == 3).all()


@pytest.mark.parametrize("B,T,K,C", [(16, 2000, 32, 32), (8, 2000, 32, 64), (4, 4000, 20, 48), (4, 4000, 64, 24), (2, 8000, 128, 12)])
@pytest.mark.parametrize("sd,own", [(0.3, True), (0.3, False), (1.0, True), (1.0, False), (1.5, True)])
def test_sharper_transitions_are_not_scanned_twice(B, T, K, C, sd, own):
    x = labelled(B, T, K, C, sd, own)
    lz, acc = score(x, B, T, K, C)
    print(f"[case] K={K} C={C} sd={sd} own {own} verified at {acc.tolist()}", flush=True)
    assert ((acc == 1) | (acc == 2)).all() and (acc == 1).mean() >= 0.75  # a boundary that takes longer is mended
    ref = score(x, B, T, K, C, sb.SEMICRF_CENTER | sb.SEMICRF_SEQUENTIAL_SCAN)[0]
    assert np.abs(lz - ref).max() <= 1e-10 * (T / 8)  # the bound of a boundary, and at most that many of them


@pytest.mark.parametrize("B,T,K,C,sd", [(2, 512, 8, 4, 1.5), (64, 256, 16, 24, 1.0), (64, 256, 16, 24, 1.5), (8, 1000, 34, 12, 1.0),
                                        (8, 1000, 34, 12, 2.0), (4, 4000, 100, 3, 2.0)])
def test_chosen_warm_ups_cost_no_digits(B, T, K, C, sd):
    """logZ in 64 bits, next to the sequential scan's: a few units in the last place, as after a warm-up of 1.5 K, although windows that
    agree in what they still contribute are accepted too."""
    x = labelled(B, T, K, C, sd)
    lz, acc = score(x, B, T, K, C)
    ref = score(x, B, T, K, C, sb.SEMICRF_CENTER | sb.SEMICRF_SEQUENTIAL_SCAN)[0]
    rel = (np.abs(lz - ref) / np.abs(ref)).max()
    print(f"[case] K={K} C={C} sd={sd} verified at {sorted(set(acc.tolist()))}, logZ differs by {rel:.1e}", flush=True)
    assert rel <= 1e-15
