"""GPU parity of the Viterbi decode against the fp64 CPU oracle.

The best score is unique: it must match the oracle's (relative 1e-6: the score is returned in
fp32).  The best PATH need not be unique, so the decoded segmentation is checked for validity
(segments tile the sequence, one label each, no segment longer than K, flags and counts agree,
nothing beyond the sequence) and for optimality: its score, recomputed by the oracle's independent
path scorer, must equal the best score.  Ties are structural, not accidental (a run of one label
cut as 1+2 or as 2+1 tokens scores the same), and in the oracle rounding decides them, so the paths
themselves are not compared here (test_gpu_viterbi_ties.py compares those of the decode's own routes); the
fraction of tokens on which both decoders agree is printed.
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
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to(DEV)


def nan_pad(a, lengths):
    a = a.copy()
    for b in range(a.shape[0]):
        a[b, int(lengths[b]):] = np.nan
    return a


def check(w, terms=(None, None, None, None), center=True, label="", extra_flags=0, expect_chunked=None):
    print(f"[case] viterbi {label} B={w.B} T={w.T} K={w.K} C={w.C}", flush=True)
    ps, pe, pis, pie = terms
    flags = (sb.SEMICRF_CENTER if center else 0) | extra_flags
    n = sb.semicrf_viterbi_workspace_bytes(w.B, w.T, w.K, w.C)
    raw = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    off = (-raw.data_ptr()) % 256
    ws = raw[off:off + n]
    score, labels, starts, nseg = sb.semicrf_viterbi(
        dev(nan_pad(w.emis, w.lengths)), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur),
        dev(None if ps is None else nan_pad(ps, w.lengths)), dev(None if pe is None else nan_pad(pe, w.lengths)),
        dev(pis), dev(pie), flags, workspace=ws)
    acc, mis = sb.semicrf_scan_report(ws, w.B, w.T, w.K, w.C, 0, False)
    torch.cuda.synchronize()
    acc = acc.cpu().numpy()[:, 0]
    print(f"       chunk-parallel scan accepted for {int(acc.sum())} of {w.B} sequences, largest mismatch "
          f"{mis[:, 0].max().item():.2e}", flush=True)
    if expect_chunked is not None:
        assert np.all(acc == (1 if expect_chunked else 0))
    score = score.double().cpu().numpy()
    labels, starts, nseg = labels.cpu().numpy(), starts.cpu().numpy(), nseg.cpu().numpy()
    r_score, r_labels, r_starts, r_nseg = oracle.viterbi(w.emis, w.lengths, w.trans, w.dur, center=center,
                                                         proj_start=ps, proj_end=pe, pi_start=pis, pi_end=pie)
    assert np.all(np.isfinite(score))
    assert np.abs(score - r_score).max() <= 1e-6 * max(1.0, np.abs(r_score).max()), (score, r_score)
    for b in range(w.B):
        L = int(w.lengths[b])
        assert np.all(labels[b, L:] == -1) and np.all(starts[b, L:] == 0)
        assert nseg[b] == starts[b].sum()
        if L == 0:
            continue
        assert starts[b, 0] == 1 and labels[b, :L].min() >= 0 and labels[b, :L].max() < w.C
        got = oracle.path_score(w.emis[b], L, w.trans, w.dur, labels[b], starts[b], center=center,
                                proj_start=None if ps is None else ps[b], proj_end=None if pe is None else pe[b],
                                pi_start=pis, pi_end=pie)                 # also asserts the structure
        assert abs(got - r_score[b]) <= 1e-9 * max(1.0, abs(r_score[b])), (b, got, r_score[b])
    valid = np.arange(w.T)[None, :] < w.lengths[:, None]
    if valid.any():
        print(f"       same label on {np.mean(labels[valid] == r_labels[valid]):.4f} of the tokens, same start flag on "
              f"{np.mean(starts[valid] == r_starts[valid]):.4f}", flush=True)


@pytest.mark.parametrize("seed,B,T,K,C", [
    (1, 3, 40, 5, 3), (2, 4, 300, 8, 6), (3, 2, 700, 33, 24), (4, 5, 130, 1, 7),
    (5, 3, 90, 2, 5), (6, 2, 50, 80, 4), (7, 3, 257, 16, 64), (8, 6, 33, 7, 1), (9, 1, 1, 1, 1),
])
def test_random_ragged_cases(seed, B, T, K, C):
    w = synth.small_random(seed, B, T, K, C, ragged=True)
    if seed == 2:
        w.lengths[0] = 0
        w.lengths[1] = T
    check(w)
    rng = np.random.default_rng(200 + seed)
    terms = ((0.5 * rng.standard_normal((B, T, C))).astype(np.float32),
             (0.5 * rng.standard_normal((B, T, C))).astype(np.float32),
             rng.standard_normal(C).astype(np.float32), rng.standard_normal(C).astype(np.float32))
    check(w, terms, center=(seed % 2 == 0), label="with boundary terms")


def test_workload_shapes():
    check(synth.make("nlp"), label="nlp")
    check(synth.make("speech", B=4, T=600), label="speech shape")
    check(synth.make("genomic", T=6000, B=2), label="genomic shape")
    check(synth.make("longgen", T=3000), label="longgen shape")


def test_unsupported_sizes_are_refused():
    w = synth.small_random(61, 1, 8, 2, 70, ragged=False)
    with pytest.raises(sb.SemiCRFError) as ei:
        sb.semicrf_viterbi(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur))
    assert ei.value.status == -3


def test_full_size_genomic_decode():
    """The genomic workload at full size, as `bench.py --viterbi` runs it: best score against the
    stored oracle value (tests/golden/make_golden.py, oracle only), and the decoded segmentation
    validated and re-scored by the oracle's independent path scorer."""
    import os
    path = os.path.join(os.path.dirname(__file__), "golden", "full_genomic_viterbi.npz")
    if not os.path.exists(path):
        pytest.skip(f"{path} not generated")
    g = np.load(path)
    w = synth.make("genomic")
    score, labels, starts, nseg = sb.semicrf_viterbi(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur))
    torch.cuda.synchronize()
    score = score.double().cpu().numpy()
    labels, starts, nseg = labels.cpu().numpy(), starts.cpu().numpy(), nseg.cpu().numpy()
    assert np.abs(score - g["score"]).max() <= 1e-6 * np.abs(g["score"]).max()
    for b in range(w.B):
        L = int(w.lengths[b])
        got = oracle.path_score(w.emis[b], L, w.trans, w.dur, labels[b], starts[b])
        assert abs(got - g["score"][b]) <= 1e-9 * abs(g["score"][b]), (b, got, g["score"][b])
        assert nseg[b] == starts[b].sum()
    print(f"       segments per sequence {nseg} (oracle {g['nseg']})", flush=True)


def test_chunk_parallel_and_sequential_scans_give_the_same_score():
    w = synth.small_random(41, 3, 1500, 12, 10, ragged=True)
    w.lengths[:] = [1500, 1499, 64]
    check(w, label="default (chunk-parallel, verified)", expect_chunked=True)
    check(w, label="sequential", extra_flags=sb.SEMICRF_SEQUENTIAL_SCAN, expect_chunked=False)


def test_paths_that_do_not_merge_fall_back_to_the_sequential_scan():
    """A nearly deterministic two-label chain with weak emissions: the best path into a position
    depends on how the sequence started for thousands of positions, so the warmed-up chunk states
    differ from the true ones by more than one constant; the boundary check must fail and the
    sequential scan must deliver the result."""
    rng = np.random.default_rng(42)
    B, T, K, C = 2, 2000, 2, 2
    w = synth.small_random(42, B, T, K, C, ragged=False)
    w.emis[:] = (0.05 * rng.standard_normal((B, T, C))).astype(np.float32)
    w.trans[:] = np.array([[0.0, -40.0], [-40.0, 0.0]], dtype=np.float32)
    w.dur[:] = 0.0
    check(w, label="no merging", expect_chunked=False)



def test_both_trace_back_routes_write_the_same_path():
    """The trace-back in tiles, and the one by pointer doubling over all nodes that a flag asks for: same candidates, same
    rule for ties, same path."""
    w = synth.small_random(77, 3, 3000, 12, 6, ragged=True)
    dev = [torch.from_numpy(a).to(DEV) for a in (w.emis, w.lengths, w.trans, w.dur)]
    a = [o.cpu().numpy() for o in sb.semicrf_viterbi(*dev)]
    b = [o.cpu().numpy() for o in sb.semicrf_viterbi(*dev, flags=sb.SEMICRF_CENTER | sb.SEMICRF_VITERBI_GLOBAL_TRACE)]
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert a[3].sum() > 0
