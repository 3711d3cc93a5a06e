"""Nothing may be read before the call has written it: every entry point and route in a workspace full of 0xff (NaN, -1), for an odd
and an even number of intervals, so that the first interval of a sequence falls to every wave of a workgroup."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_parity import assert_outputs_match_oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(5, 3), (20, 8), (196, 9), (400, 8), (40, 24), (100, 20), (120, 30), (30, 40), (60, 64)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("K,C", SHAPES)
@pytest.mark.parametrize("T", [330, 360])
@pytest.mark.parametrize("flag", [0, sb.SEMICRF_ONE_WAVE_SCAN, sb.SEMICRF_TWO_WAVE_SCAN, sb.SEMICRF_SEQUENTIAL_SCAN,
                                  sb.SEMICRF_MARGINALS_INTERVAL, sb.SEMICRF_LOW_MEMORY, sb.SEMICRF_MATRIX_SCAN])
def test_training_and_scoring(flag, T, K, C):
    w = synth.small_random(K + T, 4, T, K, C, ragged=True)
    w.lengths[:] = [T, 331 - 40, 0, T - 1]
    x = dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur)
    flags = sb.SEMICRF_CENTER | flag
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur)
    for delta in (32, 40, 0):
        ws = sb.alloc_workspace(w.B, T, K, C, delta, sb.grad_workspace_kind(flags), DEV).fill_(255)
        out = sb.semicrf_fwd_bwd(*x, None, delta, flags, workspace=ws)
        acc, _ = sb.semicrf_scan_report(ws, w.B, T, K, C, delta, sb.grad_workspace_kind(flags))
        assert ((acc >= 0) & (acc <= 3)).all()
        assert_outputs_match_oracle([o.double().cpu().numpy() for o in out], r)
        ws = sb.alloc_workspace(w.B, T, K, C, delta, sb.fwd_workspace_kind(flags), DEV).fill_(255)
        lz = sb.semicrf_logz_fwd(*x, delta, flags, workspace=ws).double().cpu().numpy()
        assert np.abs(lz - r.logz).max() <= 1e-5 * np.abs(r.logz).max()


@pytest.mark.parametrize("K,C", SHAPES)
@pytest.mark.parametrize("flag", [0, sb.SEMICRF_SEQUENTIAL_SCAN, sb.SEMICRF_VITERBI_GLOBAL_TRACE])
def test_decoding(flag, K, C):
    for T in (1, 330, 360):
        w = synth.small_random(K + T, 4, T, K, C, ragged=True)
        w.lengths[:] = [T, T // 2 + 1, 0, T]
        ws = torch.full((sb.semicrf_viterbi_workspace_bytes(4, T, K, C) + 256,), 255, dtype=torch.uint8, device=DEV)
        off = (-ws.data_ptr()) % 256
        score, labels, starts, nseg = sb.semicrf_viterbi(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur),
                                                         flags=sb.SEMICRF_CENTER | flag, workspace=ws[off:ws.numel() - 256 + off])
        ref = oracle.viterbi(w.emis, w.lengths, w.trans, w.dur)[0]
        assert np.abs(score.double().cpu().numpy() - ref).max() <= 1e-6 * max(1.0, np.abs(ref).max())
        for b in range(4):
            L = int(w.lengths[b])
            if L:
                got = oracle.path_score(w.emis[b], L, w.trans, w.dur, labels[b].cpu().numpy(), starts[b].cpu().numpy())
                assert abs(got - ref[b]) <= 1e-9 * max(1.0, abs(ref[b]))
            assert nseg[b].item() == starts[b].sum().item()


@pytest.mark.parametrize("K,C", [(5, 3), (40, 24), (12, 32), (400, 8), (512, 8), (130, 7)])
@pytest.mark.parametrize("flag", [0, sb.SEMICRF_SEQUENTIAL_SCAN])
def test_duration_dependent_transitions(flag, K, C):
    w = synth.small_random(K, 3, 260, K, C, ragged=True)
    w.lengths[:] = [260, 0, 233]
    t3 = synth.duration_transitions(w, 3, 0.3)
    r = oracle.fwd_bwd_durtrans(w.emis, w.lengths, t3, w.dur)
    for delta in (0, 40):
        ws = sb.alloc_durtrans_workspace(3, 260, K, C, delta, True, DEV).fill_(255)
        out = sb.semicrf_fwd_bwd_durtrans(dev(w.emis), dev(w.lengths), dev(t3), dev(w.dur), None, delta, sb.SEMICRF_CENTER | flag,
                                          workspace=ws)
        assert_outputs_match_oracle([o.double().cpu().numpy() for o in out], r)


@pytest.mark.parametrize("K,C", SHAPES)
def test_boundary_terms(K, C):
    w = synth.small_random(K, 3, 360, K, C, ragged=True)
    w.lengths[:] = [360, 0, 291]
    ps, pe, pis, pie = synth.boundary_terms(w)
    ws = sb.alloc_workspace(3, 360, K, C, 40, 1, DEV).fill_(255)
    out = sb.semicrf_fwd_bwd_boundary(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur), None, dev(ps), dev(pe), dev(pis), dev(pie),
                                      40, workspace=ws)
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, proj_start=ps, proj_end=pe, pi_start=pis, pi_end=pie, boundary=True)
    for name in ("logz", "grad_emis", "pos_marg", "grad_proj_start", "grad_proj_end", "bdy_post", "grad_trans", "grad_dur",
                 "grad_pi_start", "grad_pi_end"):
        g, ref = out[name].double().cpu().numpy(), getattr(r, name)
        assert np.abs(g - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max()), name
