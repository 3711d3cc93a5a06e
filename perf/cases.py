"""The calls a user of this library makes, over the sizes they are made at, for timing and comparing two builds.

A case is one call of a public entry point of ``paper_2604_18780_amd.binding`` on a batch of B sequences of up to T
positions with C labels and segments of up to K positions:

  op "train"     semicrf_fwd_bwd            logZ and the gradients of a mean negative log-likelihood (forward and backward)
  op "score"     semicrf_logz_fwd           logZ alone, as in validation (forward only)
  op "decode"    semicrf_viterbi            best segmentation, as in inference
  op "analyse"   semicrf_fwd_bwd_boundary   start / end projections and scalar boundaries with all their gradients, the
                 + semicrf_entropies        boundary posterior, and the two entropies formed from it
  op "durtrans"  semicrf_fwd_bwd_durtrans   one transition matrix per duration, with gradients

The other fields: "emis", the type the encoder hands its scores over in; "ragged", whether lengths are spread over
[T/2, T]; "segment", the mean length of the segments in the data; "trans_sd", how sharp the transition scores are (0.1:
as initialised, 1: trained); "band", 0 or the distance beyond which a label may not follow another (segment grammars;
forbidden pairs score -1e4).  Sizes are those of ``synth.CONFIGS`` and odd ones around them.
"""
import math

import torch

from paper_2604_18780_amd import binding

DTYPES = {"float32": torch.float32, "bfloat16": torch.bfloat16, "float16": torch.float16}
ACTIVE_MEAN = 2.0      # score of the label a position has in the data; everything else is unit noise around 0
FORBIDDEN = -1.0e4
DURTRANS_OPS = 400_000 * 64 * 24 * 24  # multiply-adds per pass and recurrence of the largest listed case
NODES = 400_000 * 24                   # positions times labels of the largest listed cases with one shared matrix


def _case(name, op, B, T, K, C, emis="float32", ragged=False, segment=12, trans_sd=0.1, band=0):
    c = dict(op=op, B=B, T=T, K=K, C=C, emis=emis, ragged=ragged, segment=segment, trans_sd=trans_sd, band=band)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a single short example, as in notebooks and tests: latency and launches are all there is
        _case("tiny_train", "train", 2, 512, 8, 4, segment=6),
        # named-entity sized batches: many short sentences, training and decoding
        _case("nlp_train", "train", 64, 256, 16, 24, ragged=True, segment=6),
        _case("nlp_decode", "decode", 64, 256, 16, 24, ragged=True, segment=6),
        # the same batches with a transition matrix for each duration
        _case("nlp_durtrans", "durtrans", 64, 256, 16, 24, ragged=True, segment=6),
        # phone segmentation: a wide label set, scores from an encoder that runs in bfloat16
        _case("speech_train", "train", 32, 2000, 32, 64, emis="bfloat16", ragged=True, segment=12),
        # a segment grammar over an odd number of labels, ragged batch of odd lengths, trained transitions
        _case("grammar_train", "train", 11, 3001, 37, 19, ragged=True, segment=15, trans_sd=1.0, band=2),
        # genome-scale sequences: training, validation, decoding, posterior analysis
        _case("genomic_train", "train", 4, 100_000, 64, 24, segment=40),
        _case("genomic_score", "score", 4, 100_000, 64, 24, segment=40),
        _case("genomic_decode", "decode", 4, 100_000, 64, 24, segment=40),
        _case("genomic_analyse", "analyse", 4, 100_000, 64, 24, segment=40),
        # ... and with a transition matrix for each duration, the most work a call does here
        _case("genomic_durtrans", "durtrans", 4, 100_000, 64, 24, segment=40),
        # one chromosome-sized sequence with long segments
        _case("longgen_train", "train", 1, 400_000, 512, 8, segment=150),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("train", "train", "train", "score", "decode", "decode", "analyse", "durtrans"))
    wide = op != "durtrans"
    C = _log_int(rng, 3, 64 if wide else 32)
    lanes = max(8, 1 << (C - 1).bit_length())
    K = _log_int(rng, 4, 64 * (64 // lanes) if wide else min(64 * (1024 // (C * C)), 8 * (1024 // C), 512))
    positions = NODES // C if wide else min(NODES // C, DURTRANS_OPS // (K * C * C))
    T = _log_int(rng, 96, min(100_000, positions))
    B = _log_int(rng, 1, max(1, min(64, positions // T)))
    # grammars whose labels are slow to mix are met on sequences of moderate length
    band = rng.choice((0, 2)) if op in ("train", "score") and T <= 4000 and C >= 8 else 0
    return _case(None, op, B, T, K, C, emis=rng.choice(("float32", "float32", "bfloat16", "float16")),
                 ragged=B > 1 and rng.random() < 0.7, segment=max(2, _log_int(rng, 3, max(4, K))),
                 trans_sd=rng.choice((0.1, 0.3, 1.0)), band=band)


def prepare(case, seed):
    B, T, K, C, op = (case[k] for k in ("B", "T", "K", "C", "op"))
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    normal = lambda *shape: torch.randn(*shape, generator=g, device=dev)  # noqa: E731
    lengths = torch.full((B,), T, dtype=torch.int32, device=dev)
    if case["ragged"]:
        lengths = torch.randint((T + 1) // 2, T + 1, (B,), generator=g, device=dev, dtype=torch.int32)
    trans = case["trans_sd"] * normal(C, C)
    if case["band"]:
        i = torch.arange(C, device=dev)
        d = (i[:, None] - i[None, :]).abs()
        trans = torch.where(torch.minimum(d, C - d) <= case["band"], trans, torch.full_like(trans, FORBIDDEN))
    dur = 0.1 * normal(K, C)
    # label path: a new segment begins at each position with probability 1/segment
    which = (torch.rand(B, T, generator=g, device=dev) < 1.0 / case["segment"]).cumsum(1)
    label = torch.randint(0, C, (B, T + 1), generator=g, device=dev).gather(1, which)
    emis = normal(B, T, C)
    emis.scatter_add_(2, label[:, :, None], torch.full((B, T, 1), ACTIVE_MEAN, device=dev))
    s = {"op": op, "emis": emis.to(DTYPES[case["emis"]]), "lengths": lengths, "trans": trans, "dur": dur}
    if op in ("train", "analyse", "durtrans"):
        s["weights"] = torch.full((B,), 1.0 / B, device=dev)
    f32 = lambda *shape: torch.empty(shape, dtype=torch.float32, device=dev)  # noqa: E731
    if op == "train":
        s["workspace"] = binding.alloc_workspace(B, T, K, C, 0, 1, dev)
        s["out"] = (f32(B), f32(B, T, C), f32(C, C), f32(K, C), f32(B, T, C))
    elif op == "score":
        s["workspace"] = binding.alloc_workspace(B, T, K, C, 0, 0, dev)
        s["out"] = f32(B)
    elif op == "decode":
        n = binding.semicrf_viterbi_workspace_bytes(B, T, K, C)
        ws = torch.empty(n + 256, dtype=torch.uint8, device=dev)
        off = (-ws.data_ptr()) % 256
        s["workspace"] = ws[off:off + n]
    elif op == "analyse":
        s["workspace"] = binding.alloc_workspace(B, T, K, C, 0, 1, dev)
        s["proj"] = (0.5 * normal(B, T, C), 0.5 * normal(B, T, C), normal(C), normal(C))
    elif op == "durtrans":
        s["workspace"] = binding.alloc_durtrans_workspace(B, T, K, C, 0, True, dev)
        s["trans3"] = (trans[None] + 0.1 * normal(K, C, C)).contiguous()
    return s


def run(s):
    op = s["op"]
    if op == "train":
        return binding.semicrf_fwd_bwd(s["emis"], s["lengths"], s["trans"], s["dur"], s["weights"],
                                       workspace=s["workspace"], out=s["out"])
    if op == "score":
        return binding.semicrf_logz_fwd(s["emis"], s["lengths"], s["trans"], s["dur"], workspace=s["workspace"],
                                        logz=s["out"])
    if op == "decode":
        return binding.semicrf_viterbi(s["emis"], s["lengths"], s["trans"], s["dur"], workspace=s["workspace"])
    if op == "durtrans":
        return binding.semicrf_fwd_bwd_durtrans(s["emis"], s["lengths"], s["trans3"], s["dur"], s["weights"],
                                                workspace=s["workspace"])
    ps, pe, pis, pie = s["proj"]
    out = binding.semicrf_fwd_bwd_boundary(s["emis"], s["lengths"], s["trans"], s["dur"], s["weights"], ps, pe, pis,
                                           pie, workspace=s["workspace"])
    out["h_pos"], out["h_bdy"] = binding.semicrf_entropies(out["pos_marg"], out["bdy_post"], s["lengths"])
    return out


def work(case):
    """Bytes: every input and output once.  Flops: one multiply-add (or add and compare) for each window entry and each
    label pair of a position, for each of the forward, the backward and the statistics' pass the call asks for."""
    B, T, K, C, op = (case[k] for k in ("B", "T", "K", "C", "op"))
    share = 0.75 if case["ragged"] else 1.0
    pos = share * B * T
    read = pos * C * (4 if case["emis"] == "float32" else 2)
    pair = K * C * C if op == "durtrans" else K * C + C * C
    passes = 1 if op in ("score", "decode") else 3
    table = 4 * (K * C + (K * C * C if op == "durtrans" else C * C))
    wrote = {"train": 8 * B * T * C + table, "durtrans": 8 * B * T * C + table, "score": 4 * B, "decode": 8 * B * T,
             "analyse": 16 * B * T * C + 4 * B * T + table}[op]
    if op == "analyse":
        # the projections; the entropies read the position marginals and the boundary posterior
        read += 2 * pos * C * 4 + pos * C * 4 + pos * 4
    return {"bytes": float(read + table + wrote), "flops": float(2 * passes * pos * pair)}


def tolerance(case):
    if case["op"] == "decode":
        # a run of one label can be split into the same durations in any order at the same score: ties that the last
        # bit of a 64-bit sum decides
        return {"rel": 1e-5, "differ": 2e-3}
    return {"rel": 1e-5}
