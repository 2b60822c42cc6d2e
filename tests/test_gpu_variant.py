"""Parity of the paper's own model on the GPU (section 5.2: encoder 64/128/128,
one Mamba block with d_state 8, decoder 64/32/1; features 26 x 22 and 41 x 20)
with the fp64 oracle, and of the Top-k score (Eq. (12)) with the oracle's.

Scores are held to the fp32 tolerance and ranking check of the other
scoring tests. The Top-k score is a ratio of sums of exact fp64 products
(fp32 latency times fp32 weight): only the summation order differs, so the
three values must match to rel 1e-12."""
import numpy as np
import pytest
import torch

from oracle import metric as omet
from paper_2604_12891_amd import binding as tb
from paper_2604_12891_amd import workload as wl
from tests.parity import assert_scores_match, oracle_scores
from tests.test_gpu_score import _model, _sample, _score

pytestmark = pytest.mark.gpu

PAPER = ["paper_B4096_L26_F22_f32", "paper_B4096_L41_F20_f32"]


@pytest.mark.parametrize("f32_matmul", ["split", "native"])
@pytest.mark.parametrize("name", PAPER)
def test_paper_model_small_batch(name, f32_matmul):
    """300 programs (several tiles and a ragged tail), perturbed weights."""
    w = wl.WORKLOADS[name]
    print(f"tcl_score {name} B=300 perturbed {f32_matmul}", flush=True)
    blob, X, lengths = wl.make_workload(name, B=300, perturb=True)
    g = _score(_model(w.model, blob, f32_matmul=f32_matmul), X, lengths)
    assert_scores_match(g, oracle_scores(blob, X, lengths, w.model), "f32", name)


@pytest.mark.parametrize("f32_matmul", ["split", "native"])
@pytest.mark.parametrize("name", PAPER)
def test_paper_model_full_size_sampled(name, f32_matmul):
    """The full batch in the benchmark's launch configuration, compared on a
    sample that the oracle scores (programs are independent)."""
    w = wl.WORKLOADS[name]
    print(f"tcl_score {name} full batch {f32_matmul}", flush=True)
    blob, X, lengths = wl.make_workload(name)
    g = _score(_model(w.model, blob, f32_matmul=f32_matmul), X, lengths)
    assert np.all(np.isfinite(g))
    idx = _sample(lengths, 96)
    assert_scores_match(g[idx], oracle_scores(blob, X[idx], lengths[idx], w.model), "f32", name)


def test_paper_model_edge_lengths():
    """One program; every program of length 1; every program at full length."""
    w = wl.WORKLOADS["paper_B4096_L41_F20_f32"]
    blob, X, lengths = wl.make_workload(w.name, B=70, perturb=True)
    m = _model(w.model, blob)
    for what, lens in [("one", None), ("len1", np.ones(70, np.int32)), ("full", np.full(70, w.L, np.int32))]:
        print(f"tcl_score paper edge {what}", flush=True)
        if lens is None:
            Xs, ls = X[:1], lengths[:1]
        else:
            Xs = X.copy()
            Xs[:, :, :] = wl.make_inputs(70, w.L, w.model.F, w.L, w.L, np.random.default_rng(3))[0]
            Xs[np.arange(w.L)[None, :] >= lens[:, None]] = 0.0
            ls = lens
        assert_scores_match(_score(m, Xs, ls), oracle_scores(blob, Xs, ls, w.model), "f32", what)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_variant_pieces_on_other_shapes(dtype):
    """The pieces one at a time on other shapes: F = 22 with the one-Linear
    encoder (the padded-feature path, also for bf16 models), one hidden
    encoder layer, and the three-layer decoder on a d_state 16 model."""
    shapes = [wl.ModelShape(F=22, d_model=64, d_inner=128, dt_rank=4, n_layers=2, head_hidden=64),
              wl.ModelShape(F=22, d_model=64, d_inner=128, dt_rank=4, n_layers=2, head_hidden=64, dec_hidden2=48)]
    if dtype == "f32":
        shapes.append(wl.ModelShape(F=164, d_model=64, d_inner=128, dt_rank=4, n_layers=1, head_hidden=128,
                                    enc_hidden=(96,), dec_hidden2=16))
    for i, shape in enumerate(shapes):
        print(f"tcl_score variant piece {i} {dtype}", flush=True)
        rng = np.random.default_rng(40 + i)
        blob = wl.init_params(shape, rng, perturb=True)
        if dtype == "bf16":
            blob = wl.round_to_bf16(blob)
        X, lengths = wl.make_inputs(150, 25, shape.F, 1, 25, rng)
        g = _score(_model(shape, blob, dtype=dtype), X, lengths)
        assert_scores_match(g, oracle_scores(blob, X, lengths, shape), dtype, f"piece {i}")


def test_paper_model_long_sequences_small_batch():
    """A few long programs: the small-batch scan with d_state 8."""
    shape = wl.PAPER_GPU
    rng = np.random.default_rng(7)
    blob = wl.init_params(shape, rng, perturb=True)
    X, lengths = wl.make_inputs(6, 256, shape.F, 100, 256, rng)
    print("tcl_score paper model B=6 L=256", flush=True)
    g = _score(_model(shape, blob), X, lengths)
    assert_scores_match(g, oracle_scores(blob, X, lengths, shape), "f32", "long")


# ---------------------------------------------------------------- Eq. (12)

def _metric_inputs(n_seg, lo, hi, seed, ties=False):
    rng = np.random.default_rng(seed)
    sizes = rng.integers(lo, hi + 1, size=n_seg)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(offs[-1])
    s = rng.standard_normal(n).astype(np.float32)
    if ties:
        s = (np.round(s * 4) / 4).astype(np.float32)
        s[rng.random(n) < 0.05] = np.nan
    lat = rng.lognormal(-7.0, 1.0, n).astype(np.float32)  # seconds
    w = rng.integers(1, 9, size=n_seg).astype(np.float32)
    return offs, s, lat, w


def _gpu_metric(offs, s, lat, w, k):
    d = lambda a: torch.from_numpy(a).cuda()
    out = tb.topk_score(d(s), d(lat), d(w), d(offs), k)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("k", [1, 5, 64, 1024])
def test_topk_score_matches_oracle(k):
    """Segments of 0 to 300 candidates (empty ones included), ties and NaN
    scores."""
    offs, s, lat, w = _metric_inputs(60, 0, 300, 100 + k, ties=True)
    print(f"tcl_topk_score k={k}", flush=True)
    g = _gpu_metric(offs, s, lat, w, k)
    o = omet.top_k_score(s, lat, offs, w, k)
    np.testing.assert_allclose(g, np.array(o), rtol=1e-12)


def test_topk_score_at_scale():
    """512 subgraphs of up to 4,000 measured candidates each (Top-1 and
    Top-5, the paper's two reported values)."""
    offs, s, lat, w = _metric_inputs(512, 1000, 4000, 9)
    for k in (1, 5):
        print(f"tcl_topk_score 512 segments k={k}", flush=True)
        g = _gpu_metric(offs, s, lat, w, k)
        np.testing.assert_allclose(g, np.array(omet.top_k_score(s, lat, offs, w, k)), rtol=1e-12)
