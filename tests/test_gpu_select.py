"""Parity of the score consumers with the oracle (oracle/select.py), bit-exact
on indices: per-segment top-K (tcl_topk) and the RDU selection of Alg. 1
(tcl_rdu_select).

Top-K compares fp32 scores exactly on both sides, so the indices must be
identical. The RDU selection is an argmax over fp64 t_s; the oracle
computes Eq. (2)-(3) two-pass from their definitions and the kernel from
running sums, so the two t_s differ in the last bits; the selected sequences
must still be identical (seeded continuous scores have no near-ties at that
level) -- and if a step ever differs, the test reports whether the oracle's
own t_s of the two picks tie to 1e-12.
"""
import numpy as np
import pytest
import torch

from oracle import select as osel
from paper_2604_12891_amd import workload as wl

pytestmark = pytest.mark.gpu


def _tb():
    from paper_2604_12891_amd import binding as tb
    return tb


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype)


@pytest.mark.parametrize("sizes,K", [([0, 1, 5, 64, 65, 300, 4096], 64), ([1000, 3, 2500], 1),
                                     ([70000], 1024), ([257, 1024, 1025], 256), ([5, 7], 10)])
def test_topk_matches_oracle(sizes, K):
    print(f"topk sizes={sizes} K={K}", flush=True)
    rng = np.random.default_rng(sum(sizes) + K)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    s = (0.3 * rng.standard_normal(offs[-1])).astype(np.float32)
    s[rng.random(offs[-1]) < 0.02] = np.nan          # unscored programs
    s[rng.random(offs[-1]) < 0.05] = 0.125           # ties
    s[rng.random(offs[-1]) < 0.01] = -0.0
    got = _tb().topk(_dev(s, torch.float32), _dev(offs, torch.int32), K)
    torch.cuda.synchronize()
    ref = osel.topk_segments(s, offs, K)
    assert np.array_equal(got.cpu().numpy(), ref)


@pytest.mark.parametrize("K", [64, 65, 256, 1024])
@pytest.mark.parametrize("kind", ["random", "equal", "close", "nan"])
def test_topk_radix_edges(kind, K):
    """Segments around K and around the 8,192 keys that stay in registers;
    scores all equal, or closer than the first digits tell apart (more
    candidates than fit, so further digits and the index order decide), or
    NaN but for a few."""
    sizes = [K - 1, K, K + 1, 8191, 8192, 8193, 16385]
    print(f"topk edges {kind} K={K}", flush=True)
    rng = np.random.default_rng(K)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(offs[-1])
    s = {"random": lambda: 0.3 * rng.standard_normal(n),
         "equal": lambda: np.full(n, -0.5),
         "close": lambda: 1.0 + rng.integers(0, 40, n) * 2.0 ** -23,
         "nan": lambda: np.where(rng.random(n) < 0.002, rng.standard_normal(n), np.nan)}[kind]().astype(np.float32)
    got = _tb().topk(_dev(s, torch.float32), _dev(offs, torch.int32), K)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), osel.topk_segments(s, offs, K))


def test_topk_of_a_scored_round():
    """The top 64 of the headline tuning round's scores as the model would
    produce them (seeded score-like values, one segment per 512 candidates)."""
    w = wl.WORKLOADS["score_B4096_L25_d256_f32"]
    rng = np.random.default_rng(3)
    s = (0.1 * rng.standard_normal(w.B)).astype(np.float32)
    offs = np.arange(0, w.B + 1, 512, dtype=np.int32)
    got = _tb().topk(_dev(s, torch.float32), _dev(offs, torch.int32), 64).cpu().numpy()
    assert np.array_equal(got, osel.topk_segments(s, offs, 64))


def _rdu_case(N, n_ops, n_init, seed):
    rng = np.random.default_rng(seed)
    s = (0.3 * rng.standard_normal(N)).astype(np.float32)
    p = rng.random(n_ops) + 0.2
    op = rng.choice(n_ops, N, p=p / p.sum()).astype(np.int32)
    init = rng.choice(N, n_init, replace=False).astype(np.int32)
    return s, op, init


def _check_rdu(s, op, n_ops, init, n_select):
    sel, cnt = _tb().rdu_select(_dev(s, torch.float32), _dev(op, torch.int32), n_ops, _dev(init, torch.int32),
                                n_select)
    torch.cuda.synchronize()
    got = sel.cpu().numpy().tolist()
    c = int(cnt.cpu().numpy()[0])
    ref = osel.rdu_select(s.astype(np.float64), op, n_ops, init, n_select)
    assert c == len(ref)
    if got[:c] != ref:
        k = next(i for i in range(c) if got[i] != ref[i])
        f = osel.normalise(s.astype(np.float64))
        lab = set(init.tolist()) | set(ref[:k])
        tt = osel.rdu_scores(f, lab, [got[k], ref[k]])
        pytest.fail(f"step {k}: gpu {got[k]} oracle {ref[k]}; oracle t_s {tt[0]!r} vs {tt[1]!r}")
    assert all(g == -1 for g in got[c:])


@pytest.mark.parametrize("N,n_ops,n_init,n_select", [(50, 1, 1, 10), (300, 4, 10, 40), (1000, 8, 32, 64),
                                                     (5000, 16, 64, 32), (64, 3, 60, 10)])
def test_rdu_select_matches_oracle(N, n_ops, n_init, n_select):
    print(f"rdu N={N} ops={n_ops} init={n_init} select={n_select}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, N + n_ops)
    _check_rdu(s, op, n_ops, init, n_select)


def test_rdu_select_budgets_bind_and_pool_runs_out():
    """Skewed operator types so that budgets bind and candidates are dropped;
    then more selections asked than candidates left (the count reports it)."""
    rng = np.random.default_rng(9)
    N = 400
    s = (0.3 * rng.standard_normal(N)).astype(np.float32)
    op = np.where(rng.random(N) < 0.9, 0, 1 + rng.integers(0, 3, N)).astype(np.int32)
    init = rng.choice(N, 8, replace=False).astype(np.int32)
    _check_rdu(s, op, 4, init, 50)
    small_s, small_op = s[:20].copy(), np.zeros(20, np.int32)
    _check_rdu(small_s, small_op, 1, np.array([3, 7], np.int32), 30)


def _check_rdu_pool(s, op, n_ops, init, n_select):
    sel, cnt = _tb().rdu_select(_dev(s, torch.float32), _dev(op, torch.int32), n_ops, _dev(init, torch.int32),
                                n_select)
    torch.cuda.synchronize()
    got = sel.cpu().numpy().tolist()
    c = int(cnt.cpu().numpy()[0])
    ref = osel.rdu_select_pool(s.astype(np.float64), op, n_ops, init, n_select)
    assert c == len(ref) and got[:c] == ref, (got[:c], ref)


def test_rdu_select_grid_stride_pool():
    """A pool of 1.2 M programs: more candidates than one pass of the
    selection grid covers (1024 blocks x 256 threads x 4), so every kernel's
    grid-stride loop runs more than once; 20 operator types, 64 initial
    programs, 6 selections, against the oracle's blocked form."""
    N, n_ops, n_init, n_sel = 1_200_000, 20, 64, 6
    assert N > 1024 * 256 * 4
    print(f"rdu pool N={N} init={n_init} select={n_sel}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, 77)
    _check_rdu_pool(s, op, n_ops, init, n_sel)


def test_rdu_select_large_initial_set():
    """More initial labeled programs (8,500) than the sorted-set path holds
    (8,192): the distances to the initial set come from the direct pass."""
    N, n_ops, n_init, n_sel = 60_000, 8, 8_500, 3
    print(f"rdu N={N} init={n_init} select={n_sel}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, 78)
    _check_rdu_pool(s, op, n_ops, init, n_sel)


@pytest.mark.parametrize("kind", ["random", "sorted", "coarse", "constant", "skewed_ops"])
def test_rdu_select_short_list(kind):
    """Pools large enough (over 131,072) for launches on a short list of
    candidates: random scores; sorted ones (the best all in a few blocks);
    scores on a grid of 64 values (ties, and lists that overflow); equal
    scores; an operator type that takes most of the pool, so that budgets mask
    listed candidates."""
    N, n_ops, n_init, n_sel = 140_003, 6, 40, 14
    print(f"rdu list {kind}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, 200)
    rng = np.random.default_rng(201)
    if kind == "sorted":
        s = np.sort(s)
    elif kind == "coarse":
        s = (np.round(s * 16) / 16).astype(np.float32)
    elif kind == "constant":
        s[:] = 0.25
    elif kind == "skewed_ops":
        op = np.where(rng.random(N) < 0.97, 0, 1 + rng.integers(0, n_ops - 1, N)).astype(np.int32)
    _check_rdu_pool(s, op, n_ops, init, n_sel)


def test_rdu_select_beside_other_work():
    """Selections on a short list while products on another stream hold the
    CUs, so that the blocks a launch on the list has no work for start late:
    the same selections as alone."""
    N, n_ops, n_init, n_sel = 1_000_003, 12, 40, 96
    print(f"rdu beside other work N={N}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, 300)
    args = (_dev(s, torch.float32), _dev(op, torch.int32), n_ops, _dev(init, torch.int32), n_sel)
    alone, count = _tb().rdu_select(*args)
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(12):
            torch.mm(a, a)
    got, c = _tb().rdu_select(*args)
    torch.cuda.synchronize()
    assert torch.equal(c, count) and torch.equal(got, alone)


def _least_us(f, calls=3, rounds=7):
    """The least time of a call, over rounds of a few calls each."""
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / calls * 1e3)
    return best


@pytest.mark.parametrize("kind", ["constant", "coarse"])
def test_rdu_select_pools_that_defeat_the_list(kind):
    """Equal scores, and 64 different ones, give short lists that are empty or
    overflow: the call costs what it costs with too few initial programs for
    the list (24: passes over the whole pool only), not a multiple (it was
    2.0 and 2.2 times, and is within 10 %)."""
    N, n_ops, n_sel = 1_000_003, 20, 64
    print(f"rdu without a list {kind}", flush=True)
    s, op, init = _rdu_case(N, n_ops, 1024, 400)
    s = np.full(N, 0.25, np.float32) if kind == "constant" else (np.round(s * 16) / 16).astype(np.float32)
    s, op, init = _dev(s, torch.float32), _dev(op, torch.int32), _dev(init, torch.int32)
    ws = torch.empty(_tb().lib().tcl_rdu_workspace_bytes(N, n_ops), dtype=torch.uint8, device="cuda")
    us = [_least_us(lambda i=i: _tb().rdu_select(s, op, n_ops, i, n_sel, workspace=ws)) for i in (init, init[:24])]
    assert us[0] < 1.4 * us[1], us


def _rdu_bytes_without_list(N, n_ops):
    def up(b):
        return (b + 255) // 256 * 256
    grid = min((N + 255) // 256, 1024)
    return 256 + up(8 * N) + up(8 * n_ops) + 2 * up(4 * (n_ops + 1)) + up(8 * grid) + up(16 * grid) + up(8 * 8192) + 256


@pytest.mark.parametrize("N", [200_003, 600_001])
@pytest.mark.parametrize("kind", ["normal", "coarse", "ties", "constant", "lognormal", "sorted", "budgets", "nan",
                                  "few", "many_initial"])
def test_rdu_select_without_room_for_the_list(N, kind):
    """A workspace of the size that large pools needed before they had the
    short list is accepted, nothing past its end is written, and the
    selections are those with the list: 200 of them, so that lists come to
    little, are waited for and tried again; one byte less is refused."""
    n_ops, n_init, n_sel = 9, 9_000 if kind == "many_initial" else 48, 200
    print(f"rdu without room {kind} N={N}", flush=True)
    s, op, init = _rdu_case(N, n_ops, n_init, 500)
    rng = np.random.default_rng(501)
    if kind in ("coarse", "ties"):
        step = 16 if kind == "coarse" else 1000
        s = (np.round(s * step) / step).astype(np.float32)
    elif kind == "constant":
        s[:] = -3.0
    elif kind == "lognormal":
        s = np.exp(10 * s).astype(np.float32)
    elif kind == "sorted":
        s = np.sort(s)
    elif kind == "budgets":  # most programs of one type, some of types that are never selected
        op = np.where(rng.random(N) < 0.9, 0, rng.integers(-2, n_ops + 2, N)).astype(np.int32)
    elif kind == "few":  # the pool runs out: most programs are of no type, and each type's budget is one
        op = np.where(rng.random(N) < 0.999, -1, op).astype(np.int32)
    elif kind == "nan":
        s[np.setdiff1d(rng.integers(0, N, N // 50), init)] = np.nan
    s, op, init = _dev(s, torch.float32), _dev(op, torch.int32), _dev(init, torch.int32)
    tb = _tb()
    least = _rdu_bytes_without_list(N, n_ops)
    assert least < tb.lib().tcl_rdu_workspace_bytes(N, n_ops)
    assert _rdu_bytes_without_list(131_072, n_ops) == tb.lib().tcl_rdu_workspace_bytes(131_072, n_ops)
    listed, count = tb.rdu_select(s, op, n_ops, init, n_sel)
    buf = torch.full((least + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    plain, c = tb.rdu_select(s, op, n_ops, init, n_sel, workspace=buf[:least])
    torch.cuda.synchronize()
    assert torch.equal(count, c) and torch.equal(listed, plain)
    assert (int(c) < n_sel) == (kind in ("few", "budgets")), int(c)
    assert (buf[least:] == 0x5A).all() and not (buf[:least] == 0x5A).all()
    st = tb.lib().tcl_rdu_select(N, s.data_ptr(), op.data_ptr(), n_ops, init.data_ptr(), n_init, n_sel,
                                 plain.data_ptr(), c.data_ptr(), buf.data_ptr(), least - 1, None)
    assert st == -3  # TCL_ERR_WORKSPACE


@pytest.mark.parametrize("kind", ["equal", "close"])
def test_topk_of_crowded_scores_costs_no_multiple(kind):
    """More segments than CUs whose scores are equal, or closer than the first
    digit tells apart: they take at most 1.6 times the time of spread ones (2.0
    and 1.7 times with one workgroup a CU and one atomic a key)."""
    n_seg, seg = 300, 600
    print(f"topk crowded {kind}", flush=True)
    offs = _dev(np.arange(n_seg + 1) * seg, torch.int32)
    spread = torch.randn(n_seg * seg, device="cuda")
    s = torch.full_like(spread, 0.5) if kind == "equal" else 1 + 1e-5 * spread
    us = [_least_us(lambda x=x: _tb().topk(x, offs, 10), calls=100) for x in (s, spread)]
    assert us[0] < 1.6 * us[1], us
