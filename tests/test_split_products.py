"""The wide contractions as split float32 products (csrc/split.h,
csrc/k_delayed.hip): every tile of the forward and of the block update at its
edges, whole and ragged, and operands of very different magnitudes, against
the CPU oracle.

Tolerance: the 1e-4 gate of the parity tests for whole parameter blocks.  For
the magnitudes test the same 1e-4 holds for every hidden unit by itself:
each row of W1 has its own scale, so a unit's relative error (float32
rounding of sums of at most 200 terms, about 1e-6) does not depend on the
other units' magnitudes.
"""

import numpy as np
import pytest

import cases
from oracle import method as M
from test_gpu_parity import TOL, _check, _momentum_run, _oracle, _run_gpu

pytestmark = pytest.mark.gpu

# name -> (case, mode, tile it is there for)
TILES = {
    # forward tiles by rows per group: 32 (one padded 16-row minibatch), 64
    # (33 samples, 48 rows), 128 (65 samples, 80 rows; 150: two row tiles)
    "rows_16": (cases.case("mlp", 3, 1, 2, 1, B=16, IN=65, H=65, C=40, N=90, lr=0.1, seed=201), "eager"),
    "rows_48": (cases.case("mlp", 4, 2, 2, 1, B=33, IN=190, H=130, C=70, N=90, lr=0.05, seed=202), "eager"),
    "rows_80": (cases.case("mlp", 2, 2, 2, 1, B=65, IN=320, H=100, C=130, N=90, lr=0.05, seed=203), "eager"),
    "rows_160": (cases.case("mlp", 2, 1, 1, 2, B=150, IN=129, H=192, C=33, N=90, lr=0.05, seed=204), "eager"),
    # few rows over weights beyond the cache (71 MB for 16 rows, 273 MB for 32):
    # float32 16-column blocks, ragged in rows and units
    "stream_16": (cases.case("mlp", 16, 4, 1, 2, B=13, IN=4090, H=270, C=20, N=90, lr=0.05, seed=225), "eager"),
    "stream_32": (cases.case("mlp", 16, 2, 1, 1, B=23, IN=4090, H=1035, C=20, N=90, lr=0.05, seed=226), "eager"),
    # 128 x 256 tiles, full and ragged in rows, units and features; the block
    # update in 64 x 64 tiles
    "delayed_full": (cases.case("mlp", 16, 4, 4, 2, B=32, IN=512, H=256, C=7, N=300, sigma=0.5, lr=0.05, seed=205),
                     "delayed"),
    "delayed_ragged": (cases.case("mlp", 12, 3, 3, 2, B=27, IN=333, H=300, C=37, N=300, sigma=0.5, lr=0.05, seed=206),
                       "delayed"),
    # 256 x 256 forward tiles (16 groups of 256 rows, 1024 units, 4 splits of
    # 1024 features)
    "delayed_256": (cases.case("mlp", 32, 2, 8, 1, B=16, IN=4096, H=1024, C=5, N=300, sigma=0.5, lr=0.05, seed=207),
                    "delayed"),
    # the same tiles with minibatches that do not fill their padded rows
    "delayed_256_ragged": (cases.case("mlp", 32, 2, 8, 1, B=13, IN=4096, H=1024, C=5, N=300, sigma=0.5, lr=0.05, seed=227),
                           "delayed"),
    # 256 x 256 block-update tiles, ragged in features (16 clusters of 256 rows,
    # 512 units, 4160 features: 17 column tiles, the last of 64)
    "delayed_update_256": (cases.case("mlp", 32, 2, 4, 2, B=32, IN=4150, H=500, C=5, N=300, sigma=0.5, lr=0.05, seed=228),
                           "delayed"),
    # 128 x 128 block-update tiles, ragged (320 units, 3008 features)
    "delayed_update_128": (cases.case("mlp", 16, 4, 2, 2, B=9, IN=3001, H=310, C=5, N=300, sigma=0.5, lr=0.05, seed=208),
                           "delayed"),
    # more than 32 samples under AUTO (W1 of 2^19 and more, (K1 - 1) * B <= H):
    # whole and ragged minibatches (Gram tiles across steps), both heads, one
    # step per block, the Gram blocks in feature splits
    "wide_64": (cases.case("mlp", 4, 2, 4, 2, B=64, IN=2048, H=256, C=7, N=300, sigma=0.5, lr=0.02, seed=221), "auto"),
    "wide_40": (cases.case("mlp", 6, 3, 3, 2, B=40, IN=1900, H=300, C=20, N=300, sigma=0.5, lr=0.02, seed=222), "auto"),
    "wide_100_c50": (cases.case("mlp", 4, 2, 3, 2, B=100, IN=2100, H=250, C=50, N=300, sigma=0.5, lr=0.02, seed=223), "auto"),
    "wide_128_c33": (cases.case("mlp", 2, 1, 2, 1, B=128, IN=4096, H=128, C=33, N=300, sigma=0.5, lr=0.02, seed=224), "auto"),
    "wide_one_step": (cases.case("mlp", 4, 4, 1, 2, B=33, IN=3000, H=192, C=3, N=300, sigma=0.5, lr=0.02, seed=225), "auto"),
    # one step per block, one sample: the shortest contractions
    "delayed_one_sample": (cases.case("mlp", 2, 1, 1, 2, B=1, IN=64, H=64, C=3, N=30, lr=0.1, seed=209), "delayed"),
}


@pytest.mark.parametrize("name", sorted(TILES))
def test_tiles_match_oracle(name, gpu_lib):
    c, mode = TILES[name]
    rounds = 1 if "256" in name else 2
    got, idx, _ = _run_gpu(c, rounds, mode)
    _check(c, got, idx, *_oracle(c, rounds), mode=mode)


@pytest.mark.parametrize("P,S,K1,K2,B,IN,H", [(32, 2, 4, 2, 32, 4150, 500), (32, 2, 4, 2, 32, 4096, 512),
                                              (16, 4, 2, 2, 9, 3001, 310), (4, 2, 2, 2, 7, 130, 70)],
                         ids=["256_ragged", "256", "128", "64"])
def test_heavy_ball_block_update_tiles(P, S, K1, K2, B, IN, H, gpu_lib):
    """The block update's tiles with buffers: parameters and every learner's
    buffers against the oracle (its run with the decisions at rounding that the
    kernels took)."""
    c = cases.case("mlp", P, S, K1, K2, B=B, IN=IN, H=H, C=5, N=300, sigma=0.5, lr=0.01, momentum=0.9,
                   weight_decay=1e-3, seed=229)
    got, vgot, idx, stats = _momentum_run(c, "delayed", rounds=1)
    assert "buffer_update_gemm" in stats
    st, mon, rerun = _oracle(c, 1)
    _check(c, got, idx, st, mon, rerun, mode="delayed")
    # A decision that the mean of the parameters hides moves its own learner's buffer.
    prob = cases.oracle_problem(c)
    ok, det = cases.branch_parity(prob, vgot, st.V, mon, lambda flips: M.run(prob, 1, flips=flips).V)
    assert ok, det


@pytest.mark.parametrize("name", [n for n in sorted(TILES) if n.startswith("wide")])
def test_wide_minibatch_schedule(name, gpu_lib):
    """AUTO takes the delayed schedule for these; set_batch moves the handle
    between it, the 32-sample form and eager rounds."""
    from paper_1903_05133_amd import HierAvg
    from dataclasses import replace
    c, _ = TILES[name]
    prob = cases.oracle_problem(c)
    st = M.create(prob)
    print(f"[gpu case] schedule {c}", flush=True)
    with HierAvg(config=cases.native_config(c)) as h:
        for B in (c["B"], 20, c["B"] - 1):
            h.set_batch(B)
            h.profile(True)
            h.round()
            stats = h.profile_read()
            h.profile(False)
            assert "fwd1_block_gemm" in stats and ("gram" in stats) == (c["K1"] > 1), stats
            if B > 32:
                assert ("head_fused" if c["C"] <= 32 else "b1_step") in stats, stats
            prob = replace(prob, B=B)
            M.hieravg_round(prob, st)
            assert np.array_equal(h.last_indices().astype(np.int64), st.last_indices)
            ok, det = cases.parity_report(prob, h.params(), st.W)
            assert ok, (B, det)


@pytest.mark.parametrize("mode", ["delayed", "eager"])
@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_units_of_any_magnitude(mode, momentum, gpu_lib):
    """Rows of W1 scaled by 10^-12 .. 10^12 (their W2 columns by the inverse,
    so the logits stay ordinary): every unit keeps its own relative accuracy."""
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 4, 2, 2, 2, B=16, IN=200, H=96, C=5, N=300, sigma=0.5, lr=1e-3, momentum=momentum, seed=211)
    prob = cases.oracle_problem(c)
    scale = 10.0 ** np.linspace(-12, 12, prob.H)
    st = M.create(prob)
    for p in range(prob.P):
        b = M.unpack(prob, st.W[p])
        b["W1"] *= scale[:, None]
        b["W2"] /= scale[None, :]
    st.W[:] = st.W.astype(np.float32).astype(np.float64)
    print(f"[gpu case] {mode} {c}", flush=True)
    with HierAvg(config=cases.native_config(c, mode)) as h:
        h.set_params(st.W.astype(np.float32))
        h.round()
        got = [h.params()] + ([h.momentum()] if momentum else [])
    M.hieravg_round(prob, st)
    for arr, want in zip(got, (st.W, st.V)):  # every unit's parameters, and its row of every learner's buffer
        for p in range(prob.P):
            g, w = M.unpack(prob, arr[p].astype(np.float64)), M.unpack(prob, want[p])
            err, size = np.abs(g["W1"] - w["W1"]).max(axis=1), np.abs(w["W1"]).max(axis=1)
            assert (err <= TOL * size).all(), np.flatnonzero(~(err <= TOL * size))


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_weights_stay_visible(value, gpu_lib):
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 4, 2, 2, 2, B=16, IN=200, H=96, C=5, N=300, sigma=0.5, lr=1e-3, seed=212)
    print(f"[gpu case] {value} {c}", flush=True)
    with HierAvg(config=cases.native_config(c, "delayed")) as h:
        w = h.params()
        w[:, 200 * 7 + 3] = value
        h.set_params(w)
        assert not h.finite()
        assert not np.isfinite(h.evaluate(0, 0, 64)[0])
        h.round()
        assert not h.finite()


@pytest.mark.parametrize("rows,H", [(2032, 100), (2033, 100), (4096, 100), (4097, 100), (4096, 512), (4090, 300)])
def test_evaluate_around_the_measured_form(rows, H, gpu_lib):
    """Chunks of 2048 padded rows and more take W1's rows as two parts, in 128-
    or 256-column tiles; ragged widths, rows of W1 of very different magnitudes."""
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 2, 1, 1, 1, B=16, IN=101, H=H, C=7, N=4200, sigma=0.5, lr=0.05, seed=231)
    prob = cases.oracle_problem(c)
    st = M.create(prob)
    scale = 10.0 ** np.linspace(-6, 6, prob.H)
    for p in range(prob.P):
        b = M.unpack(prob, st.W[p])
        b["W1"] *= scale[:, None]
        b["W2"] /= scale[None, :]
    w = st.W.astype(np.float32)
    print(f"[gpu case] evaluate {rows}", flush=True)
    with HierAvg(config=cases.native_config(c)) as h:
        h.set_params(w)
        for split in (0, 1):
            loss, correct = h.evaluate(1, split, rows)
            want, wc, gaps = M.evaluate(prob, w[1].astype(np.float64), np.arange(rows), split)
            assert abs(loss - want) <= TOL * max(1.0, abs(want)), (loss, want)
            assert abs(correct - wc) <= int(np.sum(gaps < 1e-5)), (correct, wc)


def test_heavy_ball_block_end_rounds_the_parameters_once(gpu_lib):
    """A heavy-ball block end adds the buffer's and the errors' share to the
    block-start parameters.  The share is far below the parameters here (about
    2^-9 of them), so its own rounding does not count, and n block ends leave
    n roundings: errors of variance n/12 in units in the last place of the
    parameter.  A second rounding per block end would give 2n/12; the line is
    halfway.  One learner (means are exact), no decay (the base's coefficient
    is exactly 1); the median over the hidden units keeps out units with a
    ReLU decision at rounding."""
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 1, 1, 4, 8, B=16, IN=256, H=64, C=5, N=300, sigma=0.5, momentum=0.875, lr=2.0 ** -14, seed=213)
    prob = cases.oracle_problem(c)
    st = M.create(prob)
    print(f"[gpu case] {c}", flush=True)
    with HierAvg(config=cases.native_config(c, "delayed")) as h:
        for _ in range(2):
            h.round()
            M.hieravg_round(prob, st)
        got = M.unpack(prob, h.params()[0].astype(np.float64))["W1"]
    want = M.unpack(prob, st.W[0])["W1"]
    ulps = (got - want) / np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
    rms = np.sqrt(np.median((ulps ** 2).mean(axis=1)))
    n = 2 * c["K2"]
    print("rms", rms, "one rounding", np.sqrt(n / 12), flush=True)
    assert rms <= np.sqrt(1.5 * n / 12), rms


@pytest.mark.parametrize("c,B", [
    # K1 * S * B = 15776 rows at 116 samples: delayed; 17408 at the padded 128 and at create's B: not
    (cases.case("mlp", 17, 17, 8, 1, B=128, IN=600, H=1000, C=10, N=500, sigma=0.5, lr=0.02, seed=214), 116),
    # the same up to 32 samples: 12000 rows at 20, 19200 at the padded 32
    (cases.case("mlp", 75, 75, 8, 1, B=32, IN=200, H=510, C=3, N=500, sigma=0.5, lr=0.02, seed=215), 20),
], ids=["wide", "narrow"])
def test_set_batch_into_the_delayed_schedule(c, B, gpu_lib):
    """A minibatch whose round is delayed on a handle whose create-time and
    padded minibatches are not: its buffers hold the padded rows."""
    from paper_1903_05133_amd import HierAvg
    from dataclasses import replace
    prob = replace(cases.oracle_problem(c), B=B)
    st = M.create(prob)
    print(f"[gpu case] set_batch {B} {c}", flush=True)
    with HierAvg(config=cases.native_config(c)) as h:
        h.set_batch(B)
        h.profile(True)
        h.round()
        assert "fwd1_block_gemm" in h.profile_read()
        M.hieravg_round(prob, st)
        ok, det = cases.parity_report(prob, h.params(), st.W)
        assert ok, det


@pytest.mark.parametrize("C", [5, 40])
def test_buffers_of_learners_with_errors_of_any_magnitude(C, gpu_lib):
    """One cluster whose second learner's W2, and with it its hidden errors, is
    2^-36 of the first's: its own buffer of W1 keeps its relative accuracy (the
    parity tolerance by learner; sums of at most 32 terms), whatever the
    cluster's other errors are.  The step size leaves the parameters alone."""
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 3, 3, 2, 1, B=16, IN=130, H=96, C=C, N=300, sigma=0.5, lr=1e-30, momentum=0.875, seed=216)
    prob = cases.oracle_problem(c)
    st = M.create(prob)
    M.unpack(prob, st.W[1])["W2"][:] *= 2.0 ** -36
    print(f"[gpu case] {c}", flush=True)
    with HierAvg(config=cases.native_config(c, "delayed")) as h:
        h.set_params(st.W.astype(np.float32))
        h.profile(True)
        h.round()
        assert "buffer_update_gemm" in h.profile_read()
        got = h.momentum()
    M.hieravg_round(prob, st)
    for p in range(prob.P):
        g, w = M.unpack(prob, got[p].astype(np.float64))["W1"], M.unpack(prob, st.V[p])["W1"]
        err = np.abs(g - w).max() / np.abs(w).max()
        print("learner", p, "max", np.abs(w).max(), "error", err, flush=True)
        assert err <= TOL, (p, err)


@pytest.mark.parametrize("momentum", [0.0, 0.9])
def test_resume_is_exact_where_scales_lie_at_a_power_of_two(momentum, gpu_lib, tmp_path):
    """Units whose largest weight is just below 1: in a cluster's copy it may
    pass 1, in the mean of the copies not.  A running handle takes the next
    round's scale (an exponent) from the mean, as a handle that resumes from
    it does; the low bits of the other, tiny weights depend on it."""
    from paper_1903_05133_amd import HierAvg
    c = cases.case("mlp", 8, 2, 2, 2, B=32, IN=200, H=512, C=10, N=300, sigma=0.5, lr=0.05, momentum=momentum, seed=217)
    cfg = cases.native_config(c, "delayed")
    rng = np.random.default_rng(7)
    print(f"[gpu case] {c}", flush=True)
    with HierAvg(config=cfg) as h, HierAvg(config=cfg) as h2:
        w = h.params()
        W1 = (1e-7 * rng.standard_normal((c["H"], c["IN"]))).astype(np.float32)
        W1[:, 0] = 1.0 - 1e-4 * rng.random(c["H"])
        w[:, :W1.size] = W1.reshape(-1)
        h.set_params(w)
        for _ in range(4):
            h.round()
            h.save(str(tmp_path / "ck.npz"))
            h.round()
            h2.load(str(tmp_path / "ck.npz"))
            h2.round()
            assert np.array_equal(h2.params(), h.params())
            w = h.params()  # back to the power of two
            w[:, :W1.size] = W1.reshape(-1)
            h.set_params(w)


@pytest.mark.parametrize("P,B,C", [(1024, 32, 64), (512, 48, 64), (256, 80, 64), (256, 80, 192)],
                         ids=["32", "64", "128", "128x256"])
def test_three_part_forward_is_as_exact_as_a_float32_sum(P, B, C, gpu_lib):
    """Logits z_c = v x + e_c x whose large common share v x (about 1000) drops
    out of the softmax but sets the rounding of every logit, so that one step's
    bias gradient shows the logits' error, far above its own rounding.  It is at
    most that of a float32 sum that rounds once per four terms (the 16x16x4
    matrix instruction), computed here; with all six products rounding one sum
    it is above.  As many learners as leave one split of the features, so that
    both sum 512 terms in one run; forward tiles of 32, 64 and 128 rows."""
    from paper_1903_05133_amd import HierAvg
    from oracle import rng as R
    c = cases.case("softmax", P, 1, 1, 1, B=B, IN=512, C=C, N=400, sigma=0.5, lr=1e-30, momentum=0.5, seed=218)
    gen = np.random.default_rng(3)
    W = (gen.standard_normal((C, c["IN"])) + 1000.0 * gen.standard_normal(c["IN"])) / np.sqrt(c["IN"])
    W = W.astype(np.float32)
    row = np.concatenate([W.reshape(-1), np.zeros(C, np.float32)])
    print(f"[gpu case] {c}", flush=True)
    with HierAvg(config=cases.native_config(c)) as h:
        h.set_params(np.broadcast_to(row, (P, row.size)).copy())
        h.round()
        got = h.momentum()[:, -C:].astype(np.float64)
        idx = h.last_indices().reshape(P, B).astype(np.int64)
    X, y = R.data_rows(c["seed"], np.arange(c["N"]), c["IN"], C, c["sigma"])
    terms = [X[:, k:k + 4] @ W[:, k:k + 4].T.astype(np.float64) for k in range(0, c["IN"], 4)]
    z4 = np.zeros((c["N"], C), np.float32)
    for t in terms:
        z4 = (z4.astype(np.float64) + t).astype(np.float32)
    grad = lambda z: (M.softmax_probs(z) - np.eye(C)[y])[idx].mean(axis=1)  # noqa: E731
    want = grad(sum(terms))
    err, err4 = (np.sqrt(np.mean((g - want) ** 2)) for g in (got, grad(z4.astype(np.float64))))
    print("error", err, "of a float32 sum", err4, "ratio", err / err4, flush=True)
    assert err <= err4, (err, err4)


# (update mode, minibatch, hidden units, classes): the forward's forms and tiles
@pytest.mark.parametrize("mode,B,H,C", [("delayed", 16, 96, 5), ("delayed", 16, 300, 40), ("auto", 48, 512, 5),
                                        ("eager", 16, 96, 5), ("eager", 48, 96, 40), ("eager", 80, 300, 70)])
def test_an_infinite_weight_acts_as_in_float32(mode, B, H, C, gpu_lib):
    """A weight of -infinity at a feature that is positive in every row (five
    rows without noise: class means): the unit's pre-activations are -infinity,
    it is off for good, and every other parameter takes the steps of the oracle's
    run with a huge weight there."""
    from paper_1903_05133_amd import HierAvg
    from oracle import rng as R
    c = cases.case("mlp", 4, 2, 2, 2, B=B, IN=1100, H=H, C=C, N=5, sigma=0.0, lr=0.01, seed=219)
    X, _ = R.data_rows(c["seed"], np.arange(c["N"]), c["IN"], C, 0.0)
    prob = cases.oracle_problem(c)
    st = M.create(prob)
    k = 7 * c["IN"] + int(np.flatnonzero((X > 0.01).all(axis=0))[-1])
    st.W[:, k] = -np.inf
    print(f"[gpu case] infinite weight {mode} {c}", flush=True)
    with HierAvg(config=cases.native_config(c, mode)) as h:
        h.set_params(st.W.astype(np.float32))
        h.round()
        got = h.params()
    st.W[:, k] = -1e30  # as good as infinite (the oracle's 0 * weight of no decay is finite)
    M.hieravg_round(prob, st)
    assert (got[:, k] == -np.inf).all() and (np.isinf(got).sum(axis=1) == 1).all()
    got[:, k] = st.W[:, k] = 0.0
    ok, det = cases.parity_report(prob, got, st.W)
    assert ok, det


@pytest.mark.parametrize("rows", [64, 1500, 2100])
def test_evaluate_with_an_infinite_weight(rows, gpu_lib):
    """One weight of -infinity: its unit is off in the rows that are positive
    there, and in the others its logits are infinite, the first positively
    infinite one being the prediction."""
    from paper_1903_05133_amd import HierAvg
    from oracle import rng as R
    c = cases.case("mlp", 1, 1, 1, 1, B=16, IN=300, H=520, C=70, N=2100, sigma=0.5, lr=0.05, seed=220)
    prob = cases.oracle_problem(c)
    w = M.create(prob).W.astype(np.float32)
    w[0, 7 * c["IN"] + 3] = -np.inf
    X, y = R.data_rows(c["seed"], np.arange(rows), c["IN"], c["C"], c["sigma"])
    b = M.unpack(prob, w[0].astype(np.float64))
    z = np.maximum(X @ b["W1"].T + b["b1"], 0.0) @ b["W2"].T + b["b2"]
    assert not np.isnan(z).any() and np.isinf(z).any(axis=1).sum() > rows / 4
    print(f"[gpu case] infinite weight, evaluate {rows}", flush=True)
    with HierAvg(config=cases.native_config(c)) as h:
        h.set_params(w)
        _, correct = h.evaluate(0, 0, rows)
    assert abs(correct - int((z.argmax(axis=1) == y).sum())) <= 1  # (a near-tie of finite logits)


@pytest.mark.parametrize("momentum", [0.0, 0.5])
def test_an_infinite_error_acts_as_in_float32(momentum, gpu_lib):
    """One learner, one sample, one step: a unit just above zero whose weights
    of 3e38 in W2 make its error overflow to infinity; its row of W1 (and of
    its buffer) takes the infinities of error times input."""
    from paper_1903_05133_amd import HierAvg
    from oracle import rng as R
    c = cases.case("mlp", 1, 1, 1, 1, B=1, IN=64, H=64, C=2, N=9, sigma=0.5, lr=0.5, momentum=momentum, seed=221)
    prob = cases.oracle_problem(c)
    row = int(R.draw_indices(c["seed"], 0, 0, 1, c["N"])[0])
    X, y = R.data_rows(c["seed"], np.array([row]), c["IN"], c["C"], c["sigma"])
    w = M.create(prob).W.astype(np.float32)
    b = M.unpack(prob, w[0])
    b["W1"][7] = 0.0
    b["b1"][7] = 1e-30
    b["W2"][:, 7] = 3e38
    b["W2"][y[0], 7] = -3e38  # the label's logit is the lowest: error 3e38 + 3e38
    print(f"[gpu case] infinite error {c}", flush=True)
    with HierAvg(config=cases.native_config(c, "delayed")) as h:
        h.set_params(w)
        h.round()
        got = M.unpack(prob, h.params()[0])["W1"]
        buf = M.unpack(prob, h.momentum()[0])["W1"] if momentum else None
    want = np.where(X[0] > 0, -np.inf, np.inf)
    assert np.array_equal(got[7], want) and np.isfinite(np.delete(got, 7, axis=0)).all()
    if momentum:
        assert np.array_equal(buf[7], -want)


def test_no_memory_for_the_wide_schedule_leaves_eager_rounds(gpu_lib, monkeypatch):
    """AUTO with 64 samples: an allocation that fails (by the debug hook) leaves a
    handle of eager rounds, whose smaller minibatches stay delayed."""
    from dataclasses import replace
    from paper_1903_05133_amd import HierAvg
    c, _ = TILES["wide_64"]
    n = 2  # (the first one comes before the schedule is known: the create fails)
    print(f"[gpu case] no memory {c}", flush=True)
    while True:  # allocations of a whole create
        monkeypatch.setenv("HIERAVG_FAIL_ALLOC", str(n))
        with HierAvg(config=cases.native_config(c)) as h:
            h.profile(True)
            h.round()
            if "fwd1_block_gemm" in h.profile_read():
                break
        n += 1
    assert n > 10
    for fail in (2, n - 10, n - 1):
        monkeypatch.setenv("HIERAVG_FAIL_ALLOC", str(fail))
        prob = cases.oracle_problem(c)
        st = M.create(prob)
        with HierAvg(config=cases.native_config(c)) as h:
            for B, delayed in ((64, False), (20, True)):
                prob = replace(prob, B=B)
                h.set_batch(B)
                h.profile(True)
                h.round()
                assert ("fwd1_block_gemm" in h.profile_read()) == delayed
                h.profile(False)
                M.hieravg_round(prob, st)
                ok, det = cases.parity_report(prob, h.params(), st.W)
                assert ok, det
